"""Sliced rows, band tiles in FP32 with a window of more than 32,768 rows: the top
bit of a 16-bit column, which marks an entry outside the window, would be a column
of the window there, so such tiles have 32-bit columns.  206 chains of 70,000 states
get two tiles each, of 35,008 rows and a band of 50 states to either side.

A row's entries are added in column order by fused multiply-adds, as one lane per row
adds them, so the sweeps of one FP32 inner solve are those of schedule 1 bit for bit."""
import numpy as np
import pytest

import chaingen as cg
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu

N, K = 70_000, 206


def _chain():
    """Rows of three targets: one below, one above within 50 states, the third above
    too or, for 2% of the rows, anywhere; every 25th row reaches the goal (0) or sink (1)."""
    rng = np.random.Generator(np.random.PCG64(31))
    i = np.arange(2, N)
    off = np.stack([-rng.integers(1, 26, N - 2), rng.integers(1, 26, N - 2),
                    np.where(rng.random(N - 2) < 0.02, rng.integers(60, N - 62, N - 2), rng.integers(26, 51, N - 2))], 1)
    t = (i[:, None] - 2 + off) % (N - 2) + 2
    t[::25, 1] = 0
    t[12::25, 1] = 1
    t.sort(axis=1)
    w = rng.random(t.shape) + 0.1
    ptr = np.concatenate([[0, 1], 2 + 3 * np.arange(N - 1)]).astype(np.int32)
    goal = np.zeros(N, dtype=np.uint8)
    goal[0] = 1
    return cg.Chain(N, ptr, np.concatenate([[0, 1], t.ravel()]).astype(np.int32),
                    np.concatenate([[1.0, 1.0], (w / w.sum(1, keepdims=True)).ravel()]), goal, np.array([0, N], np.int64), "band")


def test_fp32_sweeps_are_those_of_one_lane_per_row():
    c = cg.concat([_chain()] * K, name="wide bands")
    G.banner(f"wide band: n={c.n} nnz={c.nnz}")
    sys = G.precompute(c)[0]
    for max_iter in (1, 30):
        kw = dict(tol=1e-300, stop=rp.RP_STOP_RESIDUAL, precision=rp.RP_FP32_REFINED, max_iter=max_iter)
        x0, i0, _ = G.solve(sys, "jacobi", schedule=0, **kw)
        x1, i1, _ = G.solve(sys, "jacobi", schedule=1, **kw)
        assert i0[0]["lanes"] == 0 and i0[0]["iterations"] == i1[0]["iterations"] == max_iter
        assert np.array_equal(x0, x1)
