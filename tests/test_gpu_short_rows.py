"""Sliced rows (schedule 0): how a wavefront takes its slices.  Sets with at most
two slices per wavefront on average, sets of narrow slices (FP64: with a band) and
the others run kernels of their own; the batches below lie on either side of each
line, with whole windows and with a band, in FP64 and in FP32.

A row's entries are added in column order by fused multiply-adds in every one, as
one lane per row adds them, so Jacobi iterates and counts are those of schedule 1
bit for bit; BiCGStab solves are held to 1e-10, the certificate's own bound."""
import numpy as np
import pytest

import chaingen as cg
import oracle
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu

SEED = cg.SEED_BASE + 1700


def _band(n, degree, seed):
    """Coin flips of `degree` outcomes within 50 states, 2% anywhere; goal 0, sink 1."""
    rng = np.random.Generator(np.random.PCG64(seed))
    i = np.arange(2, n).repeat(degree).reshape(-1, degree)
    t = np.clip(i + rng.integers(-50, 51, i.shape), 2, n - 1)
    t = np.where(rng.random(i.shape) < 0.02, rng.integers(2, n, i.shape), t)
    t[::25, -1] = 0
    t[13::25, -1] = 1
    rows = [np.unique(r) for r in t]
    ptr = np.concatenate([[0, 1, 2], 2 + np.cumsum([len(r) for r in rows])]).astype(np.int32)
    val = np.concatenate([[1.0, 1.0]] + [np.full(len(r), 1.0 / len(r)) for r in rows])
    goal = np.zeros(n, dtype=np.uint8)
    goal[0] = 1
    return cg.Chain(n, ptr, np.concatenate([[0], [1]] + rows).astype(np.int32), val, goal, np.array([0, n], np.int64), "band")


def _whole(k, n, dmax):
    return lambda: cg.concat([cg.random_sparse(n - 3 * i, 1, dmax, 0.02, 0.02, seed=SEED + i) for i in range(k)])


SHAPES = {
    "whole, few, narrow": _whole(4, 16_001, 4),
    "whole, few, wide": _whole(4, 12_007, 13),
    "whole, many, narrow": _whole(90, 17_557, 4),
    "whole, many, wide": _whole(80, 17_557, 9),
    "band, few": lambda: _band(70_001, 3, 1),
    "band, on the line": lambda: _band(524_290, 2, 2),
    "band, many": lambda: _band(1_100_003, 2, 3),
}


@pytest.fixture(scope="module", params=list(SHAPES))
def case(request):
    c = SHAPES[request.param]()
    G.banner(f"short rows: {request.param}, n={c.n} nnz={c.nnz}")
    return c, G.precompute(c)[0]


@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
def test_jacobi_iterates_are_those_of_one_lane_per_row(case, precision):
    c, sys = case
    kw = dict(tol=1e-300, stop=rp.RP_STOP_RESIDUAL, precision=precision, max_iter=41)
    x0, i0, _ = G.solve(sys, "jacobi", schedule=0, **kw)
    x1, i1, _ = G.solve(sys, "jacobi", schedule=1, **kw)
    assert i0[0]["lanes"] == 0 and [i["iterations"] for i in i0] == [i["iterations"] for i in i1]
    assert np.array_equal(x0, x1)


@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
def test_bicgstab_matches_oracle(case, precision):
    c, sys = case
    x, info, code = G.solve(sys, "bicgstab", schedule=0, tol=1e-10, stop=rp.RP_STOP_CERTIFIED, precision=precision)
    assert code == rp.binding.RP_OK
    k = c.num_instances - 1
    ck = c.instance(k)
    ref = oracle.solve(ck.n, ck.rp, ck.col, ck.val, ck.goal, "bicgstab", tol=1e-12, stop_mode=1)
    assert np.abs(x[int(c.inst_off[k]):int(c.inst_off[k + 1])] - ref.x).max() <= 1e-10
