"""A starting point that is not finite in one state: the value spreads along the
transitions to that state and no further, in every row layout.  One sweep under the
paper's rule from x0 = 1 with an infinity or NaN in the first state of the window, on
rows of 1 to 300 entries: the rows it reaches are those of a product with the matrix in
numpy, the same under 1 to 64 lanes per row, and all other values are finite."""
import numpy as np
import pytest
import torch

import chaingen as cg
import oracle
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    rng = np.random.Generator(np.random.PCG64(77))
    n = 6_000
    ptr, cols, vals = [0, 1, 2], [[0], [1]], [[1.0], [1.0]]
    for i in range(2, n):
        k = (1, 2, 3, 129, 300)[i % 5]
        c = np.sort(rng.choice(np.arange(3, n), size=k, replace=False))
        if i % 11 == 0:
            c = np.concatenate([[2], c])  # state 2 is the first row of the reduced system
        c = np.concatenate([[0, 1], c])
        w = rng.random(len(c)) + 0.1
        cols.append(c)
        vals.append(w / w.sum())
        ptr.append(ptr[-1] + len(c))
    goal = np.zeros(n, dtype=np.uint8)
    goal[0] = 1
    c = cg.Chain(n, np.array(ptr, np.int32), np.concatenate(cols).astype(np.int32), np.concatenate(vals), goal,
                 np.array([0, n], np.int64), "start")
    sys, cls, _ = G.precompute(c)
    assert cls[2] == oracle.SQ and cls[0] != oracle.SQ and cls[1] != oracle.SQ
    rows = np.arange(n).repeat(np.diff(c.rp))
    reached = np.zeros(n, dtype=bool)
    reached[rows[(c.col == 2) & (cls[rows] == oracle.SQ) & (rows != 2)]] = True
    return c, sys, reached


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("schedule", [1, 2, 8, 32, 64])
def test_spreads_along_transitions_only(case, schedule, bad):
    c, sys, reached = case
    G.banner(f"non-finite start: schedule {schedule}, {bad}")
    x0 = torch.ones(c.n, dtype=torch.float64, device="cuda")
    x0[2] = bad
    x, info, code = G.solve(sys, "jacobi", tol=1e-10, stop=rp.RP_STOP_DELTA, max_iter=1, schedule=schedule, x0=x0)
    assert code == rp.binding.RP_ERR_NONFINITE and info[0]["lanes"] == schedule
    assert np.array_equal(~np.isfinite(x), reached)
