"""Backward searches on both sides of the size from which the first pull steps
run over the whole GPU (4,096 states) and of the one-workgroup limit (32,768):
a path that needs one step per state, and a random chain that needs a few.
Classes are the oracle's, exactly."""
import numpy as np
import pytest

import chaingen as cg
import oracle
from tests import _gpu as G

pytestmark = pytest.mark.gpu


def _path(n):
    """State i steps to i+1; the last one is the goal; every 97th state may also
    fall into a sink behind it."""
    ptr, col, val = [0], [], []
    for i in range(n):
        if i == 0 or i == n - 1:
            col.append(i)
            val.append(1.0)
        elif i % 97 == 0:
            col += [0, i + 1]
            val += [0.5, 0.5]
        else:
            col.append(i + 1)
            val.append(1.0)
        ptr.append(len(col))
    goal = np.zeros(n, np.uint8)
    goal[n - 1] = 1
    return cg.Chain(n, np.array(ptr, np.int32), np.array(col, np.int32), np.array(val), goal,
                    np.array([0, n], np.int64), "path")


@pytest.mark.parametrize("n", [4_095, 4_096, 4_097, 32_768, 32_769])
@pytest.mark.parametrize("kind", ["path", "random"])
def test_classes_match_oracle(kind, n):
    c = _path(n) if kind == "path" else cg.random_sparse(n, 1, 4, 0.01, 0.05, seed=cg.SEED_BASE + n)
    G.banner(f"reach: {kind}, n={n}")
    _, cls, _ = G.precompute(c)
    ref = oracle.solve(c.n, c.rp, c.col, c.val, c.goal, "bicgstab", tol=1e-6, stop_mode=1)
    assert np.array_equal(cls, ref.cls)
