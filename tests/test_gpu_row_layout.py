"""Laying a system out: the row counts and rows read one run of 8 entries at a
time where rows are short and four where their mean length is 12 or more.  Chains
with rows around the lengths of one run, four runs and more, on either side of
that line, with self-loops, transitions into S_{=1} and S_{=0} and stored zeros of
probability, and a general system with entries of both signs.

Bar: the reduced system equals the oracle's exactly (same order, same sums)."""
import numpy as np
import pytest
import torch

import chaingen as cg
import oracle
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu

LENGTHS = {
    "short": (1, 2, 7, 8, 9, 3, 16, 17),           # mean 7.9
    "below the line": (11, 11, 12, 11),            # 11.2
    "on the line": (12, 12, 12, 13),               # 12.2
    "long": (7, 8, 9, 31, 32, 33, 63, 64, 65, 1),
}


def _chain(lengths, n=3_001, seed=5):
    """State 0: goal; 1: sink; 2: certain to reach the goal; the others have rows of
    `lengths` transitions, the first few to 0..2 now and then, self-loops on every
    fifth state, one stored zero on every seventh."""
    rng = np.random.Generator(np.random.PCG64(seed))
    ptr, cols, vals = [0, 1, 2, 3], [[0], [1], [0]], [[1.0]] * 3
    for i in range(3, n):
        k = lengths[i % len(lengths)]
        c = set(rng.choice(np.arange(3, n), size=k, replace=False).tolist())
        if i % 4 == 0:
            c = set(list(c)[1:]) | {int(rng.integers(0, 3))}
        if i % 5 == 0 and k > 2:
            c = set(list(c)[1:]) | {i}
        c = np.array(sorted(c | ({0} if k == 1 and i % 2 else set())))
        w = rng.random(len(c)) + 0.1
        if i % 7 == 0 and len(c) > 3:
            w[len(c) // 2] = 0.0
        cols.append(c)
        vals.append(w / w.sum())
        ptr.append(ptr[-1] + len(c))
    goal = np.zeros(n, dtype=np.uint8)
    goal[0] = 1
    return cg.Chain(n, np.array(ptr, np.int32), np.concatenate(cols).astype(np.int32), np.concatenate(vals), goal,
                    np.array([0, n], np.int64), "layout")


@pytest.mark.parametrize("lengths", list(LENGTHS))
def test_reduced_system_is_the_oracles(lengths):
    c = _chain(LENGTHS[lengths])
    G.banner(f"row layout: {lengths}, mean {c.nnz / c.n:.2f}")
    sys, cls, _ = G.precompute(c)
    red = oracle.assemble(c.n, c.rp, c.col, c.val, cls)
    got = [t.cpu().numpy() for t in rp.rp_system_export(G.ctx(), sys)]
    for name, a, b in zip(("rows", "columns", "values", "diagonal", "right-hand side"), got,
                          (red.arp, red.acol, red.aval, red.d, red.b)):
        assert np.array_equal(a, b), name


@pytest.mark.parametrize("lengths", list(LENGTHS))
def test_general_system_is_the_oracles(lengths):
    c = _chain(LENGTHS[lengths], n=901, seed=6)
    G.banner(f"row layout, general: {lengths}")
    rng = np.random.Generator(np.random.PCG64(7))
    a = np.zeros((c.n, c.n))
    a[np.arange(c.n).repeat(np.diff(c.rp)), c.col] = rng.standard_normal(c.nnz)
    np.fill_diagonal(a, 0.0)
    np.fill_diagonal(a, np.abs(a).sum(1) + 1.0)
    rows, cols = np.nonzero(a)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=c.n))]).astype(np.int32)
    val, rhs = a[rows, cols], rng.standard_normal(c.n)
    dev = [torch.from_numpy(v).cuda() for v in (ptr, cols.astype(np.int32), val, rhs)]
    sys = rp.rp_matrix_system(G.ctx(), *dev, [0, c.n])
    red = oracle.matrix_system(c.n, ptr, cols.astype(np.int32), val, rhs)
    got = [t.cpu().numpy() for t in rp.rp_system_export(G.ctx(), sys)]
    for name, x, y in zip(("rows", "columns", "values", "diagonal", "right-hand side"), got,
                          (red.arp, red.acol, red.aval, red.d, red.b)):
        assert np.array_equal(x, y), name
