"""Sliced rows (schedule 0): the compact forms of a slice.  Band tiles keep
16-bit columns and gather their entries outside the window through the slice's
list; a slice with more than 64 of them turns its tile to 32-bit columns; FP64
values that are all exact in FP32 are held so; diagonals of 1 are not read;
slices of few entries (up to four on average) take a kernel of their own.

A row's entries are added in column order by fused multiply-adds in every form,
as one lane per row adds them, so Jacobi iterates and counts are those of
schedule 1 bit for bit.  Solves and the adjoint are held to the oracle within
1e-10, the certificate's own bound."""
import numpy as np
import pytest
import torch

import chaingen as cg
import oracle
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu


def _graph(n, degrees, step, far, exact, lazy, seed, cluster=()):
    """States 2.. with degrees[i % len] targets within `step` (a share `far` of
    them, and all of the states in `cluster`, anywhere), a self-loop on every
    third state if lazy; each state goes to the goal (0) or the sink (1) now and
    then.  exact: coin flips, else random weights."""
    rng = np.random.Generator(np.random.PCG64(seed))
    ptr, cols, vals = [0, 1, 2], [[0], [1]], [[1.0], [1.0]]
    for i in range(2, n):
        k = degrees[i % len(degrees)]
        anywhere = rng.random(k) < (1.0 if cluster and cluster[0] <= i < cluster[1] else far)
        t = np.where(anywhere, rng.integers(2, n, k), np.clip(i + rng.integers(-step, step + 1, k), 2, n - 1))
        if lazy and i % 3 == 0:
            t[0] = i
        if i % 20 == 0:
            t[-1] = 0 if i % 40 == 0 else 1
        t = np.unique(t if lazy else np.where(t == i, 0, t))
        k = len(t)
        if exact:
            w = np.full(k, 0.5 ** (k - 1))
            w[:k - 1] = 0.5 ** np.arange(1, k)
            w = rng.permutation(w)
        else:
            w = rng.random(k) + 0.1
            w = w / w.sum()
        cols.append(t)
        vals.append(w)
        ptr.append(ptr[-1] + k)
    goal = np.zeros(n, dtype=np.uint8)
    goal[0] = 1
    return cg.Chain(n, np.array(ptr, np.int32), np.concatenate(cols).astype(np.int32), np.concatenate(vals), goal,
                    np.array([0, n], np.int64), "slices")


SHAPES = {
    "coin flips": lambda: _graph(50_003, (2, 3, 4), 64, 0.02, True, False, 11),
    "wide tiles": lambda: _graph(50_003, (2, 3, 4), 64, 0.02, True, False, 12, cluster=(20_000, 20_500)),
    "self-loops": lambda: _graph(50_003, (1, 2, 3, 4), 64, 0.02, False, True, 13),
    "broad": lambda: _graph(30_003, (5, 9, 16), 100, 0.01, False, True, 14),
    "broad, exact": lambda: _graph(9_001, (5, 9, 16), 100, 0.01, True, False, 15),
    "whole": lambda: _graph(3_001, (1, 2, 3), 3_000, 0.0, False, True, 16),
    "tiny": lambda: _graph(70, (1, 2, 3, 4), 70, 0.0, True, False, 17),
}


@pytest.fixture(scope="module", params=list(SHAPES))
def case(request):
    c = SHAPES[request.param]()
    G.banner(f"slices: {request.param}, n={c.n} nnz={c.nnz}")
    ref = oracle.solve(c.n, c.rp, c.col, c.val, c.goal, "bicgstab", tol=1e-12, stop_mode=1)
    sq = np.nonzero(ref.cls == oracle.SQ)[0]
    seed, lam = np.zeros(c.n), np.zeros(c.n)
    seed[sq[:: max(1, len(sq) // 7)]] = 1.0
    lam_o, _, _, rc = oracle.adjoint(ref, seed, tol=1e-12)
    lam[sq] = lam_o[ref.red.map[sq]]
    return c, G.precompute(c)[0], ref, seed, lam


@pytest.mark.parametrize("max_iter", [1, 2, 40])
@pytest.mark.parametrize("stop, precision", [(rp.RP_STOP_DELTA, rp.RP_FP64), (rp.RP_STOP_RESIDUAL, rp.RP_FP64),
                                             (rp.RP_STOP_RESIDUAL, rp.RP_FP32_REFINED)])
def test_jacobi_iterates_are_those_of_one_lane_per_row(case, stop, precision, max_iter):
    c, sys, *_ = case
    kw = dict(tol=1e-300, stop=stop, precision=precision, max_iter=max_iter)
    x0, i0, _ = G.solve(sys, "jacobi", schedule=0, **kw)
    x1, i1, _ = G.solve(sys, "jacobi", schedule=1, **kw)
    assert i0[0]["lanes"] == 0 and i0[0]["iterations"] == i1[0]["iterations"]
    assert np.array_equal(x0, x1)


@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
def test_solves_and_adjoint_match_oracle(case, precision):
    c, sys, ref, seed, want = case
    kw = dict(tol=1e-10, stop=rp.RP_STOP_CERTIFIED, precision=precision, schedule=0)
    for method in ("jacobi", "bicgstab"):
        x, info, code = G.solve(sys, method, **kw)
        assert code == rp.binding.RP_OK
        assert np.abs(x - ref.x).max() <= 1e-10, method
    lam, g, info, code = rp.rp_adjoint(G.ctx(), sys, torch.from_numpy(x).cuda(), torch.from_numpy(seed).cuda(), 1, **kw)
    assert code == rp.binding.RP_OK
    assert np.abs(lam.cpu().numpy() - want).max() <= 1e-10 * max(1.0, np.abs(want).max())
