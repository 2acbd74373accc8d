"""Cells: the layout the default schedule takes for batches whose chains are
mostly too large for one LDS window and have no band.  The batch below is one
by the library's rule (its modelled sweep is well under the gathers'): chains
of 60,000 states beside small ones, whose tiles end on odd rows, with self-loops
(a diagonal other than 1), a single undecided state, and one with none.

A row's entries are added in column order by fused multiply-adds, as one lane
per row adds them, so the Jacobi iterates and counts are those of schedule 1
bit for bit: under the paper's rule and the certified stop in FP64, also as
graph replays, and over the sweeps of one FP32 inner solve.  (A whole
FP32-refined solve also holds FP64 residuals, whose last bit differs between
the layouts where a diagonal is not 1.)  BiCGStab, the FP32-refined solves and
the adjoint are held to the oracle within 1e-10, the certificate's own bound."""
import numpy as np
import pytest
import torch

import chaingen as cg
import oracle
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu

SEED = cg.SEED_BASE + 900


@pytest.fixture(scope="module")
def batch():
    parts = [cg.random_sparse(60_000 - 37 * i, 1, 8, 0.01, 0.01, seed=SEED + i) for i in range(14)]
    parts += [cg.random_sparse(700, 1, 16, 0.02, 0.02, seed=SEED + 50), cg.from_dense([[0.5, 0.3, 0.2], [0, 1, 0], [0, 0, 1]], [1]),
              cg.from_dense([[0.5, 0.5], [0, 1]], [1]), cg.random_sparse(20_483, 1, 3, 0.05, 0.05, seed=SEED + 51)]
    c = cg.concat(parts, name="cells")
    G.banner(f"cells: n={c.n} nnz={c.nnz}")
    sys, cls, _ = G.precompute(c)
    refs = {k: oracle.solve(parts[k].n, parts[k].rp, parts[k].col, parts[k].val, parts[k].goal, "bicgstab", tol=1e-12,
                            stop_mode=1) for k in (0, 13, 14, 15, 16, 17)}
    return c, parts, sys, cls, refs


@pytest.mark.parametrize("max_iter", [1, 2, 60])
def test_jacobi_iterates_are_those_of_one_lane_per_row(batch, max_iter):
    c, parts, sys, cls, refs = batch
    kw = dict(tol=1e-300, stop=rp.RP_STOP_DELTA, max_iter=max_iter)
    x0, i0, _ = G.solve(sys, "jacobi", **kw)
    x1, i1, _ = G.solve(sys, "jacobi", schedule=1, **kw)
    assert all(i["lanes"] == 0 and i["panels"] == 0 for i in i0)
    assert [i["iterations"] for i in i0] == [i["iterations"] for i in i1]
    assert np.array_equal(x0, x1)


@pytest.mark.parametrize("max_iter", [1, 2, 50])
def test_fp32_inner_sweeps_are_those_of_one_lane_per_row(batch, max_iter):
    c, parts, sys, cls, refs = batch
    kw = dict(tol=1e-300, stop=rp.RP_STOP_RESIDUAL, precision=rp.RP_FP32_REFINED, max_iter=max_iter)
    x0, i0, _ = G.solve(sys, "jacobi", **kw)
    x1, i1, _ = G.solve(sys, "jacobi", schedule=1, **kw)
    assert [i["iterations"] for i in i0] == [i["iterations"] for i in i1]
    assert np.array_equal(x0, x1)


@pytest.mark.parametrize("graph", [0, 1])
def test_certified_fp64_jacobi_is_that_of_one_lane_per_row(batch, graph):
    c, parts, sys, cls, refs = batch
    kw = dict(tol=1e-10, stop=rp.RP_STOP_CERTIFIED)
    x0, i0, code0 = G.solve(sys, "jacobi", graph=graph, **kw)
    x1, i1, code1 = G.solve(sys, "jacobi", schedule=1, **kw)
    assert code0 == code1 == rp.binding.RP_OK
    assert [i["iterations"] for i in i0] == [i["iterations"] for i in i1]
    assert np.array_equal(x0, x1)


@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
def test_solves_and_adjoint_match_oracle(batch, precision):
    c, parts, sys, cls, refs = batch
    kw = dict(tol=1e-10, stop=rp.RP_STOP_CERTIFIED, precision=precision)
    x, info, code = G.solve(sys, "jacobi", **kw)
    assert code == rp.binding.RP_OK
    for k, ref in refs.items():
        assert np.abs(x[c.inst_off[k]:c.inst_off[k + 1]] - ref.x).max() <= 1e-10, k
    x, info, code = G.solve(sys, "bicgstab", **kw)
    assert code == rp.binding.RP_OK
    seed = np.zeros(c.n)
    for k, ref in refs.items():
        lo, hi = c.inst_off[k], c.inst_off[k + 1]
        assert np.abs(x[lo:hi] - ref.x).max() <= 1e-10, k
        if (ref.cls == oracle.SQ).any():
            seed[lo + np.nonzero(ref.cls == oracle.SQ)[0][0]] = 1.0
    lam, g, info, code = rp.rp_adjoint(G.ctx(), sys, torch.from_numpy(x).cuda(), torch.from_numpy(seed).cuda(), 1, **kw)
    assert code == rp.binding.RP_OK
    lam = lam.cpu().numpy()
    for k, ref in refs.items():
        lo, hi = c.inst_off[k], c.inst_off[k + 1]
        sq = np.nonzero(ref.cls == oracle.SQ)[0]
        if sq.size == 0:
            continue
        lam_o, _, _, rc = oracle.adjoint(ref, seed[lo:hi], tol=1e-12)
        want = np.zeros(hi - lo)
        want[sq] = lam_o[ref.red.map[sq]]
        assert np.abs(lam[lo:hi] - want).max() <= 1e-10 * max(1.0, np.abs(lam_o).max()), k
