"""The tail of a solve whose sweeps run on cells: chains of 60,000 states that mix
fast, on cells, beside small ones that mix slowly, short and long rows, whose last
sweeps run resident on slices built for them alone.

Bars: graph replays (which never switch) are the reference, bit for bit in the
iterates and equal in the sweep counts, in FP64 and in FP32 inside FP64
refinement, forward and transposed; under the paper's rule (no FP64 residuals, whose
last bit depends on the layout) one lane per row is.  The profile counters show that the tail ran resident; the first and last small chains
are held to the oracle within 1e-10, the certificate's own bound."""
import numpy as np
import pytest
import torch

import chaingen as cg
import oracle
import paper_1210_6412_amd as rp
from paper_1210_6412_amd import binding as B
from tests import _gpu as G

pytestmark = pytest.mark.gpu

SEED = cg.SEED_BASE + 2200
SMALL = [(1500, 4), (2049, 3), (70, 4), (3000, 16), (8000, 2), (2500, 20)]


@pytest.fixture(scope="module")
def case():
    parts = [cg.random_sparse(60_000 - 41 * i, 1, 8, 0.05, 0.05, seed=SEED + i) for i in range(14)]
    for i, (n, d) in enumerate(SMALL):
        parts.insert(3 * i, cg.random_sparse(n, 1, d, 0.003, 0.003, seed=SEED + 50 + i))
    c = cg.concat(parts, name="cells with a tail")
    G.banner(f"cells tail: n={c.n} nnz={c.nnz}")
    return c, G.precompute(c)[0]


def _profiled(call):
    B.rp_profile_enable(G.ctx(), True)
    r = call()
    prof = B.rp_profile_read(G.ctx())
    B.rp_profile_enable(G.ctx(), False)
    return r, prof


def _tail(prof, precision):
    return prof["jacobi_tail_fp64" if precision == rp.RP_FP64 else "jacobi_tail_fp32"][0]


@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
def test_tail_equals_graph_replays(case, precision):
    c, sys = case
    kw = dict(tol=1e-10, stop=rp.RP_STOP_CERTIFIED, precision=precision)
    (x1, i1, c1), p1 = _profiled(lambda: G.solve(sys, "jacobi", graph=1, **kw))
    for again in range(2):
        (x0, i0, c0), p0 = _profiled(lambda: G.solve(sys, "jacobi", **kw))
        assert c0 == c1 == rp.binding.RP_OK
        assert all(i["lanes"] == 0 and i["panels"] == 0 for i in i0)
        assert _tail(p0, precision) > 0 and _tail(p1, precision) == 0
        assert [i["iterations"] for i in i0] == [i["iterations"] for i in i1]
        assert np.array_equal(x0, x1)
    for k in (0, 15):
        ck = c.instance(k)
        ref = oracle.solve(ck.n, ck.rp, ck.col, ck.val, ck.goal, "bicgstab", tol=1e-12, stop_mode=1)
        assert np.abs(x0[int(c.inst_off[k]):int(c.inst_off[k + 1])] - ref.x).max() <= 1e-10, k


def test_tail_paper_rule(case):
    c, sys = case
    kw = dict(tol=1e-10, stop=rp.RP_STOP_DELTA)
    (x0, i0, c0), p0 = _profiled(lambda: G.solve(sys, "jacobi", **kw))
    (x1, i1, c1), p1 = _profiled(lambda: G.solve(sys, "jacobi", schedule=1, **kw))
    assert c0 == c1 == rp.binding.RP_OK
    assert _tail(p0, rp.RP_FP64) > 0 and _tail(p1, rp.RP_FP64) > 0
    assert [i["iterations"] for i in i0] == [i["iterations"] for i in i1]
    assert np.array_equal(x0, x1)


@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
def test_adjoint_tail_equals_graph_replays(case, precision):
    c, sys = case
    kw = dict(tol=1e-10, stop=rp.RP_STOP_CERTIFIED, precision=precision)
    x, info, code = rp.rp_jacobi(G.ctx(), sys, **kw)
    seed = torch.zeros(c.n, dtype=torch.float64, device="cuda")
    seed[torch.arange(5, c.n, 977, device="cuda")] = 1.0
    (l1, g1, i1, c1), p1 = _profiled(lambda: rp.rp_adjoint(G.ctx(), sys, x, seed, 0, graph=1, **kw))
    (l0, g0, i0, c0), p0 = _profiled(lambda: rp.rp_adjoint(G.ctx(), sys, x, seed, 0, **kw))
    assert c0 == c1 == rp.binding.RP_OK
    assert _tail(p0, precision) > 0 and _tail(p1, precision) == 0
    assert [i["iterations"] for i in i0] == [i["iterations"] for i in i1]
    assert torch.equal(l0, l1) and torch.equal(g0, g1)
