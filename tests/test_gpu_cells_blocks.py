"""Cells, what a block does between tiles, and what the library falls back on.

The block of a compute unit takes a list of tiles: the first batch has more than
three tiles per compute unit, and every third chain in it mixes fast, so that tiles
of finished chains lie between live ones.  Jacobi iterates and counts are those of
one lane per row bit for bit: under the paper's rule in FP64, and in FP32 for a
residual that one inner solve reaches (no FP64 residual enters the iterate then).
BiCGStab and the adjoint are held to the oracle within 1e-10, the certificate's own
bound.

The second batch has the shape of cells, but a row of 20,000 entries in one chain or
in every one, whose entries would be taken one at a time: its forward products stay off the cells,
its transposed ones do not."""
import numpy as np
import pytest
import torch

import chaingen as cg
import oracle
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu

SEED = cg.SEED_BASE + 2400


@pytest.fixture(scope="module")
def lists():
    fast = {0.2: [], 0.02: []}
    for i in range(6):
        leak = 0.2 if i % 3 == 1 else 0.02
        fast[leak].append(cg.random_sparse(81_003 - 4_111 * i, 1, 8, leak, leak, seed=SEED + i))
    parts = [fast[0.2][(k // 3) % 2] if k % 3 == 1 else fast[0.02][k % 4] for k in range(90)]
    c = cg.concat(parts, name="lists of tiles")
    G.banner(f"cells lists: n={c.n} nnz={c.nnz}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert c.n // 8192 > 3 * cus  # a tile has at most 8,192 rows
    return c, parts, G.precompute(c)[0]


def _same(a, b):
    (x0, i0, c0), (x1, i1, c1) = a, b
    assert c0 == c1
    assert all(i["cells"] == 1 and i["lanes"] == 0 for i in i0) and all(i["cells"] == 0 and i["lanes"] == 1 for i in i1)
    n = [i["iterations"] for i in i0]
    assert n == [i["iterations"] for i in i1]
    assert np.array_equal(x0, x1)
    return n


@pytest.mark.parametrize("graph", [0, 1])
def test_paper_rule_is_that_of_one_lane_per_row(lists, graph):
    c, parts, sys = lists
    kw = dict(tol=1e-6, stop=rp.RP_STOP_DELTA, graph=graph)
    n = _same(G.solve(sys, "jacobi", **kw), G.solve(sys, "jacobi", schedule=1, **kw))
    assert 3 * max(n[1::3]) < min(n[0::3])


def test_fp32_inner_solve_is_that_of_one_lane_per_row(lists):
    c, parts, sys = lists
    kw = dict(tol=0.05, stop=rp.RP_STOP_RESIDUAL, precision=rp.RP_FP32_REFINED)
    n = _same(G.solve(sys, "jacobi", **kw), G.solve(sys, "jacobi", schedule=1, **kw))
    assert max(n[1::3]) < min(n[0::3])  # tiles of finished chains between live ones


@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
def test_bicgstab_and_adjoint_match_oracle(lists, precision):
    c, parts, sys = lists
    kw = dict(tol=1e-10, stop=rp.RP_STOP_CERTIFIED, precision=precision)
    x, info, code = G.solve(sys, "bicgstab", **kw)
    assert code == rp.binding.RP_OK and all(i["cells"] == 1 for i in info)
    ref = oracle.solve(parts[1].n, parts[1].rp, parts[1].col, parts[1].val, parts[1].goal, "bicgstab", tol=1e-12, stop_mode=1)
    sq = np.nonzero(ref.cls == oracle.SQ)[0]
    seed = np.zeros(c.n)
    alike = [k for k in range(90) if parts[k] is parts[1]]
    for k in alike:
        assert np.abs(x[c.inst_off[k]:c.inst_off[k + 1]] - ref.x).max() <= 1e-10, k
        seed[c.inst_off[k] + sq[7]] = 1.0
    lam, g, info, code = rp.rp_adjoint(G.ctx(), sys, torch.from_numpy(x).cuda(), torch.from_numpy(seed).cuda(), 1, **kw)
    assert code == rp.binding.RP_OK and all(i["cells"] == 1 for i in info)
    lam = lam.cpu().numpy()
    lam_o, _, _, rc = oracle.adjoint(ref, seed[c.inst_off[alike[0]]:c.inst_off[alike[0] + 1]], tol=1e-12)
    want = np.zeros(parts[1].n)
    want[sq] = lam_o[ref.red.map[sq]]
    for k in alike:
        got = lam[c.inst_off[k]:c.inst_off[k + 1]]
        assert np.abs(got - want).max() <= 1e-10 * max(1.0, np.abs(want).max()), k


def _hub(n, width, seed):
    """random_sparse with state 2's row replaced by one of `width` transitions."""
    c = cg.random_sparse(n, 1, 8, 0.05, 0.05, seed=seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    at = int(np.nonzero((np.diff(c.rp) > 1) & (c.goal == 0))[0][0])
    cols = np.sort(rng.choice(n, width, replace=False)).astype(np.int32)
    w = rng.random(width) + 0.1
    lo, hi = c.rp[at], c.rp[at + 1]
    ptr = c.rp.copy()
    ptr[at + 1:] += width - (hi - lo)
    return cg.Chain(n, ptr, np.concatenate([c.col[:lo], cols, c.col[hi:]]),
                    np.concatenate([c.val[:lo], w / w.sum(), c.val[hi:]]), c.goal, np.array([0, n], np.int64), "hub")


@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
@pytest.mark.parametrize("hubs", [1, 28])
def test_hub_rows_stay_off_the_cells(hubs, precision):
    plain = [cg.random_sparse(60_000 - 37 * i, 1, 8, 0.05, 0.05, seed=SEED + 100 + i) for i in range(4)]
    parts = [_hub(60_000 - 37 * i, 20_000, SEED + 100 + i) if i < hubs else plain[i % 4] for i in range(28)]
    c = cg.concat(parts, name="hubs")
    G.banner(f"cells, hub rows: n={c.n} nnz={c.nnz}")
    sys = G.precompute(c)[0]
    kw = dict(tol=1e-10, stop=rp.RP_STOP_CERTIFIED, precision=precision)
    ref = oracle.solve(parts[0].n, parts[0].rp, parts[0].col, parts[0].val, parts[0].goal, "bicgstab", tol=1e-12, stop_mode=1)
    sq = np.nonzero(ref.cls == oracle.SQ)[0]
    for method in ("jacobi", "bicgstab"):
        x, info, code = G.solve(sys, method, **kw)
        assert code == rp.binding.RP_OK and all(i["cells"] == 0 for i in info)
        assert np.abs(x[:parts[0].n] - ref.x).max() <= 1e-10, method
    seed = np.zeros(c.n)
    seed[sq[3]] = 1.0
    lam, g, info, code = rp.rp_adjoint(G.ctx(), sys, torch.from_numpy(x).cuda(), torch.from_numpy(seed).cuda(), 1, **kw)
    assert code == rp.binding.RP_OK and all(i["cells"] == 1 for i in info)
    lam_o, _, _, rc = oracle.adjoint(ref, seed[:parts[0].n], tol=1e-12)
    want = np.zeros(parts[0].n)
    want[sq] = lam_o[ref.red.map[sq]]
    assert np.abs(lam.cpu().numpy()[:parts[0].n] - want).max() <= 1e-10 * max(1.0, np.abs(want).max())
