"""Memory of the cells: an FP32-refined solve whose sweeps run on cells builds the
FP32 ones alone (8 bytes per entry); the FP64 residuals around it take what is
there.  Free memory of the device before and after the solve, in contexts of their
own, against the same solve on one lane per row."""
import pytest
import torch

import chaingen as cg
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu

SEED = cg.SEED_BASE + 2300


def test_fp32_refined_solve_builds_no_fp64_cells():
    c = cg.concat([cg.random_sparse(60_000 - 31 * i, 1, 8, 0.05, 0.05, seed=SEED + i) for i in range(28)], name="cells")
    t = G.dev(c)
    used = {}
    for schedule in (1, -1):
        G.banner(f"cells memory: schedule {schedule}")
        ctx = rp.rp_context_create(0)
        sys = rp.rp_precompute(ctx, t["row_ptr"], t["col"], t["val"], t["goal"], t["off"])
        torch.cuda.synchronize()
        x = torch.empty(c.n, dtype=torch.float64, device="cuda")
        before = torch.cuda.mem_get_info()[0]
        _, info, code = rp.rp_jacobi(ctx, sys, x, tol=1e-10, stop=rp.RP_STOP_CERTIFIED, precision=rp.RP_FP32_REFINED,
                                     schedule=schedule)
        torch.cuda.synchronize()
        used[schedule] = before - torch.cuda.mem_get_info()[0]
        assert code == rp.binding.RP_OK
        z = rp.rp_system_sizes(sys)[3]
        rp.rp_system_destroy(sys)
        rp.rp_context_destroy(ctx)
    assert all(i["lanes"] == 0 and i["panels"] == 0 for i in info)
    extra = used[-1] - used[1]
    # 8 bytes per entry; up to 16 blocks of 2 MB for the steps, records and tail
    assert extra <= 8 * z + 16 * 2 ** 21 < 20 * z, (extra, z)
