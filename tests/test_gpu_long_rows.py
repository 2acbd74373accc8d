"""One wavefront per row (schedule 64): rows around the sizes at which a lane's
pair of entries is cut or a row needs another batch (2 x 64 entries per load,
8 loads per batch, 4 per further one), with a whole-block window, with a band
window whose rows also reach outside it, and without a window; matrices of one
and of two entries.  Solutions are held to the oracle within 1e-10, the
certificate's own bound."""
import numpy as np
import pytest

import chaingen as cg
import oracle
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu

LENGTHS = (1, 2, 3, 63, 64, 65, 127, 128, 129, 130, 255, 256, 257, 1023, 1024, 1025, 1026, 1151, 1152, 1153, 1535,
           1536, 1537, 2047, 2048, 2049)


def _chain(n, span, seed):
    """States 2.. have rows of LENGTHS[i] undecided targets (every 16th state
    from a small set of lengths to keep the matrix small) and go to the goal
    (state 0) or the sink (state 1) with probability 0.1 each."""
    rng = np.random.Generator(np.random.PCG64(seed))
    rp_, cols, vals = [0, 1, 2], [np.array([0]), np.array([1])], [np.ones(1), np.ones(1)]
    for i in range(2, n):
        k = LENGTHS[(i // 16) % len(LENGTHS)] if i % 16 == 0 else (1, 2, 3, 5)[i % 4]
        lo, hi = (2, n) if span is None or (i % 3 == 0 and k < 4) else (max(2, i - span), min(n, i + span))
        k = min(k, hi - lo - 1)
        c = np.sort(rng.choice(hi - lo, size=k, replace=False) + lo)
        w = rng.random(k) + 0.1
        cols.append(np.concatenate([[0, 1], c]))
        vals.append(np.concatenate([[0.1, 0.1], 0.8 * w / w.sum()]))
        rp_.append(rp_[-1] + k + 2)
    goal = np.zeros(n, dtype=np.uint8)
    goal[0] = 1
    return cg.Chain(n, np.array(rp_, np.int32), np.concatenate(cols).astype(np.int32), np.concatenate(vals), goal,
                    np.array([0, n], np.int64), "long rows")


def _few(entries):
    p = np.zeros((5, 5))
    p[3, 3] = p[4, 4] = 1.0
    p[0, :] = [0, 0.5, 0, 0.5, 0]
    p[1, :] = [0, 0, 0.25 * (entries - 1), 0.6 - 0.25 * (entries - 1), 0.4]
    p[2, :] = [0, 0, 0, 0.3, 0.7]
    return cg.from_dense(p, [3])


@pytest.mark.parametrize("shape", ["one entry", "two entries", "whole", "band", "none"])
@pytest.mark.parametrize("precision", [rp.RP_FP64, rp.RP_FP32_REFINED])
def test_one_wavefront_per_row_matches_oracle(shape, precision):
    c = {"one entry": lambda: _few(1), "two entries": lambda: _few(2), "whole": lambda: _chain(4_003, None, 7),
         "band": lambda: _chain(44_003, 1_300, 8), "none": lambda: _chain(44_003, None, 9)}[shape]()
    G.banner(f"long rows: {shape}, n={c.n} nnz={c.nnz}")
    ref = oracle.solve(c.n, c.rp, c.col, c.val, c.goal, "bicgstab", tol=1e-12, stop_mode=1)
    sys, _, _ = G.precompute(c)
    for method in ("jacobi", "bicgstab"):
        x, info, code = G.solve(sys, method, tol=1e-10, stop=rp.RP_STOP_CERTIFIED, schedule=64, precision=precision)
        assert code == rp.binding.RP_OK and info[0]["lanes"] == 64
        assert np.abs(x - ref.x).max() <= 1e-10, method
