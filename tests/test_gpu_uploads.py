"""A system's small arrays reach the device through one ring of pinned memory
(parts of up to 64 KB, a ring of 1 MB): batches of three-state chains whose
per-chain arrays lie just below and above a part, and above the ring, solved
twice in one context so that the ring wraps.  The probability of each chain is
known: p / (1 - s), with one division's rounding in the library and here."""
import numpy as np
import pytest

import chaingen as cg
import paper_1210_6412_amd as rp
from tests import _gpu as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 16_383, 16_385, 140_000])
def test_many_small_chains(k):
    G.banner(f"uploads: {k} chains")
    i = np.arange(k)
    p, s = 0.25 + 0.25 * (i % 7) / 7.0, 0.125 * (i % 3)
    val = np.stack([s, p, 1.0 - s - p, np.ones(k), np.ones(k)], 1)
    col = np.stack([3 * i, 3 * i + 1, 3 * i + 2, 3 * i + 1, 3 * i + 2], 1)
    keep = np.ones((k, 5), bool)
    keep[:, 0] = s > 0
    ptr = np.zeros(3 * k + 1, np.int32)
    ptr[1:] = np.cumsum(np.stack([keep[:, :3].sum(1), keep[:, 3], keep[:, 4]], 1).ravel())
    goal = np.zeros(3 * k, np.uint8)
    goal[1::3] = 1
    c = cg.Chain(3 * k, ptr, col[keep].astype(np.int32), val[keep], goal, 3 * np.arange(k + 1, dtype=np.int64), "many")
    for _ in range(2):
        sys, _, _ = G.precompute(c)
        x, info, code = G.solve(sys, "jacobi", tol=1e-12, stop=rp.RP_STOP_CERTIFIED)
        assert code == rp.binding.RP_OK
        assert np.abs(x[0::3] - p / (1.0 - s)).max() <= 1e-12
