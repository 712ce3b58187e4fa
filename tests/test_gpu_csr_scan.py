"""GPU: the CSR row offsets at match counts around the scan's segments (4096)
and groups (16384), and the seed counts on both sides of the count from which
blocks add them up (8192): the device's own checks of the stored graph find nothing
(row pointers, symmetric lists) and the statistics agree with the matches
themselves.  Whole numbers: exact."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 5, 63, 4095, 4096, 4099, 8192, 8193, 16383, 16385, 33001])
def test_scan_segments(N):
    import torch
    import paper_1501_02565_amd as epic
    H, W = 192, 256
    rng = np.random.default_rng(N)
    cost = torch.from_numpy(rng.uniform(0.1, 1.0, (H, W)).astype(np.float32)).cuda()
    pix = rng.permutation(H * W)[:N]
    m = np.stack([pix % W, pix // W, pix % W + 1.0, pix // W + 1.0], -1).astype(np.float32)
    dup, out = min(N // 3, 40), min(N // 5, 17)       # some repeated, some outside
    m[N - dup:, :2] = m[:dup, :2]
    m[N // 2:N // 2 + out, 0] = W + 3.0
    p = np.floor(m[:, :2] + 0.5)
    inside = (p[:, 0] >= 0) & (p[:, 0] < W) & (p[:, 1] >= 0) & (p[:, 1] < H)
    used = len(np.unique(p[inside, 1] * W + p[inside, 0]))
    print(f"[case] scan N={N}", flush=True)
    with epic.Context(0, debug_validate=True) as ctx:
        ctx.interp(cost, torch.from_numpy(m).cuda(), 8, 1.0, epic.NW)
        torch.cuda.synchronize()
        st = ctx.stats()
    assert st["n_invariant"] == 0
    assert st["n_used"] == used
    assert st["n_outside"] == int((~inside).sum())
    assert st["n_duplicate"] == int(inside.sum()) - used
