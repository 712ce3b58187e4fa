"""GPU: the exact interpolation's sources at the edges of the two sizes of page
pools in LDS (271 and 543 blocks of 8 x 8 pixels) and page tables (40 and 60
blocks across).  With fewer matches than K there is no bound, so every match
reaches every block of the image; the result is bitwise that of the batched
transforms (the least workspace)."""
from __future__ import annotations

import pytest

from test_gpu_exact_reach import _flat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,conn", [
    (120, 144, 8), (128, 136, 8), (129, 143, 4), (184, 184, 8), (181, 177, 4), (181, 187, 8),   # 270 .. 552 blocks
    (8, 166, 8), (15, 321, 8), (9, 472, 4), (16, 600, 8)])                                      # 21 .. 75 across
def test_wide_sources(H, W, conn):
    import torch
    import paper_1501_02565_amd as epic
    sc = _flat(H, W, 14, 16, H * 7 + W)
    print(f"[case] exact {sc.name} conn {conn}", flush=True)
    cost, m = torch.from_numpy(sc.cost).cuda(), torch.from_numpy(sc.matches).cuda()
    HW = H * W
    tail = 8 * sc.K * HW + 4 * HW + sc.N + 8 * sc.N * sc.K + (36 << 10)
    per = epic.workspace_bytes(H, W, 1, 1) - epic.workspace_bytes(1, 1, 1, 1) + 4096
    least = max(epic.workspace_bytes(H, W, sc.N, sc.K), epic.workspace_bytes(1, 1, 1, 1) + 2 * per) + tail
    got = []
    for ws in (least, least + (256 << 20)):
        with epic.Context(0, ws, connectivity=conn) as c:
            got.append(c.interp_exact(cost, m, sc.K, sc.a, sc.mode).cpu())
    assert torch.isfinite(got[0]).all()
    assert torch.equal(got[0], got[1])
