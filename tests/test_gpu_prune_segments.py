"""GPU: the compaction of the kept matches at counts around its segments (1024)
and groups (8192).  With K = 1 the first estimate at a match is its own
displacement, so the kept matches are exactly the placed ones: inside the image
and the lowest index of their pixel, in index order.  Whole numbers: exact."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 63, 65, 1023, 1025, 4100, 8191, 8192, 8193, 16385, 20011])
def test_kept_in_index_order(N):
    import torch
    import paper_1501_02565_amd as epic
    H, W = 160, 192
    rng = np.random.default_rng(N)
    cost = torch.from_numpy(rng.uniform(0.1, 1.0, (H, W)).astype(np.float32)).cuda()
    m = np.empty((N, 4), np.float32)
    m[:, 0] = rng.integers(0, W + W // 2, N)          # a third outside
    m[:, 1] = rng.integers(0, H, N)                   # and some on the same pixel
    m[0, 0] = 0
    m[:, 2:] = m[:, :2] + rng.uniform(-5, 5, (N, 2)).astype(np.float32)
    inside = np.flatnonzero(m[:, 0] < W)
    _, first = np.unique(m[inside, 1].astype(np.int64) * W + m[inside, 0].astype(np.int64), return_index=True)
    want = np.sort(inside[first])
    print(f"[case] prune segments N={N}", flush=True)
    with epic.Context(0) as ctx:
        got = ctx.prune(cost, torch.from_numpy(m).cuda(), 1, 1.0, 1.0).cpu().numpy()
    assert np.array_equal(got, want)
