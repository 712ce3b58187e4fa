"""GPU: the exact interpolation's per-match path against its batched form.

The same call with workspaces from the least the batched transforms accept
(which the per-match path leaves to them) to plenty: in between, the entry
pool overflows and sources are put off to further rounds.  Every result is
bitwise that of the least one.  Flat cost maps make single matches reach more
blocks than the page table or LDS holds; K at the edges of the register sort,
K above the number of matches (no bound), 4 neighbours, odd sizes.
"""
from __future__ import annotations

import numpy as np
import pytest

from scenes import Scene, random_case

pytestmark = pytest.mark.gpu


def _flat(H, W, N, K, seed):
    rng = np.random.default_rng(seed)
    pix = np.sort(rng.choice(H * W, N, replace=False))
    m = np.stack([pix % W, pix // W, pix % W, pix // W], 1).astype(np.float32)
    m[:, 2:] += rng.uniform(-2.0, 2.0, (N, 2)).astype(np.float32)
    cost = (0.01 + 1e-3 * rng.uniform(0.0, 1.0, (H, W))).astype(np.float32)
    return Scene(cost, m, K, 1.0, 1, f"flat_{W}x{H}_n{N}_k{K}")


CASES = [
    (lambda: random_case(50, 64, 90, seed=85, K=12), 8),
    (lambda: random_case(61, 83, 200, seed=86, K=64, outside=3, duplicates=4), 8),
    (lambda: random_case(61, 83, 200, seed=87, K=65), 4),
    (lambda: random_case(40, 131, 260, seed=88, K=128, mode=0), 8),
    (lambda: random_case(33, 47, 20, seed=89, K=40), 8),             # K above the matches: no bound
    (lambda: random_case(9, 8, 5, seed=90, K=1), 8),
    (lambda: _flat(150, 170, 60, 50, 91), 8),                        # more blocks than LDS holds
    (lambda: _flat(8, 700, 40, 30, 92), 8),                          # further than the page table reaches
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_every_workspace_gives_the_same(case):
    import torch
    import paper_1501_02565_amd as epic
    make, conn = CASES[case]
    sc = make()
    cost, m = torch.from_numpy(sc.cost).cuda(), torch.from_numpy(sc.matches).cuda()
    HW = sc.H * sc.W
    tail = 8 * sc.K * HW + 4 * HW + sc.N + 8 * sc.N * sc.K + (36 << 10)
    per = epic.workspace_bytes(sc.H, sc.W, 1, 1) - epic.workspace_bytes(1, 1, 1, 1) + 4096
    least = max(epic.workspace_bytes(sc.H, sc.W, sc.N, sc.K), epic.workspace_bytes(1, 1, 1, 1) + 2 * per) + tail
    blocks = -(-sc.H // 8) * -(-sc.W // 8)
    worst = 280 * blocks * (sc.N + 2) * 4 // 3          # every match reaching every block
    print(f"[case] exact {sc.name} conn {conn}: {blocks} blocks", flush=True)
    ref = None
    for part in (0.0, 0.13, 0.16, 0.2, 0.3, 0.5, 1.0, 3.0):
        ws = least + int(part * worst) + (8 * HW + 16 * sc.N + 16 * blocks + 8192 if part else 0)
        with epic.Context(0, ws, connectivity=conn) as c:
            out = c.interp_exact(cost, m, sc.K, sc.a, sc.mode).cpu().numpy()
        assert np.isfinite(out).all()
        if ref is None:
            ref = out
        np.testing.assert_array_equal(out, ref, err_msg=f"workspace {ws} ({part})")
