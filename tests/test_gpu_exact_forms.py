"""GPU: the exact interpolation's per-match form against its batched form.

The reference comes from a context with debug_validate, which always takes
the batched transforms; that the other call takes the per-match form, and in
how many rounds, is read from its plan (csrc/exact_plan.h, compiled for the
host).  Results are bitwise equal.  Scenes put the matches' reach below, at
and above the two page pools in LDS (271 and 543 blocks of 8 x 8 pixels) and
the two page tables (40 and 60 blocks across), and, with little room, put
matches off to further rounds.
"""
from __future__ import annotations

import numpy as np
import pytest

from exact_plan import lists_bytes, plan
from scenes import Scene, random_case
from test_gpu_exact_reach import _flat

pytestmark = pytest.mark.gpu


def _rough(H, W, N, K, seed):
    """Costs over two decades: matches reach from few to many blocks."""
    sc = _flat(H, W, N, K, seed)
    rng = np.random.default_rng(seed)
    coarse = np.exp(rng.uniform(np.log(0.01), 0.0, (-(-H // 16), -(-W // 16))))
    cost = (np.kron(coarse, np.ones((16, 16)))[:H, :W] * rng.uniform(0.8, 1.2, (H, W))).astype(np.float32)
    return Scene(cost, sc.matches, K, 1.0, 1, f"rough_{W}x{H}_n{N}_k{K}")


PLENTY = 1.2
CASES = [
    # around half a CU's pages, around a whole CU's, beyond both
    (lambda: _flat(150, 170, 390, 126, 1), 8, PLENTY), (lambda: _rough(150, 170, 390, 126, 2), 4, PLENTY),
    (lambda: _rough(150, 170, 64, 4, 3), 8, PLENTY),
    (lambda: _flat(237, 318, 560, 127, 4), 8, PLENTY), (lambda: _rough(237, 318, 560, 127, 5), 8, PLENTY),
    (lambda: _rough(237, 318, 800, 128, 6), 4, PLENTY),
    (lambda: _flat(300, 640, 770, 100, 7), 8, PLENTY), (lambda: _rough(301, 637, 770, 65, 8), 8, PLENTY),
    # the page tables' edges; no bound (K above the matches)
    (lambda: _flat(8, 166, 14, 16, 9), 8, PLENTY), (lambda: _flat(15, 321, 14, 16, 10), 8, PLENTY),
    (lambda: _flat(9, 472, 14, 16, 11), 4, PLENTY), (lambda: _flat(16, 600, 18, 24, 12), 8, PLENTY),
    (lambda: random_case(33, 47, 20, seed=89, K=40), 8, PLENTY), (lambda: random_case(9, 8, 5, seed=90, K=1), 8, PLENTY),
    (lambda: random_case(61, 83, 200, seed=87, K=65, outside=3, duplicates=4), 4, PLENTY),
    # further rounds
    (lambda: _rough(96, 128, 64, 64, 13), 8, 0.16), (lambda: _rough(96, 128, 64, 64, 14), 4, 0.4),
    (lambda: _flat(120, 130, 100, 128, 15), 8, 0.2), (lambda: random_case(33, 47, 20, seed=91, K=40), 8, 0.3),
    (lambda: _rough(150, 170, 390, 126, 16), 8, 0.2),
]


def test_four_million_matches():
    """Above the per-match form's launch (1024 threads a match): nearly all of
    the matches fall on pixels that a lower index holds."""
    import torch
    import paper_1501_02565_amd as epic
    H = W = 16
    N, K = 1 << 22, 4
    sc = random_case(H, W, 120, seed=92, K=K)
    assert sc.N == 120
    m = torch.from_numpy(sc.matches).cuda()
    many = m.repeat(-(-N // 120), 1)[:N].contiguous()
    many[120:, 2:] += 5.0
    cost = torch.from_numpy(sc.cost).cuda()
    ws = lists_bytes(H, W, N, K) + epic.workspace_bytes(H, W, N, K) + (2 << 30)
    assert plan(ws, H, W, N - 1, K)["rounds"] >= 1 and plan(ws, H, W, N, K)["rounds"] == 0
    print(f"[case] exact 16x16, {N} matches", flush=True)
    with epic.Context(0, 64 << 20) as c:
        ref = c.interp_exact(cost, m, K, 1.0, 1)
    with epic.Context(0, ws) as c:
        got = c.interp_exact(cost, many, K, 1.0, 1)
    assert torch.equal(got, ref)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_forms_agree(case):
    import torch
    import paper_1501_02565_amd as epic
    make, conn, part = CASES[case]
    sc = make()
    H, W, N, K = sc.H, sc.W, sc.N, sc.K
    nb = -(-H // 8) * -(-W // 8)
    # room for the worst case (every match reaching every block), times `part`
    pool = 8 * H * W + 16 * N + 600 * nb + int(280 * nb * (N + 2) * part * 4 / 3) + (1 << 16)
    if part == PLENTY:
        pool += 256 * 4 * 280 * nb
    ws = lists_bytes(H, W, N, K) + max(epic.workspace_bytes(H, W, N, K) + 8 * H * W,
                                       epic.workspace_bytes(1, 1, 1, 1) + pool) + 4096
    p = plan(ws, H, W, N, K)
    print(f"[case] exact {sc.name} conn {conn}: {nb} blocks, {p['rounds']} rounds", flush=True)
    assert p["rounds"] == 1 if part == PLENTY else p["rounds"] > 1
    cost, m = torch.from_numpy(sc.cost).cuda(), torch.from_numpy(sc.matches).cuda()
    with epic.Context(0, ws, connectivity=conn) as c:
        got = [c.interp_exact(cost, m, K, sc.a, sc.mode) for _ in range(2)]
    with epic.Context(0, max(ws, 256 << 20), connectivity=conn, debug_validate=1) as c:
        ref = c.interp_exact(cost, m, K, sc.a, sc.mode)
    assert torch.isfinite(ref).all()
    assert torch.equal(got[0], ref) and torch.equal(got[1], ref)
