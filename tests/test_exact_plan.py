"""The exact interpolation's choice between its two forms, and the layout of
the per-match one, on the host."""
from __future__ import annotations

import numpy as np
import pytest

from exact_plan import plan, plan_at, up

# (H, W, N, K) and which form was faster there, times in us (batched, per match)
MEASURED = [
    ((300, 640, 8, 16), "batched"),          # 2110, 12615
    ((300, 640, 64, 16), "batched"),         # 2531, 7136
    ((300, 640, 192, 16), "batched"),        # 2141, 3274
    ((300, 640, 320, 16), "per match"),      # 2024, 1261
    ((300, 640, 2560, 16), "per match"),     # 3160, 865
    ((300, 640, 256, 64), "batched"),        # 6199, 7666
    ((300, 640, 1280, 64), "per match"),     # 6398, 2572
    ((300, 640, 300, 128), "batched"),       # (N = 256: 12390, 13055)
    ((300, 640, 384, 128), "batched"),       # 12393, 16070
    ((300, 640, 1536, 128), "per match"),    # 12763, 7732
    ((436, 1024, 96, 16), "batched"),        # 4568, 10435
    ((436, 1024, 128, 4), "batched"),        # 1952, 3157
    ((436, 1024, 256, 8), "batched"),        # 2683, 3160
    ((436, 1024, 640, 16), "per match"),     # 4032, 2271
    ((436, 1024, 64, 128), "batched"),       # 20758, 39795
    ((436, 1024, 1024, 128), "per match"),   # 27192, 23588
    ((436, 1024, 8000, 100), "per match"),   # 28894, 5298
    ((1080, 2048, 512, 128), "batched"),     # 165803, 201448
    ((1080, 2048, 1536, 128), "per match"),  # 145867, 120114
    ((1080, 2048, 3000, 128), "per match"),  # 144672, 99497
    ((64, 64, 1, 16), "per match"),          # 256, 206
    ((64, 64, 32, 128), "per match"),        # 355, 221
    ((96, 128, 8, 16), "batched"),           # 436, 535
    ((96, 128, 12, 4), "per match"),         # 398, 319
    ((96, 128, 64, 16), "per match"),        # 459, 296
    ((96, 128, 300, 32), "per match"),       # 1016, 231
    ((128, 160, 32, 16), "batched"),         # 599, 758
    ((128, 160, 32, 4), "per match"),        # 385, 308
    ((150, 170, 64, 16), "batched"),         # 673, 826
    ((150, 170, 64, 4), "per match"),        # 432, 267
    ((8, 2048, 64, 16), "per match"),        # 1055, 685
]


@pytest.mark.parametrize("size,form", MEASURED)
def test_form_by_reach(size, form):
    H, W, N, K = size
    p = plan(40 << 30, H, W, N, K)
    assert ("per match" if p["rounds"] else "batched") == form


@pytest.mark.parametrize("size,part,form", [
    ((436, 1024, 768, 128), 0.5, "batched"),      # 32424, 40709
    ((436, 1024, 768, 128), 0.14, "batched"),     # 47610, 160899
    ((300, 640, 1024, 128), 0.25, "batched"),     # 17551, 20732
    ((1080, 2048, 1024, 16), 0.5, "batched"),     # 19189, 22853
    ((300, 640, 320, 16), 0.14, "per match"),     # 5840, 1380
    ((436, 1024, 8000, 100), 0.14, "per match"),  # 30591, 5503
    ((96, 128, 64, 64), 0.25, "per match"),       # 2506, 1721
])
def test_form_by_room(size, part, form):
    H, W, N, K = size
    nb = -(-H // 8) * -(-W // 8)
    begin = 1 << 20
    used = begin + 64 * H * W                     # (the approximated pass needs less than the pool)
    tail = begin + up(8 * H * W) + 600 * nb + 16 * N + int(280 * nb * N * part * 4 / 3)
    p = plan_at(H, W, N, K, begin, min(used, tail - up(8 * H * W)), tail)
    assert ("per match" if p["rounds"] else "batched") == form


@pytest.mark.parametrize("size,form", [
    ((16, 16, (1 << 22) - 1, 4), "per match"), ((16, 16, 1 << 22, 4), "batched"),
    ((8192, 8184, 2000, 1), "per match"), ((8191, 8192, 1100, 1), "batched"),      # 1024 * 1023 and 2^20 blocks
])
def test_launches_below_2_32_threads(size, form):
    H, W, N, K = size
    p = plan(8 << 30, H, W, N, K) if H < 100 else plan_at(H, W, N, K, 1 << 20, 1 << 20, 400 << 30)
    nb = -(-H // 8) * -(-W // 8)
    assert ("per match" if p["rounds"] else "batched") == form
    assert p["rounds"] == 0 or max(1024 * N, 64 * 64 * nb) < 1 << 32


def test_layout():
    """Arrays of the per-match form: in order, apart, within the space the
    approximated pass and the lists leave them; every match placed in the
    planned rounds at worst."""
    rng = np.random.default_rng(3)
    seen = {"batched": 0, "one": 0, "more": 0}
    for _ in range(4000):
        H, W = (int(np.exp(rng.uniform(0, np.log(1500)))) for _ in range(2))
        N, K = int(np.exp(rng.uniform(0, np.log(20000)))), int(rng.integers(1, 129))
        nb = -(-H // 8) * -(-W // 8)
        begin = 256 * int(rng.integers(16, 10000))
        used = begin + 256 * int(rng.integers(0, 4 * nb))
        tail = 256 * int((begin + 8 * H * W) / 256 + np.exp(rng.uniform(0, np.log(4 * nb * N + 10))))
        p = plan_at(H, W, N, K, begin, used, tail)
        if p["rounds"] == 0:
            seen["batched"] += 1
            continue
        seen["one" if p["rounds"] == 1 else "more"] += 1
        cap, groups = p["pool_cap"], p["big_groups"]
        assert 1 <= groups <= 256 and 1 <= p["rounds"] <= 8
        assert p["scratch_words"] >= (nb + 1) * 64 + 5 * nb
        size = [("ctl", 4 * 96), ("pend0", 4 * N), ("pend1", 4 * N), ("wide", 4 * N), ("big", 4 * N),
                ("bcount", 4 * nb), ("offset", 4 * nb), ("scratch", 4 * p["scratch_words"] * groups),
                ("meta", 16 * cap), ("order", 8 * cap), ("pool", 256 * cap), ("cu", 8 * H * W)]
        at = begin
        for name, b in size:
            assert p[name] % 256 == 0 and p[name] >= at, name
            at = p[name] + b
        assert at <= tail and p["cu"] >= used
        # a round places matches until one does not fit: at least those that
        # fill the pool with every block
        assert N <= p["rounds"] * (cap // nb - 1)
        assert N * nb < 1 << 31 and cap < 1 << 31
    assert min(seen.values()) > 100, seen
