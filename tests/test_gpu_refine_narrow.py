"""GPU: the refinement of an image one pixel wide and 2^27 + 37 high.

Its tiles, at least 32 pixels wide, are more than a single launch holds.  One
step of one sweep reaches a few pixels, so rows away from a crop's ends are
the whole image's, bit for bit (crops start at even rows: the sweeps' colours
alternate).
"""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


def test_one_pixel_wide():
    import torch
    import paper_1501_02565_amd as epic
    H, n, edge = (1 << 27) + 37, 4096, 32
    print(f"[case] refine 1x{H}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(7)
    I1 = torch.rand((H, 1), device="cuda", generator=gen)
    I2 = torch.zeros((H, 1), device="cuda")        # (a float holds no row number of 2^27: warped alike anywhere)
    u0 = torch.rand((H, 1, 2), device="cuda", generator=gen) * 4.0 - 2.0
    step = dict(fixed_point=1, sor=1)
    with epic.Context(0, epic.refine_bytes(H, 1, 1) + (64 << 20)) as c:
        out = c.refine(I1, I2, u0, **step)
        assert torch.isfinite(out).all() and not torch.equal(out[:n], u0[:n])
        mid = (1 << 26) - n // 2                   # the slices' border and the ends
        for a in (0, mid, H - 37 - n):
            b = a + n if a < H - 37 - n else H
            crop = c.refine(I1[a:b].contiguous(), I2[a:b].contiguous(), u0[a:b].contiguous(), **step)
            lo, hi = (0 if a == 0 else edge), (b - a if b == H else b - a - edge)
            assert torch.equal(out[a + lo:a + hi], crop[lo:hi])
