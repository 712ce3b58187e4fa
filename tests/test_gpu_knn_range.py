"""GPU: the K-NN search where its sums pass the range of a float.

Costs are any finite positive numbers, so a frontier distance plus a lightest
edge can overflow while the distances themselves are finite.  A scene with its
cost multiplied by a power of two and `a` divided by it scales every FP32 sum
exactly: distances are the base scene's, scaled, and the neighbour lists are
the same, cut where a scaled distance is infinite (the search ends at an
infinite frontier).  Lists that lose nothing give the same models, and the
exact variant, whose bounds come from the lists, the same field.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest

from oracle import epic_ref
from scenes import Scene

pytestmark = pytest.mark.gpu

FMAX = float(np.finfo(np.float32).max)


def scene(name, K, conn, part):
    """The base scene, the same scaled by 2^p, and p: the base cost is drawn
    so that `part` of the sources keep their K-th distance finite."""
    rng = np.random.default_rng(K + conn)
    H, W, step = {"grid": (84, 84, 4), "strip": (9, 600, 3), "dense": (40, 40, 2)}[name]
    ys, xs = np.mgrid[1:H:step, 1:W:step]
    m = np.stack([xs.ravel(), ys.ravel(), xs.ravel(), ys.ravel()], 1).astype(np.float32)
    m[:, 2:] += rng.uniform(-2.0, 2.0, (len(m), 2)).astype(np.float32)
    cost = rng.uniform(0.5, 1.5, (H, W))
    r = epic_ref.stages(cost.astype(np.float32), m, K, 1.0, 1, conn=conn)
    kth = np.quantile(r["knn_d"][:, K - 1], part)
    p = int(np.floor(np.log2(FMAX / kth)))
    cost = (cost * (0.995 * FMAX / (kth * 2.0 ** p))).astype(np.float32)
    return (Scene(cost, m, K, 1.0, 1, f"{name}_k{K}"),
            Scene(np.ldexp(cost, p), m, K, float(np.ldexp(1.0, -p)), 1, f"{name}_k{K}_2^{p}"), p)


CASES = [("grid", 20, 8, 1.0), ("grid", 100, 8, 0.6), ("grid", 100, 8, 1.0), ("grid", 128, 4, 0.3),
         ("strip", 63, 8, 0.8), ("strip", 128, 4, 1.0), ("dense", 200, 8, 0.5), ("dense", 7, 4, 0.9)]


@pytest.mark.parametrize("name,K,conn,part", CASES)
def test_scaled_cost(name, K, conn, part):
    import torch
    import paper_1501_02565_amd as epic
    import parity
    base, scaled, p = scene(name, K, conn, part)
    print(f"[case] {scaled.name} conn {conn} part {part}", flush=True)
    with epic.Context(0, connectivity=conn) as c:
        b, s = parity.gpu_stages(c, base), parity.gpu_stages(c, scaled)
    with np.errstate(over="ignore"):
        want = np.ldexp(b["knn_d"], p)
    assert (b["knn_idx"] >= 0).all()
    whole = np.isfinite(want).all(1)
    assert 0.0 < whole.mean() <= 1.0
    np.testing.assert_array_equal(s["D"], np.ldexp(b["D"], p))
    np.testing.assert_array_equal(s["L"], b["L"])
    np.testing.assert_array_equal(s["knn_d"], want)
    np.testing.assert_array_equal(s["knn_idx"], np.where(np.isfinite(want), b["knn_idx"], -1))
    np.testing.assert_array_equal(s["params"][whole], b["params"][whole])
    # exact variant: its distances stay finite where the lists' do
    if part == 1.0 and K <= 128:
        out = []
        with epic.Context(0, 1 << 30, connectivity=conn) as c:
            for sc in (base, scaled):
                out.append(c.interp_exact(torch.from_numpy(sc.cost).cuda(), torch.from_numpy(sc.matches).cuda(),
                                          K, sc.a, 1))
        assert torch.isfinite(out[0]).all()
        assert torch.equal(out[0], out[1])
