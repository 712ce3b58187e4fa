"""GPU: the FP64 path's K nearest lists where distances tie.

Up to 128 candidates are sorted in registers by distance alone and, when two
are equal, again with the match index; on a constant cost map with matches on
a grid nearly every distance has equals.  Lists and distances must be the
oracle's, bit for bit, below, at and above the register sort's 64 and 128
candidates.
"""
from __future__ import annotations

import numpy as np
import pytest

import parity
from scenes import Scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 9, 40, 63, 64, 65, 100, 128])
@pytest.mark.parametrize("jitter", [0.0, 1e-3])
def test_tied_distances(K, jitter):
    import paper_1501_02565_amd as epic
    rng = np.random.default_rng(K)
    H, W = 61, 67
    cost = (np.full((H, W), 0.25) + jitter * rng.uniform(0.0, 1.0, (H, W))).astype(np.float32)
    ys, xs = np.mgrid[2:H:4, 2:W:4]
    m = np.stack([xs.ravel(), ys.ravel(), xs.ravel(), ys.ravel()], 1).astype(np.float32)
    m[:, 2:] += rng.uniform(-2.0, 2.0, (len(m), 2)).astype(np.float32)
    sc = Scene(cost, m, K, 1.0, 1, f"tied_k{K}")
    print(f"[case] {sc.name} jitter {jitter}", flush=True)
    r = parity.ref_stages(sc)
    with epic.Context(0, precision=1) as c:
        g = parity.gpu_stages(c, sc)
    np.testing.assert_array_equal(g["D"], r["D"])
    np.testing.assert_array_equal(g["L"], r["L"])
    np.testing.assert_array_equal(g["knn_idx"], r["knn_idx"])
    np.testing.assert_array_equal(g["knn_d"], np.float32(r["knn_d"]))
