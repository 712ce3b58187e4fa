"""GPU: the K-NN search at the edges of its relaxation windows and tables.

A cheap middle row is the cell of one match (the hub), whose edges lead to a
match on every pixel of the rows above and below it: 2 W edges in one
segment, in windows of 64, and 2 W + 1 nodes in every search's table (256
entries first, more in the retry).  Sizes put the segment's end before, on
and behind a window's end and the table below, at and above its capacity.
Every stage against the FP64 oracle: the FP32 path within parity's
tolerances, the FP64 path bit for bit in its lists and distances.
"""
from __future__ import annotations

import numpy as np
import pytest

import parity
from scenes import Scene

pytestmark = pytest.mark.gpu


def _hub(W, K, seed=5):
    rng = np.random.default_rng(seed + W)
    cost = rng.uniform(0.5, 1.5, (3, W)).astype(np.float32)
    cost[1] = rng.uniform(1e-4, 2e-4, W).astype(np.float32)
    m = np.zeros((2 * W + 1, 4), np.float32)
    m[0, :2] = (W // 2, 1)
    m[1:W + 1, 0], m[1:W + 1, 1] = np.arange(W), 0
    m[W + 1:, 0], m[W + 1:, 1] = np.arange(W), 2
    m[:, 2:] = m[:, :2] + rng.uniform(-3.0, 3.0, (2 * W + 1, 2)).astype(np.float32)
    return Scene(cost, m, min(K, 2 * W), 1.0, 1, f"hub_{W}x3_k{K}")


@pytest.mark.parametrize("W", [16, 31, 32, 33, 64, 97, 127, 128, 140])
@pytest.mark.parametrize("K", [5, 60, 128])
def test_hub_segments(W, K):
    import paper_1501_02565_amd as epic
    sc = _hub(W, K)
    r = parity.ref_stages(sc)
    assert np.bincount(np.concatenate([r["em"], r["en"]])).max() >= 2 * W       # the hub's segment
    print(f"[case] {sc.name}", flush=True)
    with epic.Context(0) as c:
        print(parity.full_check(c, sc), flush=True)
    with epic.Context(0, precision=1) as c:
        g = parity.gpu_stages(c, sc)
    n = r["K"]
    np.testing.assert_array_equal(g["knn_idx"][:, :n], r["knn_idx"][:, :n])
    np.testing.assert_array_equal(g["knn_d"][:, :n], np.float32(r["knn_d"][:, :n]))
