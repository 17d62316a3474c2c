"""The canonical yaw search where its split over lanes and blocks has edges:
yaws that fill no wave, one yaw or point, chunks with a remainder, and clouds
long enough that a launch of its own joins the chunks' extents.  Against the
oracle within 1e-12: FP64, sums of at most 1e5 terms in another order."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as orc
from test_gpu_canon import check, gpu_yaw, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K,R", [(1, 4096, 3), (31, 129, 5), (257, 3, 4), (33, 63, 2), (8193, 16, 12),
                                   (65537, 20, 20), (90001, 1, 7)])
def test_yaw_split_edges(n, K, R):
    say(f"test_yaw_split_edges[n={n}, K={K}, R={R}]")
    rng = np.random.default_rng(n + 3 * K + R)
    P = (rng.normal(size=(n, 3)) * [0.3, 0.5, 0.2] + [-1.0, 0.5, 2.0]).astype(np.float32)
    F = rng.uniform(0, 2, (R, R, R)).astype(np.float32)
    check(gpu_yaw(P, F, K), orc.canonical_yaw(P, F, K))
