"""Ranking at the edges of its two forms (one entry per thread up to 1024 filters, LDS lists above)."""
import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [1, 2, 63, 64, 65, 127, 129, 512, 1000, 1023, 1024, 1025, 2049])
def test_rank_sizes_with_ties(orc, c):
    """Scores with many exact ties (small integers: sums exact in any order): lower index first, at every keep edge."""
    rng = np.random.RandomState(c)
    w = rng.randint(-3, 4, size=(c, 2, 1, 1)).astype(np.float32)
    w[rng.rand(c) < 0.1] = 0.0
    for keep in sorted({1, max(1, c // 3), max(1, c - 1), c}):
        _, order_ref, kept_ref = orc.rank_filters(w, keep)
        _, order, kept = B.cprune_rank_filters(torch.from_numpy(w).cuda(), keep)
        assert np.array_equal(order.cpu().numpy(), order_ref), (c, keep)
        assert np.array_equal(kept.cpu().numpy(), kept_ref), (c, keep)
