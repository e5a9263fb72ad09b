"""Host time of an untimed choice: a caller without a timed shape pays it on every call."""
import time

import pytest

from paper_2207_01260_amd import binding as B


def _choice_us(d):
    best = float("inf")
    for _ in range(7):
        t0 = time.perf_counter()
        for _ in range(300):
            B.cprune_cached_tile(d)
        best = min(best, (time.perf_counter() - t0) / 300 * 1e6)
    return best


@pytest.mark.parametrize("n,c_in,hw,c_out,k", [(8, 128, 56, 83, 3), (4, 64, 112, 64, 5)])
def test_windows_cost_little_more_than_one_tap(n, c_in, hw, c_out, k):
    """The split kernel's pixel blocks are a search per block size and staging depth, not per variant: 3 and 4 us over the
    general kernel's 4 (13 and 24 when every variant searched twice)."""
    B.cprune_clear_tile_cache()
    shape = (n, c_in, hw, hw)
    window = _choice_us(B.conv_desc(shape, (c_out, c_in, k, k), 1, k // 2, 1, B.F32))
    one_tap = _choice_us(B.conv_desc(shape, (c_out, c_in, 1, 1), 1, 0, 1, B.F32))
    assert window < 3.0 * one_tap, (window, one_tap)
