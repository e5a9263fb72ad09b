"""Host time of an untimed choice, as a caller without a timed shape pays it the first time, and of the remembered one."""
import time

import pytest

from paper_2207_01260_amd import binding as B


def _choice_us(d):
    """The choice itself: nothing remembered."""
    best = float("inf")
    for _ in range(7):
        spent = 0.0
        for _ in range(300):
            B.cprune_clear_tile_cache()
            t0 = time.perf_counter()
            B.cprune_cached_tile(d)
            spent += time.perf_counter() - t0
        best = min(best, spent / 300 * 1e6)
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


@pytest.mark.parametrize("n,c_in,hw,c_out,k,stride,old", [(5, 491, 80, 151, 3, 2, "1, 2, 5"),
                                                          (44, 128, 24, 202, 3, 2, "2, 2, 5")])
def test_estimate_knows_how_many_groups_a_unit_holds(n, c_in, hw, c_out, k, stride, old):
    """Variants that stage five items per thread hold two work-groups per unit, not three: the estimate that counted three
    took them on layers others run faster (491 -> 151 at 80x80, stride 2, batch 5, 123 us; now 98)."""
    B.cprune_clear_tile_cache()
    v, timed = B.cprune_cached_tile(B.conv_desc((n, c_in, hw, hw), (c_out, c_in, k, k), stride, k // 2, 1, B.F32))
    assert not timed
    assert not B.cprune_tile_variant_name(v, False, B.F32).endswith(old + ">"), B.cprune_tile_variant_name(v, False, B.F32)


@pytest.mark.parametrize("dtype,n,c_in,h,w,c_out,strips", [
    # over 1 GFLOP (16-bit: 2) with chunks of 32 channels that are mostly padding: 68 us before, 90 on strips; 49 and 60
    (B.F32, 9, 8, 94, 77, 326, False), (B.F32, 10, 13, 76, 76, 381, False), (B.BF16, 13, 7, 74, 74, 398, False),
    # a chain of five chunks under 5 MFLOP: 10.3 and 12.2 us
    (B.F32, 1, 141, 12, 12, 13, False),
    # ... and their neighbours, where strips are the faster ones
    (B.F32, 1, 64, 32, 32, 45, True), (B.F32, 8, 128, 56, 56, 83, True), (B.F32, 3, 132, 34, 34, 12, True), (B.BF16, 2, 24, 56, 56, 64, True),
])
def test_strips_where_their_chunks_are_filled(dtype, n, c_in, h, w, c_out, strips):
    B.cprune_clear_tile_cache()
    v, timed = B.cprune_cached_tile(B.conv_desc((n, c_in, h, w), (c_out, c_in, 3, 3), 1, 1, 1, dtype))
    assert not timed
    assert ("conv_rows_nchw" in B.cprune_tile_variant_name(v, False, dtype)) == strips
