"""The split kernel: fp32 convolutions on the 16-bit matrix cores (every number cut into three bf16 parts)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import synth

pytestmark = pytest.mark.gpu


def split_variants():
    return [v for v in range(B.cprune_num_tile_variants()) if "conv_split" in B.cprune_tile_variant_name(v, False, B.F32)]


def _case(n, c_in, h, w, c_out, k, stride, dtype=B.F32, scale=1.0):
    x = synth.tensor_normal((n, c_in, h, w), 301, n, c_in) * np.float32(scale)
    wt = synth.tensor_normal((c_out, c_in, k, k), 302, c_out, k, std=(2.0 / (c_in * k * k)) ** 0.5)
    b = synth.tensor_normal((c_out,), 303, c_out, std=0.1) * np.float32(scale)
    td = B.TORCH_DTYPE[dtype]
    xd, wd, bd = torch.from_numpy(x).cuda().to(td), torch.from_numpy(wt).cuda().to(td), torch.from_numpy(b).cuda()
    d = B.conv_desc(x.shape, wt.shape, stride, k // 2, 1, dtype, B.ACT_NONE, False)
    ref = torch.nn.functional.conv2d(xd.cpu().double(), wd.cpu().double(), bd.cpu().double(), stride, k // 2)
    return d, xd, wd, bd, ref


@pytest.mark.parametrize("cfg", [
    # n, c_in, h, w, c_out, k, stride: edges of the 32-channel chunk and the 8-channel group, of the 16-filter block,
    # of the pixel block; several images per block; windows of one tap and of 49
    (1, 32, 16, 16, 16, 3, 1), (1, 33, 16, 16, 17, 3, 1), (2, 31, 13, 11, 15, 3, 1), (1, 8, 4, 4, 64, 3, 1),
    (3, 9, 7, 7, 130, 3, 1), (11, 70, 4, 4, 33, 3, 1), (1, 128, 56, 56, 83, 3, 1), (2, 40, 29, 3, 48, 3, 1),
    (2, 64, 28, 28, 67, 3, 2), (1, 24, 9, 9, 20, 5, 1), (1, 3, 40, 40, 64, 7, 2), (2, 100, 14, 14, 50, 1, 1),
    (1, 256, 4, 4, 96, 3, 1),
])
def test_split_is_no_less_exact(cfg):
    """Against 64 bits every split variant is within the bound of an fp32 sum of its terms' sizes, and its 2-norm error
    is no larger than 1.1 times the fp32 instruction's own (a fixed reference variant; 10 % for the spread between two
    orders of one sum) or half a unit in the last place, which short sums reach in either form."""
    d, x, w, b, ref = _case(*cfg)
    base = B.cprune_conv2d_bn_relu(d, x, w, b, None, 0).cpu().double()
    e_base = float((base - ref).norm() / ref.norm())
    ran = 0
    for v in split_variants():
        try:
            y = B.cprune_conv2d_bn_relu(d, x, w, b, None, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        ran += 1
        e = float((y.cpu().double() - ref).norm() / ref.norm())
        print(cfg, B.cprune_tile_variant_name(v, False, B.F32), f"{e:.2e} against {e_base:.2e}", flush=True)
        assert e <= max(1.1 * e_base, 2.0 ** -24), (v, e, e_base)
    assert ran >= 6


@pytest.mark.parametrize("dtype", [B.F16, B.BF16])
def test_split_16bit(dtype):
    d, x, w, b, ref = _case(2, 45, 13, 11, 37, 3, 1, dtype)
    ulp = 2.0 ** -11 if dtype == B.F16 else 2.0 ** -8
    for v in split_variants():
        y = B.cprune_conv2d_bn_relu(d, x, w, b, None, v).cpu().double()
        assert float((y - ref).abs().max() / ref.abs().max()) < 1.5 * ulp, v   # the rounding of the output, and the sum


def test_split_infinities_and_range():
    """An infinite or NaN input reaches exactly the outputs whose windows hold it, as the fp32 products send it there;
    numbers near both ends of the range keep their relative accuracy."""
    d, x, w, b, _ = _case(1, 20, 12, 12, 24, 3, 1)
    w[3, 4] = 1.0                       # parts that are zero
    x[0, 4, 5, 5] = float("inf")
    x[0, 7, 9, 2] = float("nan")
    want = B.cprune_conv2d_bn_relu(d, x, w, b, None, 0)
    for v in split_variants():
        y = B.cprune_conv2d_bn_relu(d, x, w, b, None, v)
        assert torch.equal(torch.isnan(y), torch.isnan(want)) and torch.equal(torch.isinf(y), torch.isinf(want))
        assert torch.equal(torch.sign(y[torch.isinf(y)]), torch.sign(want[torch.isinf(want)]))
    for scale in (1e30, 1e-25):
        d, x, w, b, ref = _case(1, 20, 12, 12, 24, 3, 1, scale=scale)
        for v in split_variants():
            y = B.cprune_conv2d_bn_relu(d, x, w, b, None, v).cpu().double()
            assert float((y - ref).norm() / ref.norm()) < 1e-6, (v, scale)


@pytest.mark.parametrize("cfg", [(1, 16, 8, 8, 16, 3, 1), (8, 128, 56, 56, 83, 3, 1), (2, 300, 8, 8, 40, 3, 1)])
def test_call_without_scratch_still_runs(cfg):
    """The library's own untimed choice never asks a caller without scratch for any."""
    d, x, w, b, ref = _case(*cfg)
    y = torch.empty(ref.shape, device="cuda")
    B.cprune_clear_tile_cache()
    st = B.lib().cprune_conv2d_bn_relu(C.byref(d), C.c_void_p(x.data_ptr()), C.c_void_p(w.data_ptr()),
                                       C.c_void_p(b.data_ptr()), None, C.c_void_p(y.data_ptr()), C.c_int(-1), None,
                                       C.c_size_t(0), None)
    assert st == B.OK
    torch.cuda.synchronize()
    assert float((y.cpu().double() - ref).norm() / ref.norm()) < 1e-6
