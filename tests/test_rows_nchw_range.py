"""Outputs at the 2 GiB that the row strips in the boundary's layout address: refused from there on, on the host; what runs such a layer
instead writes every element."""
import ctypes as C

import pytest
import torch

from paper_2207_01260_amd import binding as B

DTYPES = {"f32": B.F32, "f16": B.F16, "bf16": B.BF16}
FAKE = C.c_void_p(0x1000)   # never dereferenced: refused, or no device to launch on


def _variants(dtype):
    return [v for v in range(B.cprune_num_tile_variants()) if "conv_rows_nchw" in B.cprune_tile_variant_name(v, False, dtype)]


def _status(d, v):
    return B.lib().cprune_conv2d_bn_relu(C.byref(d), FAKE, FAKE, None, FAKE if d.has_residual else None, FAKE, v, None, 0, None)


@pytest.mark.skipif(torch.cuda.is_available(), reason="asks with addresses that a launch must not see")
@pytest.mark.parametrize("dtype", sorted(DTYPES))
@pytest.mark.parametrize("residual", [False, True])
def test_outputs_from_two_gib_on_are_refused(dtype, residual):
    es = 4 if dtype == "f32" else 2
    rows = 2 ** 31 // es // (512 * 1024)                 # of 512 planes of 1024 columns: 2 GiB
    for n, filters, h, runs in ((1, 512, rows - 1, True), (1, 512, rows, False), (2, 512, rows // 2, False), (1, 513, rows, False),
                                (3, 512, rows // 2, False), (2, 512, rows, False)):
        if n * filters * h * 1024 >= 2 ** 31:            # (more elements than any call takes)
            continue
        d = B.conv_desc((n, 8, h, 1024), (filters, 8, 3, 3), 1, 1, 1, DTYPES[dtype], B.ACT_RELU, residual)
        got = [_status(d, v) for v in _variants(DTYPES[dtype])]
        ran = [s for s in got if s != B.ERR_UNSUPPORTED]
        assert bool(ran) == runs, (n, filters, h, got)


@pytest.mark.gpu
def test_an_output_over_two_gib_is_written_whole():
    """fp32, 8 -> 513 filters at 1024x1024: the timed choice, around byte 2^31 and in the last plane, against the layer's last filters."""
    gen = torch.Generator().manual_seed(1)
    x, w = torch.randn(1, 8, 1024, 1024, generator=gen), torch.randn(513, 8, 3, 3, generator=gen)
    bias = torch.randn(513, generator=gen)
    d = B.conv_desc(x.shape, w.shape, 1, 1, 1, B.F32, B.ACT_NONE)
    xd, wd, bd = x.cuda(), w.cuda(), bias.cuda()
    B.cprune_clear_tile_cache()
    v = B.cprune_select_tile(d, xd, wd, bd, warmup=0, iters=1)[0]
    B.cprune_clear_tile_cache()
    assert v not in _variants(B.F32)
    y = torch.full(B.out_shape(d), float("nan"), device="cuda")
    B.cprune_conv2d_bn_relu(d, xd, wd, bd, tile_variant=v, y=y)
    assert y.isfinite().all()
    ref = torch.nn.functional.conv2d(x.double(), w[-2:].double(), bias[-2:].double(), 1, 1)
    # 72 terms in fp32, each rounded once
    assert float((y[:, -2:].double().cpu() - ref).abs().max() / ref.abs().max()) < 72 * 2.0 ** -24
