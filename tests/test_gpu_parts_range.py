"""Numbers below 2^-110 against large operands, within the limits of three bf16 parts (operands under 2^59): the kernels that run fp32
data that way answer as the fp32 instruction does, small sums being multiplied again."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu

SCALES = [(2.0 ** -112, 2.0 ** 55), (2.0 ** 55, 2.0 ** -112), (2.0 ** -100, 2.0 ** 50), (2.0 ** -118, 2.0 ** 58)]


def _variants(kernel, channels_last):
    return [v for v in range(B.cprune_num_tile_variants()) if kernel in B.cprune_tile_variant_name(v, channels_last, B.F32)]


def _layer(c, h, w, o, k, stride):
    net = synth.NetSpec("range", c, h, w)
    net.add(synth.Layer("conv", -1, c, o, k=k, stride=stride, pad=k // 2, act=synth.ACT_NONE, name="a"))
    return net


def _rel(got, want):
    return float((got.double() - want.double()).norm() / want.double().norm())


@pytest.mark.parametrize("scales", SCALES)
@pytest.mark.parametrize("kernel,c,h,o,k,stride", [("conv_rows_nchw", 70, 11, 40, 3, 1), ("conv_rows_s2", 70, 11, 40, 3, 2),
                                                   ("conv_pw3", 80, 9, 72, 1, 1), ("conv_pw3", 80, 9, 72, 1, 2)])
def test_layers(kernel, c, h, o, k, stride, scales):
    gen = torch.Generator().manual_seed(c + stride)
    x = (torch.randn(2, c, h, h, generator=gen) * scales[0]).cuda()
    w = (torch.randn(o, c, k, k, generator=gen) * scales[1]).cuda()
    zero = torch.zeros(o, device="cuda")
    d = B.conv_desc(x.shape, w.shape, stride, k // 2, 1, B.F32, B.ACT_NONE)
    want = B.cprune_conv2d_bn_relu(d, x, w, zero, tile_variant=0)      # the fp32 instruction
    assert want.isfinite().all() and want.any()
    boundary, ran = kernel == "conv_rows_nchw", 0
    handle = None if boundary else pipeline.build_net(_layer(c, h, h, o, k, stride), [{"w": w, "b": zero}], 2, B.F32, tune=False)
    for v in _variants(kernel, not boundary):
        try:
            if boundary:
                got = B.cprune_conv2d_bn_relu(d, x, w, zero, tile_variant=v)
            else:
                handle.set_layer_variant(0, v)
                got = handle.forward(x)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        ran += 1
        # at most 630 terms in fp32, in other orders
        assert _rel(got.view(want.shape), want) < 2e-6, (v, _rel(got.view(want.shape), want))
    assert ran >= 3
    if handle:
        handle.close()


@pytest.mark.parametrize("scales", SCALES)
@pytest.mark.parametrize("form", [None, 2])
def test_first_layer(form, scales):
    gen = torch.Generator().manual_seed(9)
    x = (torch.randn(2, 3, 40, 36, generator=gen) * scales[0]).cuda()
    net = _layer(3, 40, 36, 40, 7, 2)
    net.add(synth.Layer("maxpool", 0, 40, 40, k=3, stride=2, pad=1, name="b"))
    net.add(synth.Layer("conv", 1, 40, 8, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="c"))
    layers = [{"w": (torch.randn(40, 3, 7, 7, generator=gen) * scales[1]).cuda(), "b": torch.zeros(40, device="cuda")}, None,
              {"w": torch.ones(8, 40, 1, 1, device="cuda"), "b": torch.zeros(8, device="cuda")}]
    handle = pipeline.build_net(net, layers, 2, B.F32, tune=form is None)
    got = []
    for f in (form, 0):
        if f is not None:
            handle.first_layer_form(f)
        handle.forward(x)
        got.append(handle.activation(1, 2, (40, 10, 9)).clone())
    handle.close()
    assert got[1].isfinite().all() and got[1].any()
    assert _rel(got[0], got[1]) < 2e-6
