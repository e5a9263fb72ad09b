"""fp32 inverted-residual blocks on three bf16 parts, against the same block layer by layer or products that are exact: numbers that the
parts do not hold in every place of a block, where a later weight lifts the result to ordinary size, and projections of few terms."""
import itertools

import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu


def _block(cpi, ce, co, hw, stride, act, gen, scales, batch=3, image=False):
    """cpi channels -> ce -> depthwise 3x3 -> co, with weights and input of the given sizes (input, expansion, window, projection)."""
    sx, se, sd, sp = scales
    normal = lambda *shape: torch.randn(*shape, generator=gen)
    net = synth.NetSpec(f"range_{cpi}_{ce}_{co}_{hw}_{stride}", 3 if image else cpi, hw, hw)
    zero = lambda n: torch.zeros(n, device="cuda")
    layers = []
    if image:
        e = net.add(synth.Layer("conv", -1, 3, ce, k=3, stride=2, pad=1, act=act, name="e"))
        layers.append({"w": (normal(ce, 3, 3, 3) * se).cuda(), "b": zero(ce)})
    else:
        # (the layer in front of a block is a pool here, which changes no number: 1x1 layers on the network's input have their own kernel)
        p = net.add(synth.Layer("maxpool", -1, cpi, cpi, k=1, stride=1, name="a"))
        e = net.add(synth.Layer("conv", p, cpi, ce, k=1, act=act, name="e"))
        layers += [None, {"w": (normal(ce, cpi, 1, 1) * se).cuda(), "b": zero(ce)}]
    d = net.add(synth.Layer("conv", e, ce, ce, k=3, stride=stride, pad=1, groups=ce, act=act, name="d"))
    net.add(synth.Layer("conv", d, ce, co, k=1, act=synth.ACT_NONE, name="p"))
    layers += [{"w": (normal(ce, 1, 3, 3) * sd).cuda(), "b": zero(ce)}, {"w": (normal(co, ce, 1, 1) * sp).cuda(), "b": zero(co)}]
    x = (normal(batch, 3 if image else cpi, hw, hw) * sx).cuda()
    return net, layers, x, d


def _forms(handle, d, forms=(1, 2)):
    for form, tile, ks in itertools.product(forms, (0, 1), (1, 2, 4)):
        try:
            handle.block_form(d, form, tile, ks)
        except B.CPruneError as err:
            assert err.status == B.ERR_UNSUPPORTED
            continue
        yield form, tile, ks


def _rel(got, want):
    return float((got.double() - want.double()).norm() / want.double().norm())


SHAPES = [(24, 40, 24, 17, 1, False), (16, 33, 20, 30, 2, False), (64, 70, 50, 7, 1, False), (0, 32, 16, 40, 1, True)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("scales", [
    (2.0 ** -126, 2.0 ** 58, 2.0 ** 10, 2.0 ** 14),      # the input's last parts, lifted by three weights
    (2.0 ** -120, 2.0 ** 30, 2.0 ** 30, 2.0 ** 30),
    (2.0 ** 56, 2.0 ** -124, 2.0 ** 20, 2.0 ** 10),      # the expansion's weights
    (1.0, 2.0 ** -60, 2.0 ** -62, 2.0 ** 90),            # a depthwise result
    (2.0 ** 40, 2.0 ** 40, 2.0 ** 10, 2.0 ** -122),      # the projection's weights
    (3e37, 2.0 ** -60, 1.0, 1.0),                        # the largest finite numbers
])
def test_lost_parts_do_not_reach_the_result(shape, scales):
    cpi, ce, co, hw, stride, image = shape
    net, layers, x, d = _block(cpi, ce, co, hw, stride, synth.ACT_RELU, torch.Generator().manual_seed(5), scales, image=image)
    if scales[0] > 1e37:
        x.clamp_(-3.4028e38, 3.4028e38)
        x[1, 0, 3, 4] = 3.4028e38                        # rounds to infinity as a first part
    # in 64 bits, from the same numbers
    q = [None if l is None else l["w"].double().cpu() for l in layers]
    F = torch.nn.functional
    z = x.double().cpu()
    z = F.conv2d(z, q[-3], stride=2 if image else 1, padding=1 if image else 0).clamp(min=0)
    z = F.conv2d(z, q[-2], stride=stride, padding=1, groups=ce).clamp(min=0)
    want = F.conv2d(z, q[-1])
    assert float(want.abs().max()) < 3e38 and float(want.abs().median()) > 2.0 ** -50
    handle = pipeline.build_net(net, layers, x.shape[0], B.F32, tune=False)
    ran = 0
    for form in _forms(handle, d):
        got = handle.forward(x).cpu()
        # at most 64 + 9 + 70 terms, rounded after each: 1.2e-7 times the root of their number
        assert _rel(got, want) < 1.5e-6, (form, _rel(got, want))
        ran += 1
    assert ran >= 4
    handle.close()


@pytest.mark.parametrize("shape", SHAPES)
def test_an_infinity_stays_where_it_is(shape):
    """One infinite input number, weights of one sign per filter: every expanded number is an infinity of that sign, which ReLU6 bounds."""
    cpi, ce, co, hw, stride, image = shape
    net, layers, x, d = _block(cpi, ce, co, hw, stride, synth.ACT_RELU6, torch.Generator().manual_seed(6), (1.0, 0.3, 0.3, 0.2), image=image)
    w = layers[-3]["w"]
    w.abs_()
    w[1::2] *= -1.0
    x[1, 1, 5, 2] = float("inf")
    handle = pipeline.build_net(net, layers, x.shape[0], B.F32, tune=False)
    big = x.clone()
    big[1, 1, 5, 2] = 1e6                                # the same behind the bound
    handle.block_form(d, 0)
    want = handle.forward(big).clone()
    ran = 0
    for form in _forms(handle, d):
        got = handle.forward(x)
        assert _rel(got, want) < 1e-6, (form, _rel(got, want))
        ran += 1
    assert ran >= 4
    handle.close()


@pytest.mark.parametrize("ce", [2, 7, 15])
@pytest.mark.parametrize("co,stride", [(16, 1), (24, 2), (60, 1), (90, 1), (90, 2)])
def test_few_terms_keep_their_products(ce, co, stride):
    """One projection weight a filter, windows that copy their middle: every result is one fp32 product, rounded once."""
    gen = torch.Generator().manual_seed(ce)
    net, layers, x, d = _block(8, ce, co, 15, stride, synth.ACT_NONE, gen, (1.0, 1.0, 1.0, 1.0))
    wd, wp = layers[-2]["w"], layers[-1]["w"]
    wd.zero_()
    wd[:, 0, 1, 1] = 1.0
    keep = torch.arange(co, device="cuda") % ce
    wp *= torch.nn.functional.one_hot(keep, ce).view(co, ce, 1, 1)
    handle = pipeline.build_net(net, layers, x.shape[0], B.F32, tune=False)
    handle.block_form(d, 0)
    handle.forward(x)
    expanded = handle.activation(1, x.shape[0], (ce, 15, 15))[:, :, ::stride, ::stride]
    want = expanded[:, keep] * wp[torch.arange(co), keep, 0, 0].view(1, co, 1, 1)
    for form in _forms(handle, d, (1,)):
        assert torch.equal(handle.forward(x), want), form
    handle.close()
