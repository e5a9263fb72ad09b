"""fp32 inverted-residual blocks with 3x3 windows run both products on three bf16 parts: large, small and infinite numbers in every form, both
strides and the image form, against the oracle and the layers apart.  Three parts hold most of these; those that they do not
hold in any place of a block are test_gpu_block_range's."""
import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import nmax

pytestmark = pytest.mark.gpu


def _net(cpi, ce, co, hw, stride, image, act, bn=True):
    net = synth.NetSpec(f"parts_{cpi}_{ce}_{hw}_{stride}_{image}", 3, hw, hw)
    if image:
        e = net.add(synth.Layer("conv", -1, 3, ce, k=3, stride=2, pad=1, act=act, bn=bn, name="e"))
    else:
        a = net.add(synth.Layer("conv", -1, 3, cpi, k=1, act=synth.ACT_NONE, bn=bn, name="a"))
        e = net.add(synth.Layer("conv", a, cpi, ce, k=1, act=act, bn=bn, name="e"))
    d = net.add(synth.Layer("conv", e, ce, ce, k=3, stride=stride, pad=1, groups=ce, act=act, bn=bn, name="d"))
    net.add(synth.Layer("conv", d, ce, co, k=1, act=synth.ACT_NONE, bn=bn, name="p"))
    return net, e, d


def _forms(handle, d):
    for form in (1, 2):
        for tile in (0, 1):
            for ks in (1, 2, 4):
                try:
                    handle.block_form(d, form, tile, ks)
                except B.CPruneError as err:
                    assert err.status == B.ERR_UNSUPPORTED
                    continue
                yield form, tile, ks


CASES = [
    (24, 40, 24, 17, 1, False),     # an odd last round of the expansion, three chunks, two strips
    (16, 33, 20, 30, 2, False),
    (64, 70, 50, 7, 1, False),      # two images a strip
    (96, 50, 90, 14, 2, False),
    (0, 32, 16, 40, 1, True),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("what", ["plain", "large", "infinite", "small", "weight"])
def test_large_small_and_infinite_numbers(orc, case, what):
    cpi, ce, co, hw, stride, image = case
    # ReLU6 bounds what large numbers become; without biases small inputs keep every sum small
    net, e, d = _net(cpi, ce, co, hw, stride, image, synth.ACT_RELU if what == "small" else synth.ACT_RELU6, bn=what != "small")
    params = synth.layer_params(net, 91)
    x = synth.net_input(net, 91, 3)
    if what == "large":
        x[1, :, 2:4, 3] = 3e25
        x[2, 0] *= -1e30
    elif what == "infinite":
        x[1, 1, 3, 2] = np.inf
    elif what == "small":
        x *= np.float32(1e-25)
    elif what == "weight":
        params[e]["w"][3] *= np.float32(1e25)
    ref_layers, _ = orc.prune_net(net, params)
    with np.errstate(invalid="ignore"):
        ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params))
    handle = pipeline.build_net(net, layers, 3, B.F32, tune=False)
    xd = torch.from_numpy(x).cuda()
    # an infinity's own products with weights of both signs are NaN, which the activation turns into a bound: that image against the layers apart
    keep = [0, 2] if what == "infinite" else [0, 1, 2]
    handle.block_form(d, 0)
    apart = handle.forward(xd).clone()
    ran = 0
    for form in _forms(handle, d):
        out = handle.forward(xd)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        # 1e-5: the fp32 bar of a layer (1e-4 of the maximum) less what these few terms leave unused
        assert nmax(got[keep], ref[keep]) < 1e-5, (form, nmax(got[keep], ref[keep]))
        assert torch.isfinite(apart).all() and nmax(got, apart.cpu().numpy()) < 1e-5, (form, nmax(got, apart.cpu().numpy()))
        ran += 1
    assert ran >= 4
    handle.close()
