"""The 7x7 / stride 2 first layer of fp32 handles on three 16-bit parts, alone and with the 3x3 / stride 2 max-pool inside: one to
three channels, one and two 16-filter blocks per wavefront, several filter tiles, bands of two rows up to whole maps, odd maps, the last
strip and band cut short; numbers that three parts do not hold."""
import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import check

pytestmark = pytest.mark.gpu


def _net(c_in, c1, h, w, act=synth.ACT_RELU):
    net = synth.NetSpec(f"stem_{c_in}_{c1}_{h}_{w}", c_in, h, w)
    a = net.add(synth.Layer("conv", -1, c_in, c1, k=7, stride=2, pad=3, act=act, bn=True, name="stem"))
    p = net.add(synth.Layer("maxpool", a, c1, c1, k=3, stride=2, pad=1, name="pool"))
    net.add(synth.Layer("conv", p, c1, 8, k=1, stride=1, pad=0, act=synth.ACT_NONE, bn=True, name="b"))
    return net


@pytest.mark.parametrize("cfg", [
    # c_in, filters, height, width, batch, activation
    (3, 64, 224, 224, 1, synth.ACT_RELU), (3, 64, 56, 64, 5, synth.ACT_RELU6), (3, 20, 37, 35, 2, synth.ACT_RELU),
    (1, 40, 30, 50, 3, synth.ACT_NONE), (2, 100, 18, 22, 2, synth.ACT_RELU), (3, 32, 7, 7, 1, synth.ACT_RELU),
    (3, 33, 8, 113, 2, synth.ACT_NONE), (3, 9, 20, 20, 1100, synth.ACT_RELU), (3, 70, 61, 29, 70, synth.ACT_RELU),
])
def test_first_layer_on_three_parts(orc, cfg):
    c_in, c1, h, w, batch, act = cfg
    net = _net(c_in, c1, h, w, act)
    params = synth.layer_params(net, 71)
    x = synth.net_input(net, 72, batch)
    ref_layers, _ = orc.prune_net(net, params)
    acts = orc.forward(net, ref_layers, x, return_all=True)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params))
    handle = pipeline.build_net(net, layers, batch, tune=False)
    xd = torch.from_numpy(x).cuda()
    for form in (None, 2, 0, 2):              # as built (the kernel without the pool), with it, the general kernels
        if form is not None:
            handle.first_layer_form(form)
        out = handle.forward(xd, use_graph=form == 2)
        torch.cuda.synchronize()
        if form == 2:
            with pytest.raises(B.CPruneError):
                handle.activation(0, batch, acts[0].shape[1:])
        else:
            check(handle.activation(0, batch, acts[0].shape[1:]).cpu().numpy(), acts[0], B.F32, f"{cfg} form {form} conv")
        check(handle.activation(1, batch, acts[1].shape[1:]).cpu().numpy(), acts[1], B.F32, f"{cfg} form {form} pool")
        check(out.cpu().numpy(), acts[2], B.F32, f"{cfg} form {form}")
    with pytest.raises(B.CPruneError) as e:
        handle.first_layer_form(1)
    assert e.value.status == B.ERR_UNSUPPORTED
    handle.close()


@pytest.mark.parametrize("cfg", [
    # c_in, filters, height, width, batch, activation
    (3, 64, 112, 112, 2, synth.ACT_RELU), (3, 20, 37, 35, 3, synth.ACT_RELU6), (1, 40, 30, 57, 3, synth.ACT_NONE),
    (2, 100, 18, 22, 2, synth.ACT_RELU), (3, 33, 8, 113, 2, synth.ACT_NONE), (3, 9, 20, 20, 300, synth.ACT_RELU),
    (3, 32, 7, 7, 1, synth.ACT_RELU),
])
def test_a_timed_handle_keeps_the_conv_map(orc, cfg):
    """The pool runs inside the layer's kernel, and the layer's own map is there to be copied, at smaller batches and in graphs too."""
    c_in, c1, h, w, batch, act = cfg
    net = _net(c_in, c1, h, w, act)
    params = synth.layer_params(net, 77)
    x = synth.net_input(net, 78, batch)
    ref_layers, _ = orc.prune_net(net, params)
    acts = orc.forward(net, ref_layers, x, return_all=True)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params))
    handle = pipeline.build_net(net, layers, batch, tune=True)
    xd = torch.from_numpy(x).cuda()
    for n, graph in ((batch, False), ((batch + 1) // 2, False), (batch, True), (batch, True)):
        xn = xd[:n].contiguous()
        out = handle.forward(xn, use_graph=graph)
        for i in (0, 1):
            got = handle.activation(i, n, acts[i].shape[1:]).cpu().numpy()
            check(got, acts[i][:n], B.F32, f"{cfg} layer {i} n {n} graph {graph}")
        check(out.cpu().numpy(), acts[2][:n], B.F32, f"{cfg} n {n} graph {graph}")
    times = handle.layer_times(xd)
    assert times[0] > 0 and times[1] == 0            # one launch
    handle.close()


def test_error_is_no_larger_than_on_the_fp32_instruction():
    net = _net(3, 64, 96, 96, synth.ACT_NONE)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(synth.layer_params(net, 73)))
    handle = pipeline.build_net(net, layers, 4, tune=False)
    x = torch.from_numpy(synth.net_input(net, 74, 4)).cuda()
    w, b = layers[0]["w"].double().cpu(), layers[0]["b"].double().cpu()
    ref = torch.nn.functional.conv2d(x.double().cpu(), w, b, 2, 3)
    err = []
    for form in (None, 0):
        if form is not None:
            handle.first_layer_form(form)
        handle.forward(x)
        y = handle.activation(0, 4, ref.shape[1:]).double().cpu()
        err.append(float((y - ref).norm() / ref.norm()))
    print("three parts, fp32 instruction:", err)
    handle.close()
    assert err[0] <= err[1]


@pytest.mark.parametrize("pooled", [False, True])
def test_numbers_three_parts_do_not_hold(pooled):
    """An infinity, numbers near the largest, and images of tiny numbers: what the fp32 instruction gives."""
    net = _net(3, 64, 40, 60, synth.ACT_NONE)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(synth.layer_params(net, 75)))
    layers[0]["b"].zero_()
    handle = pipeline.build_net(net, layers, 3, tune=False)
    if pooled:
        handle.first_layer_form(2)
    x = torch.from_numpy(synth.net_input(net, 76, 3)).cuda()
    x[0, 1, 20, 30] = float("inf")
    x[0, 2, 5, 50] = 3.3e38
    x[1] *= 2.0 ** -115
    got = []
    for _ in range(2):
        handle.forward(x)
        got.append(handle.activation(1, 3, (64, 10, 15)).double().cpu())
        handle.first_layer_form(0)
    handle.close()
    assert torch.equal(got[0].isfinite(), got[1].isfinite()) and not got[1][0].isfinite().all()
    assert torch.equal(got[0][~got[0].isfinite()], got[1][~got[1].isfinite()])
    for n in range(3):
        ok = got[1][n].isfinite()
        # both sum 147 terms in fp32, in different orders: 147 * 2^-24 at most, of sums of the terms' sizes
        ref = got[1][n][ok].clamp(-1e30, 1e30)
        assert float((got[0][n][ok].clamp(-1e30, 1e30) - ref).abs().max() / ref.abs().max()) < 147 * 2.0 ** -24
