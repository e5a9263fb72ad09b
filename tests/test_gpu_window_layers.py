"""Depthwise, max-pool and average-pool layers inside a handle at the edges of their launch shapes: channel counts around a
16-byte vector and around the pools' vector groups, maps from one pixel up, one / two / four outputs per thread."""
import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [
    # channels, map height, width, window, stride, batch, dtype
    (5, 1, 1, 3, 1, 2, B.F32), (9, 3, 2, 5, 1, 3, B.BF16), (33, 7, 7, 5, 2, 2, B.F32), (130, 14, 13, 3, 1, 3, B.F16),
    (264, 7, 7, 3, 2, 2, B.BF16), (400, 29, 31, 3, 1, 8, B.F32), (520, 28, 28, 5, 1, 4, B.BF16),
    (300, 57, 56, 3, 2, 12, B.F32), (96, 90, 90, 3, 1, 12, B.F16),
])
def test_depthwise_and_pools(orc, cfg):
    c, h, w, k, stride, batch, dtype = cfg
    net = synth.NetSpec(f"window_{c}_{h}_{w}_{k}_{stride}", 3, h, w)
    a = net.add(synth.Layer("conv", -1, 3, c, k=1, stride=1, pad=0, act=synth.ACT_RELU, bn=True, name="a"))
    b = net.add(synth.Layer("conv", a, c, c, k=k, stride=stride, pad=k // 2, groups=c, act=synth.ACT_RELU, bn=True, name="dw"))
    p = net.add(synth.Layer("maxpool", b, c, c, k=3, stride=2, pad=1, name="pool"))
    g = net.add(synth.Layer("gavgpool", p, c, c, name="gap"))
    net.add(synth.Layer("fc", g, c, 7, bias=True, name="fc"))
    params = synth.layer_params(net, 40 + k)
    x = synth.net_input(net, 41 + k, batch)
    ref_layers, _ = orc.prune_net(net, params)
    acts = orc.forward(net, ref_layers, x, return_all=True)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    out = handle.forward(torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype]))
    torch.cuda.synchronize()
    for i, name in ((1, "depthwise"), (2, "max-pool"), (3, "average pool")):
        got = handle.activation(i, batch, acts[i].shape[1:])
        torch.cuda.synchronize()
        check(np.asarray(got.float().cpu()), acts[i], dtype, f"{cfg} {name}")
    check(out.float().cpu().numpy(), acts[-1], dtype, f"{cfg} fc")
    handle.close()


@pytest.mark.parametrize("cfg", [
    # channels, map height, width, window, batch, dtype: one, two and four outputs per thread
    (20, 9, 8, 3, 2, B.F32), (400, 29, 31, 3, 8, B.F32), (96, 90, 90, 3, 12, B.F16), (24, 12, 12, 5, 1, B.BF16),
    (520, 28, 28, 5, 8, B.BF16), (160, 64, 64, 5, 12, B.F16),
])
def test_infinite_weight_of_a_row_outside(cfg):
    """A window row outside the image adds nothing to a depthwise sum, even if its weight is infinite."""
    c, h, w, k, batch, dtype = cfg
    td = B.TORCH_DTYPE[dtype]
    gen = torch.Generator().manual_seed(c)
    net = synth.NetSpec("rows", 8, h, w)
    a = net.add(synth.Layer("conv", -1, 8, c, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="a"))
    net.add(synth.Layer("conv", a, c, c, k=k, stride=1, pad=k // 2, groups=c, act=synth.ACT_NONE, name="dw"))
    wa, wd = torch.randn(c, 8, 1, 1, generator=gen).to(td), torch.randn(c, 1, k, k, generator=gen).to(td)
    wd[1, 0, 0, k // 2], wd[c - 1, 0, k - 1, k // 2] = float("inf"), -float("inf")
    zero = torch.zeros(c, device="cuda")
    handle = pipeline.build_net(net, [{"w": wa.cuda(), "b": zero}, {"w": wd.cuda(), "b": zero}], batch, dtype, tune=False)
    y = handle.forward(torch.randn(batch, 8, h, w, generator=gen).to(td).cuda()).double().cpu()
    x = handle.activation(0, batch, (c, h, w)).double().cpu()
    handle.close()
    p = k // 2
    finite = torch.isfinite(y)
    assert finite[:, 1, :p].all() and not finite[:, 1, p:].any()          # the first window row is outside
    assert finite[:, c - 1, h - p:].all() and not finite[:, c - 1, :h - p].any()
    wd[1, 0, 0, p], wd[c - 1, 0, k - 1, p] = 0.0, 0.0
    ref = torch.nn.functional.conv2d(x, wd.double(), None, 1, p, groups=c)
    check(y[finite].numpy(), ref[finite].numpy(), dtype, f"{cfg}")
