"""Depthwise layers in a handle at the edges of their runs: one, two, four and seven outputs per thread at both strides, rows that a run
does not divide, maps smaller than the window, four channels per thread at 5x5, with and without a residual."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [B.F32, B.F16, B.BF16])
@pytest.mark.parametrize("cfg", [
    # channels, height, width, window, stride, batch
    (5, 1, 2, 5, 1, 2), (13, 2, 3, 5, 2, 3), (374, 5, 14, 5, 1, 3), (374, 14, 14, 5, 1, 12), (374, 15, 15, 5, 1, 12), (500, 7, 6, 5, 1, 16),
    (300, 13, 9, 5, 2, 16), (300, 26, 25, 5, 2, 16), (829, 7, 7, 3, 1, 13), (829, 14, 13, 3, 1, 26), (500, 15, 16, 3, 1, 40),
    (829, 13, 14, 3, 2, 64), (500, 15, 15, 3, 2, 48), (130, 9, 10, 3, 2, 32),
])
def test_runs(cfg, dtype):
    c, h, w, k, stride, batch = cfg
    td = B.TORCH_DTYPE[dtype]
    gen = torch.Generator().manual_seed(c + k + h)
    net = synth.NetSpec("runs", 8, h, w)
    a = net.add(synth.Layer("conv", -1, 8, c, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="a"))
    res = a if stride == 1 and h % 2 else None
    net.add(synth.Layer("conv", a, c, c, k=k, stride=stride, pad=k // 2, groups=c, act=synth.ACT_RELU6, residual=res, name="dw"))
    wa, wd = torch.randn(c, 8, 1, 1, generator=gen).to(td), (torch.randn(c, 1, k, k, generator=gen) / k).to(td)
    bd = torch.randn(c, generator=gen)
    handle = pipeline.build_net(net, [{"w": wa.cuda(), "b": torch.zeros(c, device="cuda")}, {"w": wd.cuda(), "b": bd.cuda()}], batch, dtype,
                                tune=False)
    y = handle.forward(torch.randn(batch, 8, h, w, generator=gen).to(td).cuda()).float().cpu()
    x = handle.activation(0, batch, (c, h, w)).double().cpu()
    assert handle.layer_fused(1) == 0
    handle.close()
    ref = torch.nn.functional.conv2d(x, wd.double(), bd.double(), stride, k // 2, groups=c)
    ref = (ref + x if res is not None else ref).clamp(0, 6)
    check(y.numpy(), ref.numpy(), dtype, f"{cfg}")
