"""The 7x7 / stride 2 first layer where its kernels meet their ends: as a network's last layer on a 1x1 map, where pixels lie dense in the
caller's buffer; an infinite pixel, which every window row multiplies once."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu


def _reference(x, q, act):
    """In 64 bits, from the numbers as they are stored."""
    y = torch.nn.functional.conv2d(x.double().cpu(), q["w"].double().cpu(), q["b"].double().cpu(), stride=2, padding=3)
    return y if act == synth.ACT_NONE else y.clamp(0.0, 6.0 if act == synth.ACT_RELU6 else None)


@pytest.mark.parametrize("dtype,tol", [(B.F32, 1e-6), (B.F16, 2.0 ** -11), (B.BF16, 2.0 ** -8)])   # one rounding of the result (fp32: 147 terms)
@pytest.mark.parametrize("hw", [1, 2])
@pytest.mark.parametrize("c_out", [1, 5, 6, 8, 35, 67])
def test_a_dense_last_map(dtype, tol, hw, c_out):
    gen = torch.Generator().manual_seed(c_out)
    t = B.TORCH_DTYPE[dtype]
    net = synth.NetSpec(f"dense7_{hw}_{c_out}", 3, hw, hw)
    net.add(synth.Layer("conv", -1, 3, c_out, k=7, stride=2, pad=3, act=synth.ACT_NONE, name="a"))
    q = {"w": torch.randn(c_out, 3, 7, 7, generator=gen).to(t).cuda(), "b": torch.randn(c_out, generator=gen).cuda()}
    x = torch.randn(3, 3, hw, hw, generator=gen).to(t).cuda()
    handle = pipeline.build_net(net, [q], 3, dtype, tune=False)
    want = _reference(x, q, synth.ACT_NONE).reshape(-1)
    for n in (3, 2):
        room = torch.full((n * c_out + 16,), -77.0, dtype=t, device="cuda")
        print("dense last map", dtype, hw, c_out, n, flush=True)
        handle.forward(x[:n], room)
        torch.cuda.synchronize()
        got = room[:n * c_out].double().cpu()
        assert (got - want[:n * c_out]).abs().max() <= tol * want.abs().max()
        assert (room[n * c_out:] == -77.0).all()
    handle.close()


@pytest.mark.parametrize("dtype", [B.F16, B.BF16])
@pytest.mark.parametrize("c_in", [1, 2, 3])
@pytest.mark.parametrize("c_out", [24, 40])
@pytest.mark.parametrize("at", [(6, 8), (13, 3), (0, 0), (15, 15)])
def test_an_infinite_pixel(dtype, c_in, c_out, at):
    """Positive weights: an infinity anywhere under a window is the activation's bound there, and changes nothing elsewhere (but in the
    column right of the window's reach, whose zero weight in front of the window meets it)."""
    gen = torch.Generator().manual_seed(7)
    t = B.TORCH_DTYPE[dtype]
    net = synth.NetSpec(f"inf7_{c_in}_{c_out}", c_in, 16, 16)
    a = net.add(synth.Layer("conv", -1, c_in, c_out, k=7, stride=2, pad=3, act=synth.ACT_RELU6, name="a"))
    net.add(synth.Layer("conv", a, c_out, 8, k=1, act=synth.ACT_NONE, name="b"))
    mk = lambda *s: {"w": (torch.rand(*s, generator=gen) * 0.02 + 0.001).to(t).cuda(), "b": torch.zeros(s[0], device="cuda")}
    layers = [mk(c_out, c_in, 7, 7), mk(8, c_out, 1, 1)]
    x = torch.rand(2, c_in, 16, 16, generator=gen).to(t).cuda()
    handle = pipeline.build_net(net, layers, 2, dtype, tune=False)
    handle.first_layer_form(1)
    handle.forward(x)
    plain = handle.activation(0, 2, (c_out, 8, 8)).clone()
    for c in range(c_in):
        y, z = at
        big = x.clone()
        big[1, c, y, z] = float("inf")
        handle.forward(big)
        got = handle.activation(0, 2, (c_out, 8, 8))
        rows = torch.arange(8).view(8, 1) * 2
        cols = torch.arange(8).view(1, 8) * 2
        under = ((rows - 3 <= y) & (y <= rows + 3) & (cols - 3 <= z) & (z <= cols + 3)).cuda()
        beside = (cols - 4 == z).expand(8, 8).cuda()
        assert torch.equal(got[0], plain[0])
        assert (got[1][:, under] == 6.0).all(), (c, at)
        elsewhere = ~under & ~beside
        assert torch.equal(got[1][:, elsewhere], plain[1][:, elsewhere]), (c, at)
    handle.close()
