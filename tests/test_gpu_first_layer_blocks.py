"""The 16-bit 7x7 / stride 2 first layer of up to 48 filters on both sides of its rule (strips, or 16 x 16 blocks where those fill the chip evenly):
one, two and three work-groups of blocks per CU and the next round; strips that walk over bands of several steps, their ring of image rows coming
round, which do not divide the map; one to three channels, ragged maps, with and without the pool."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(B.F16, 2.0 ** -10), (B.BF16, 2.0 ** -7)])        # one rounding of each result, and its fp32 sum's
@pytest.mark.parametrize("c_in,c_out,h,w,batch", [
    (3, 8, 224, 224, 2), (3, 16, 224, 224, 12), (3, 16, 224, 224, 16),          # strips / blocks, three per CU / strips
    (2, 17, 224, 221, 4), (1, 32, 98, 130, 23), (3, 24, 224, 224, 24),          # blocks: one, two per CU, two rounds (strips without the pool)
    (3, 33, 98, 130, 23), (3, 48, 224, 224, 8), (1, 48, 224, 223, 12),          # strips / blocks without the pool, blocks, strips
    (3, 49, 98, 130, 23),                                                       # strips only
    (3, 24, 41, 29, 700), (1, 40, 61, 29, 300), (1, 10, 85, 31, 500), (3, 33, 75, 61, 260), (2, 64, 43, 40, 400),     # bands of 4 to 11 steps
])
def test_strips_and_blocks(dtype, tol, c_in, c_out, h, w, batch):
    gen = torch.Generator().manual_seed(c_out + batch)
    t = B.TORCH_DTYPE[dtype]
    net = synth.NetSpec(f"blocks7_{c_in}_{c_out}_{h}_{w}", c_in, h, w)
    a = net.add(synth.Layer("conv", -1, c_in, c_out, k=7, stride=2, pad=3, act=synth.ACT_RELU, name="a"))
    p = net.add(synth.Layer("maxpool", a, c_out, c_out, k=3, stride=2, pad=1, name="p"))
    net.add(synth.Layer("conv", p, c_out, 8, k=1, act=synth.ACT_NONE, name="b"))
    mk = lambda *s: {"w": (torch.randn(*s, generator=gen) * 0.1).to(t).cuda(), "b": torch.randn(s[0], generator=gen).cuda()}
    layers = [mk(c_out, c_in, 7, 7), {}, mk(8, c_out, 1, 1)]
    x = torch.randn(batch, c_in, h, w, generator=gen).to(t)
    # fp32 sums on the CPU of the numbers as they are stored; the pool of rounded numbers is the rounded pool
    F = torch.nn.functional
    conv = F.conv2d(x.float(), layers[0]["w"].float().cpu(), layers[0]["b"].cpu(), stride=2, padding=3).clamp(min=0)
    pool = F.max_pool2d(conv, 3, 2, 1)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    xd = x.cuda()
    for form in (2, 1):
        handle.first_layer_form(form)
        print("strips and blocks", dtype, c_in, c_out, h, w, batch, form, flush=True)
        handle.forward(xd)
        torch.cuda.synchronize()
        checks = [(1, pool)] + ([(0, conv)] if form == 1 else [])
        for i, want in checks:
            got = handle.activation(i, batch, want.shape[1:]).float().cpu()
            assert ((got - want).abs() <= tol * want.abs() + 1e-5).all(), (i, float((got - want).abs().max()))
    handle.close()


@pytest.mark.parametrize("c_out,batch", [(24, 8), (40, 8), (24, 1)])      # blocks, blocks, strips
def test_an_input_off_a_word(c_out, batch):
    """An image that begins at an odd element of its storage gives the same bits."""
    gen = torch.Generator().manual_seed(9)
    net = synth.NetSpec("odd7", 3, 224, 224)
    a = net.add(synth.Layer("conv", -1, 3, c_out, k=7, stride=2, pad=3, act=synth.ACT_RELU, name="a"))
    p = net.add(synth.Layer("maxpool", a, c_out, c_out, k=3, stride=2, pad=1, name="p"))
    net.add(synth.Layer("conv", p, c_out, 8, k=1, act=synth.ACT_NONE, name="b"))
    mk = lambda *s: {"w": (torch.randn(*s, generator=gen) * 0.1).bfloat16().cuda(), "b": torch.zeros(s[0], device="cuda")}
    handle = pipeline.build_net(net, [mk(c_out, 3, 7, 7), {}, mk(8, c_out, 1, 1)], batch, B.BF16, tune=False)
    x = torch.randn(batch, 3, 224, 224, generator=gen).bfloat16().cuda()
    room = torch.empty(x.numel() + 1, dtype=torch.bfloat16, device="cuda")
    off = room[1:].view(x.shape)
    off.copy_(x)
    assert off.data_ptr() % 4 == 2
    assert torch.equal(handle.forward(off), handle.forward(x))
    handle.close()
