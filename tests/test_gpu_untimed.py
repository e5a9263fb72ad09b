"""What a choice of variants looks at, timed and untimed."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu


def _fc_net(c, hw, o, batch):
    gen = torch.Generator().manual_seed(c + hw)
    net = synth.NetSpec("fc", c, hw, hw)
    a = net.add(synth.Layer("conv", -1, c, c, k=1, stride=1, pad=0, act=synth.ACT_RELU, name="a"))
    net.add(synth.Layer("fc", a, c * hw * hw, o, bias=True, name="fc"))
    wa = torch.randn(c, c, 1, 1, generator=gen) / c ** 0.5
    wf = torch.randn(o, c * hw * hw, generator=gen) / (c * hw * hw) ** 0.5
    b = torch.randn(o, generator=gen)
    x = torch.randn(batch, c, hw, hw, generator=gen)
    layers = [{"w": wa.cuda(), "b": torch.zeros(c, device="cuda")}, {"w": wf.cuda(), "b": b.cuda()}]
    ref = torch.relu(torch.nn.functional.conv2d(x.double(), wa.double())).flatten(1) @ wf.double().T + b.double()
    return net, layers, x, ref


@pytest.mark.parametrize("c,hw,o,batch,split", [(256, 7, 1000, 32, False), (256, 7, 1000, 64, False), (200, 6, 700, 64, False),
                                                (128, 4, 512, 64, True)])
def test_fully_connected_layer_on_a_map(c, hw, o, batch, split):
    """A window that covers a 7x7 map leaves the split kernel two images per block, each block reading all weights: 65.8 us for
    256 -> 1000 at batch 32, the general kernel 33.5.  On a 4x4 map eight fit, and it is the faster one."""
    net, layers, x, ref = _fc_net(c, hw, o, batch)
    B.cprune_clear_tile_cache()
    handle = pipeline.build_net(net, layers, batch, B.F32, tune=False)
    name = B.cprune_tile_variant_name(handle.layer_variant(1), True, B.F32)
    y = handle.forward(x.cuda()).double().cpu()
    handle.close()
    assert ("conv_split" in name) == split, name
    assert float((y - ref).norm() / ref.norm()) < 2e-6      # 12544 terms in fp32


@pytest.mark.parametrize("shape", [(1, 16, 8, 24, 3, 1), (2, 64, 14, 45, 3, 2), (1, 256, 14, 300, 3, 1), (10, 54, 54, 5, 5, 1)])
@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_timing_tries_every_variant_that_runs(shape, dtype):
    """cprune_select_tile times each variant that runs the layer and fits the scratch; the split kernel, which costs a launch
    more per call, from 0.3 GFLOP up."""
    n, c, hw, o, k, stride = shape
    large = 2 * n * o * c * k * k * (-(-hw // stride)) ** 2 >= 3e8
    td = B.TORCH_DTYPE[dtype]
    x, w = torch.randn(n, c, hw, hw, device="cuda").to(td), torch.randn(o, c, k, k, device="cuda").to(td)
    d = B.conv_desc(x.shape, w.shape, stride, k // 2, 1, dtype)
    B.cprune_clear_tile_cache()
    best, _, ms = B.cprune_select_tile(d, x, w, iters=2)
    assert ms[best] > 0
    for v in range(B.cprune_num_tile_variants()):
        try:
            B.cprune_conv2d_bn_relu(d, x, w, None, None, v)
            runs = True
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            runs = False
        if "conv_split" in B.cprune_tile_variant_name(v, False, dtype):
            runs = runs and large
        assert (ms[v] > 0) == runs, (v, B.cprune_tile_variant_name(v, False, dtype))
    B.cprune_clear_tile_cache()


@pytest.mark.parametrize("timed", [False, True])
def test_a_call_takes_the_scratch_of_the_variant_it_runs(timed, monkeypatch):
    """cprune_conv2d_bn_relu without scratch of the caller's: what the chosen variant needs, not what the most demanding would."""
    x, w = torch.randn(8, 128, 56, 56, device="cuda"), torch.randn(83, 128, 3, 3, device="cuda") * 0.03
    d = B.conv_desc(x.shape, w.shape, 1, 1, 1, B.F32, B.ACT_NONE)
    B.cprune_clear_tile_cache()
    if timed:
        B.cprune_select_tile(d, x, w, iters=2)
    v, was_timed = B.cprune_cached_tile(d)
    assert was_timed == timed
    need, asked = B.cprune_conv_workspace_bytes(d, v), []
    make = B._ws
    monkeypatch.setattr(B, "_ws", lambda nbytes, device: asked.append(nbytes) or make(nbytes, device))
    y = B.cprune_conv2d_bn_relu(d, x, w)
    assert asked == [need] and need < B.cprune_conv_workspace_bytes(d, -1) // 10
    assert torch.equal(y, B.cprune_conv2d_bn_relu(d, x, w, None, None, v))
    B.cprune_clear_tile_cache()
