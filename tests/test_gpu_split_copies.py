"""The split kernel's packed copies of a handle's weights: there for the layers that run it, and only for those."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu


def _net(c, hw, n_layers, k=1):
    gen = torch.Generator().manual_seed(c)
    net, layers, prev = synth.NetSpec("copies", c, hw, hw), [], -1
    for i in range(n_layers):
        prev = net.add(synth.Layer("conv", prev, c, c, k=k, stride=1, pad=k // 2, act=synth.ACT_RELU, name=f"c{i}"))
        layers.append({"w": (torch.randn(c, c, k, k, generator=gen) / (c * k * k / 2) ** 0.5).cuda(), "b": torch.zeros(c, device="cuda")})
    return net, layers


def _reference(layers, x):
    y = x.double()
    for q in layers:
        w = q["w"].double().cpu()
        y = torch.relu(torch.nn.functional.conv2d(y, w, None, 1, w.shape[2] // 2))
    return y


def _is_split(v):
    return "conv_split" in B.cprune_tile_variant_name(v, True, B.F32)


def test_layers_that_do_not_run_the_kernel_keep_no_copy():
    """Each further 1x1 layer of 3072 channels costs its weights, the copy in the reduction-split kernel's order and its map: no
    third one of 1.5 times the weights."""
    used = []
    B.cprune_clear_tile_cache()
    for n_layers in (1, 4):
        net, layers = _net(3072, 4, n_layers)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        handle = pipeline.build_net(net, layers, 1, B.F32, tune=False)
        used.append(before - torch.cuda.mem_get_info()[0])
        assert not any(_is_split(handle.layer_variant(i)) for i in range(n_layers))
        handle.close()
    weights = 3072 * 3072 * 4
    assert (used[1] - used[0]) / 3 < 2.3 * weights, (used, weights)


def test_a_split_variant_can_still_be_pinned():
    """A stored tuning result applied to an untimed handle: the copy is made then, dropped when another variant is pinned."""
    net, layers = _net(96, 9, 2)
    x = torch.randn(2, 96, 9, 9)
    ref = _reference(layers, x)
    B.cprune_clear_tile_cache()
    handle = pipeline.build_net(net, layers, 2, B.F32, tune=False)
    assert not _is_split(handle.layer_variant(0))
    splits = [v for v in range(B.cprune_num_tile_variants()) if _is_split(v)]
    for v in (splits[1], 0, splits[7], splits[7], 0):
        for i in (0, 1):
            handle.set_layer_variant(i, v)
        for n in (2, 1):
            y = handle.forward(x[:n].cuda()).double().cpu()
            assert float((y - ref[:n]).norm() / ref[:n].norm()) < 1e-6, (v, n)
    handle.close()


def test_a_variant_remembered_for_a_smaller_batch_needs_its_copy():
    """A split variant timed by a handle for 16 images does not reach a handle for 32 whose layer has no packed copy."""
    net, layers = _net(128, 28, 1, k=3)
    x = torch.randn(32, 128, 28, 28)
    ref = _reference(layers, x)
    B.cprune_clear_tile_cache()
    small = pipeline.build_net(net, layers, 16, B.F32, tune=True)
    assert _is_split(small.layer_variant(0))
    large = pipeline.build_net(net, layers, 32, B.F32, tune=False)
    large.set_layer_variant(0, 0)
    for handle, n in ((large, 16), (small, 16), (large, 32)):
        y = handle.forward(x[:n].cuda()).double().cpu()
        assert float((y - ref[:n]).norm() / ref[:n].norm()) < 1e-6
    small.close()
    large.close()
    B.cprune_clear_tile_cache()


def test_leaving_a_fused_form_brings_the_copy_back():
    """VGG-16's first two layers as one kernel and apart again, in fp32, where the second runs the split kernel by itself."""
    net = synth.vgg16(10, 32)
    params = synth.layer_params(net, 74)
    params[0]["keep"] = 24                  # the fused form takes at most 32 filters
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), B.F32)
    x = torch.randn(8, 3, 32, 32, device="cuda")
    B.cprune_clear_tile_cache()
    handle = pipeline.build_net(net, layers, 8, B.F32, tune=True)
    handle.fuse_first_layers(False)
    apart = handle.forward(x)
    handle.fuse_first_layers(True)
    fused = handle.forward(x)
    handle.fuse_first_layers(False)
    again = handle.forward(x, use_graph=True)
    torch.cuda.synchronize()
    assert torch.equal(apart, again)
    assert float((fused - apart).norm() / apart.norm()) < 1e-5
    handle.close()


def test_a_16_bit_layer_gives_the_row_strips_copy_back():
    """On maps over 32 the row-strip kernel's copy is made for the layers that run it: pinned to another variant they give it back,
    pinned to that kernel again they answer as before."""
    c, n_layers = 1536, 3
    net, layers = _net(c, 34, n_layers, k=3)
    for q in layers:
        q["w"] = q["w"].to(torch.bfloat16)
    x = torch.randn(1, c, 34, 34).cuda().to(torch.bfloat16)
    B.cprune_clear_tile_cache()
    handle = pipeline.build_net(net, layers, 1, B.BF16, tune=False)
    rows = handle.layer_variant(0)
    assert "conv_rows" in B.cprune_tile_variant_name(rows, True, B.BF16)
    want = handle.forward(x).clone()
    torch.cuda.synchronize()
    with_copies = torch.cuda.mem_get_info()[0]
    for i in range(n_layers):
        handle.set_layer_variant(i, 0)
    general = handle.forward(x).clone()
    torch.cuda.synchronize()
    weights = c * c * 9 * 2
    assert torch.cuda.mem_get_info()[0] - with_copies > 0.9 * n_layers * weights
    for i in range(n_layers):
        handle.set_layer_variant(i, rows)
    again = handle.forward(x)
    torch.cuda.synchronize()
    assert torch.equal(again, want)
    assert float((general.float() - want.float()).norm() / want.float().norm()) < 2e-2
    handle.close()
