"""Inverted-residual blocks as one kernel, and their depthwise + 1x1 half alone, at the sizes where strips of 16 columns x a few
rows can go wrong: maps of one strip, one column more, odd rows at the bottom, eight lanes per row (two images side by side,
the second one missing), fewer chunks of channels than wavefronts, several filter tiles.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import nmax

pytestmark = pytest.mark.gpu

TOL = {B.F32: 1e-4, B.F16: 2e-2, B.BF16: 2e-2}


def _block(c_in, c_exp, c_out, hw, k, stride, shortcut):
    net = synth.NetSpec(f"strip_{c_in}_{c_exp}_{c_out}_{hw}_{k}_{stride}", 3, hw, hw)
    a = net.add(synth.Layer("conv", -1, 3, c_in, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    e = net.add(synth.Layer("conv", a, c_in, c_exp, k=1, act=synth.ACT_RELU, bn=True, name="e"))
    d = net.add(synth.Layer("conv", e, c_exp, c_exp, k=k, stride=stride, pad=k // 2, groups=c_exp, act=synth.ACT_RELU6,
                            bn=True, name="d"))
    net.add(synth.Layer("conv", d, c_exp, c_out, k=1, act=synth.ACT_NONE, bn=True, residual=a if shortcut else None, name="p"))
    return net, e, d


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("cfg", [
    # c_in, c_exp, c_out, hw, k, stride, shortcut, batch
    (16, 16, 16, 16, 3, 1, True, 1),       # one strip wide, a single chunk
    (16, 36, 24, 17, 3, 1, False, 3),      # one column into the second strip
    (24, 50, 24, 31, 3, 1, True, 2),       # three strips, ragged rows
    (24, 40, 32, 33, 3, 2, False, 2),      # stride 2: 17 output columns
    (32, 33, 33, 7, 3, 1, False, 3),       # two images per strip, the last one alone
    (32, 90, 64, 14, 3, 2, False, 5),      # stride 2 onto 7 columns: two images per strip
    (32, 44, 32, 8, 3, 1, True, 2),        # eight columns: too wide to share
    (16, 40, 40, 6, 5, 1, False, 3),       # 5x5 window, two images per strip
    (40, 70, 40, 29, 5, 1, True, 1),       # 5x5, three strips
    (16, 48, 40, 27, 5, 2, False, 2),      # 5x5, stride 2, odd map
    (8, 20, 100, 9, 3, 1, False, 2),       # widest built filter tile
    (8, 260, 24, 5, 3, 1, False, 1),       # many chunks, one small strip: eight wavefronts share it
    (8, 24, 20, 2, 3, 1, False, 2),        # a 2x2 map: most neighbours are padding
])
def test_block_strips(orc, cfg, dtype):
    c_in, c_exp, c_out, hw, k, stride, shortcut, batch = cfg
    print(cfg, dtype, flush=True)
    net, e, d = _block(c_in, c_exp, c_out, hw, k, stride, shortcut)
    params = synth.layer_params(net, 70)
    x = synth.net_input(net, 70, batch)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    for form in ("block", "depthwise", "apart"):
        if form == "block":
            handle.fuse_block(d, True)
        else:
            handle.fuse_depthwise(d, form == "depthwise")
        assert handle.layer_fused(e) == (form == "block") and handle.layer_fused(d) == (form != "apart")
        out = handle.forward(xd)
        torch.cuda.synchronize()
        err = nmax(out.float().cpu().numpy(), ref)
        assert err < TOL[dtype], (form, err)
    handle.close()


def test_depthwise_half_with_several_filter_tiles(orc):
    """300 projection filters: three filter tiles, each with the depthwise half of its own."""
    net, e, d = _block(16, 60, 300, 15, 3, 1, False)
    params = synth.layer_params(net, 71)
    x = synth.net_input(net, 71, 2)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), B.F32)
    handle = pipeline.build_net(net, layers, 2, B.F32, tune=False)
    handle.fuse_depthwise(d, True)
    out = handle.forward(torch.from_numpy(x).cuda())
    torch.cuda.synchronize()
    assert nmax(out.cpu().numpy(), ref) < 1e-4
    handle.close()


@pytest.mark.parametrize("form", ["block", "depthwise"])
@pytest.mark.parametrize("hw,k,stride", [(7, 3, 1), (14, 3, 2), (6, 5, 1)])
def test_images_of_one_strip_do_not_meet(hw, k, stride, form):
    """Two images share a strip's 16 columns: infinities in one leave the other's result as it was, bit for bit."""
    net, e, d = _block(16, 40, 24, hw, k, stride, False)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(synth.layer_params(net, 72)), B.F32)
    handle = pipeline.build_net(net, layers, 2, B.F32, tune=False)
    (handle.fuse_block if form == "block" else handle.fuse_depthwise)(d, True)
    x = torch.from_numpy(synth.net_input(net, 72, 2)).cuda()
    want = handle.forward(x).clone()
    for bad in (0, 1):
        xb = x.clone()
        xb[bad] = float("inf")
        got = handle.forward(xb).clone()
        torch.cuda.synchronize()
        assert torch.equal(got[1 - bad], want[1 - bad]), bad
    handle.close()


@pytest.mark.parametrize("dtype", [B.F32, B.F16, B.BF16])
@pytest.mark.parametrize("cfg", [(3, 32, 16, 224, 4), (3, 27, 24, 150, 3), (1, 40, 32, 131, 2)])
def test_first_layer_in_the_block(orc, cfg, dtype):
    """A 3x3 / stride 2 first layer, the depthwise layer and the projection behind it, as a tuned handle runs them (one kernel
    where it times faster; forced in test_pinned_image_form): even and odd images, one channel, ragged filter counts."""
    c, c_exp, c_out, hw, batch = cfg
    net = synth.NetSpec(f"first_{c}_{c_exp}_{c_out}_{hw}", c, hw, hw)
    e = net.add(synth.Layer("conv", -1, c, c_exp, k=3, stride=2, pad=1, act=synth.ACT_RELU6, bn=True, name="e"))
    d = net.add(synth.Layer("conv", e, c_exp, c_exp, k=3, stride=1, pad=1, groups=c_exp, act=synth.ACT_RELU6, bn=True, name="d"))
    net.add(synth.Layer("conv", d, c_exp, c_out, k=1, act=synth.ACT_NONE, bn=True, name="p"))
    params = synth.layer_params(net, 73)
    x = synth.net_input(net, 73, batch)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=True)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    print(cfg, dtype, "one kernel:", handle.layer_fused(e), flush=True)
    for n in (batch, 1):
        for graph in (False, True):
            out = handle.forward(xd[:n].contiguous(), use_graph=graph)
            torch.cuda.synchronize()
            assert nmax(out.float().cpu().numpy(), ref[:n]) < TOL[dtype]
    if handle.layer_fused(e):
        handle.fuse_block(d, False)                 # the first layer on its own again
        assert not handle.layer_fused(e) and handle.layer_fused(d)
        with pytest.raises(B.CPruneError):
            handle.fuse_block(d, True)
        out = handle.forward(xd)
        torch.cuda.synchronize()
        assert nmax(out.float().cpu().numpy(), ref) < TOL[dtype]
    handle.close()


@pytest.mark.parametrize("dtype", [B.F32, B.F16, B.BF16])
@pytest.mark.parametrize("cfg", [
    # c_in, c_exp, c_out, hw, k, stride, shortcut, batch: every height of strips (7 and 4 rows, 5 and 3, 3 and 2; stride 2: 4 and 2;
    # 5x5: 4 and 2), maps a row more or less than whole strips, fewer chunks than wavefronts
    (24, 50, 24, 15, 3, 1, True, 2),
    (16, 70, 60, 28, 3, 1, False, 1),
    (90, 70, 90, 16, 3, 1, True, 1),
    (40, 140, 100, 7, 3, 1, False, 3),
    (24, 40, 32, 33, 3, 2, False, 2),
    (32, 90, 64, 14, 3, 2, False, 5),
    (40, 60, 90, 18, 3, 2, False, 1),
    (16, 40, 30, 9, 5, 1, False, 3),
    (40, 70, 40, 29, 5, 1, True, 1),
    (16, 48, 40, 27, 5, 2, False, 2),
    (40, 70, 120, 13, 5, 2, False, 1),
])
def test_pinned_block_forms(orc, cfg, dtype):
    """Tall and low strips with 1, 2, 4 and 8 wavefronts each, the whole block and its depthwise half, 5x5 halves also on pixel blocks,
    against the oracle, and a smaller batch.  The forms round alike from step to step and differ in the order of the projection's sums only."""
    c_in, c_exp, c_out, hw, k, stride, shortcut, batch = cfg
    net, e, d = _block(c_in, c_exp, c_out, hw, k, stride, shortcut)
    params = synth.layer_params(net, 74)
    x = synth.net_input(net, 74, batch)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    pinned = [(form, tile, ks) for form in (2, 1) for tile in (0, 1) for ks in (1, 2, 4, 8)]
    for form, tile, ks in pinned + ([(1, 2, 4), (1, 2, 8)] if k == 5 else []):
        print(cfg, dtype, form, tile, ks, flush=True)
        handle.block_form(d, form, tile, ks)
        assert handle.layer_fused(e) == (form == 2) and handle.layer_fused(d)
        for n in (batch, 1):
            out = handle.forward(xd[:n].contiguous())
            torch.cuda.synchronize()
            err = nmax(out.float().cpu().numpy(), ref[:n])
            assert err < TOL[dtype], (form, tile, ks, n, err)
    handle.block_form(d, 0)
    assert not handle.layer_fused(e) and not handle.layer_fused(d)
    out = handle.forward(xd)
    torch.cuda.synchronize()
    assert nmax(out.float().cpu().numpy(), ref) < TOL[dtype]
    handle.close()


@pytest.mark.parametrize("dtype", [B.F32, B.F16, B.BF16])
@pytest.mark.parametrize("cfg", [
    # channels, first layer, projection, image, batch: even and odd images, one and two channels, maps of one strip, one column more
    # and a row more or less than whole strips, one and two filter blocks
    (3, 32, 16, 224, 2), (3, 27, 24, 61, 3), (1, 40, 32, 33, 2), (2, 20, 9, 31, 1), (3, 70, 17, 19, 5), (3, 5, 32, 57, 1),
])
def test_pinned_image_form(orc, cfg, dtype):
    """The network's first layer inside the first block's kernel, on request: tall and low strips, every number of wavefronts, a
    smaller batch, a replayed graph, and back to the first layer on its own, whose activation can be read again."""
    c, c_exp, c_out, hw, batch = cfg
    net = synth.NetSpec(f"image_{c}_{c_exp}_{c_out}_{hw}", c, hw, hw)
    e = net.add(synth.Layer("conv", -1, c, c_exp, k=3, stride=2, pad=1, act=synth.ACT_RELU6, bn=True, name="e"))
    d = net.add(synth.Layer("conv", e, c_exp, c_exp, k=3, stride=1, pad=1, groups=c_exp, act=synth.ACT_RELU6, bn=True, name="d"))
    net.add(synth.Layer("conv", d, c_exp, c_out, k=1, act=synth.ACT_NONE, bn=True, name="p"))
    params = synth.layer_params(net, 75)
    x = synth.net_input(net, 75, batch)
    ref_layers, _ = orc.prune_net(net, params)
    acts = orc.forward(net, ref_layers, x, return_all=True)
    ref = acts[-1]
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    for low in (0, 1):
        for ks in (1, 2, 4, 8):
            print(cfg, dtype, low, ks, flush=True)
            handle.block_form(d, 2, low, ks)
            assert handle.layer_fused(e) and handle.layer_fused(d)
            for n in (batch, 1):
                for graph in (False, True):
                    out = handle.forward(xd[:n].contiguous(), use_graph=graph)
                    torch.cuda.synchronize()
                    assert nmax(out.float().cpu().numpy(), ref[:n]) < TOL[dtype], (low, ks, n, graph)
    with pytest.raises(B.CPruneError):
        handle.activation(e, batch, acts[e].shape[1:])
    for form in (1, 0, 2, 0):
        handle.block_form(d, form)
        assert handle.layer_fused(e) == (form == 2) and handle.layer_fused(d) == (form > 0)
        out = handle.forward(xd)
        torch.cuda.synchronize()
        assert nmax(out.float().cpu().numpy(), ref) < TOL[dtype]
    assert nmax(handle.activation(e, batch, acts[e].shape[1:]).float().cpu().numpy(), acts[e]) < TOL[dtype]
    handle.close()


def test_block_form_refuses_what_it_cannot_run():
    """A depthwise layer behind the image, a block wider than the kernel is built for, values out of range; and a layer that runs
    inside another block's kernel."""
    net = synth.NetSpec("forms", 8, 20, 20)
    a = net.add(synth.Layer("conv", -1, 8, 16, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    d1 = net.add(synth.Layer("conv", a, 16, 16, k=3, stride=1, pad=1, groups=16, act=synth.ACT_RELU, bn=True, name="d1"))
    b = net.add(synth.Layer("conv", d1, 16, 24, k=1, act=synth.ACT_RELU, bn=True, name="b"))
    d2 = net.add(synth.Layer("conv", b, 24, 24, k=3, stride=1, pad=1, groups=24, act=synth.ACT_RELU, bn=True, name="d2"))
    c = net.add(synth.Layer("conv", d2, 24, 100, k=1, act=synth.ACT_RELU, bn=True, name="c"))
    d3 = net.add(synth.Layer("conv", c, 100, 100, k=3, stride=1, pad=1, groups=100, act=synth.ACT_RELU, bn=True, name="d3"))
    net.add(synth.Layer("conv", d3, 100, 300, k=1, act=synth.ACT_NONE, bn=True, name="p"))
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(synth.layer_params(net, 76)), B.F32)
    handle = pipeline.build_net(net, layers, 1, B.F32, tune=False)
    x = torch.from_numpy(synth.net_input(net, 76, 1)).cuda()

    def refused(status, *args):
        with pytest.raises(B.CPruneError) as e:
            handle.block_form(*args)
        assert e.value.status == status, args

    for layer in (d1, d2, d3):
        handle.block_form(layer, 0)
    want = handle.forward(x).clone()
    for bad in ((d2, 3, 0, 1), (d2, -1, 0, 1), (d2, 2, 3, 1), (d2, 2, 0, 3), (d2, 2, 0, 16), (99, 1, 0, 1)):
        refused(B.ERR_INVALID_ARG, *bad)
    refused(B.ERR_UNSUPPORTED, a, 1, 1, 1)               # no depthwise layer
    refused(B.ERR_UNSUPPORTED, d2, 1, 2, 4)              # pixel blocks are for 5x5 windows
    refused(B.ERR_UNSUPPORTED, d2, 2, 2, 4)              # without an expansion
    refused(B.ERR_UNSUPPORTED, d1, 2, 1, 1)              # reads a layer on the image
    refused(B.ERR_UNSUPPORTED, d3, 2, 1, 1)              # 300 filters: the whole block is built for up to 128
    handle.block_form(d1, 1)
    refused(B.ERR_UNSUPPORTED, d2, 2, 1, 1)              # its expansion already runs the first depthwise layer
    handle.block_form(d1, 0)
    handle.block_form(d2, 2, 0, 2)
    refused(B.ERR_UNSUPPORTED, d1, 1, 1, 1)              # and the other way round
    handle.block_form(d3, 1, 0, 2)
    got = handle.forward(x)
    torch.cuda.synchronize()
    assert float((got - want).norm() / want.norm()) < 1e-5
    handle.close()


def test_a_1x1_layer_between_two_depthwise_layers():
    """It is the projection of the first and the expansion of the second: whichever form is asked for last, no layer is left out."""
    net = synth.NetSpec("between", 8, 20, 20)
    a = net.add(synth.Layer("conv", -1, 8, 16, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    d1 = net.add(synth.Layer("conv", a, 16, 16, k=3, stride=1, pad=1, groups=16, act=synth.ACT_RELU, bn=True, name="d1"))
    b = net.add(synth.Layer("conv", d1, 16, 24, k=1, act=synth.ACT_RELU, bn=True, name="b"))
    d2 = net.add(synth.Layer("conv", b, 24, 24, k=3, stride=1, pad=1, groups=24, act=synth.ACT_RELU, bn=True, name="d2"))
    net.add(synth.Layer("conv", d2, 24, 20, k=1, act=synth.ACT_NONE, bn=True, name="c"))
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(synth.layer_params(net, 77)), B.F32)
    handle = pipeline.build_net(net, layers, 2, B.F32, tune=False)
    x = torch.from_numpy(synth.net_input(net, 77, 2)).cuda()
    want = handle.forward(x).clone()
    for step, fused in ((lambda: handle.fuse_block(d2, True), (d1, 0, b, 1, d2, 1)),
                        (lambda: handle.fuse_depthwise(d1, True), (d1, 1, b, 0, d2, 1)),
                        (lambda: handle.fuse_block(d2, True), (d1, 0, b, 1, d2, 1)),
                        (lambda: handle.fuse_depthwise(d1, False), (d1, 0, b, 1, d2, 1)),
                        (lambda: handle.fuse_depthwise(d1, True), (d1, 1, b, 0, d2, 1)),
                        (lambda: handle.fuse_block(d2, False), (d1, 1, b, 0, d2, 1)),
                        (lambda: handle.fuse_depthwise(d2, False), (d1, 1, b, 0, d2, 0))):
        step()
        for i, on in zip(fused[::2], fused[1::2]):
            assert handle.layer_fused(i) == bool(on), (fused, i)
        handle.forward(torch.zeros_like(x))                 # (what an earlier form left in a buffer does not help)
        got = handle.forward(x + 0)
        torch.cuda.synchronize()
        assert float((got - want).norm() / want.norm()) < 1e-5, fused
    handle.close()
