"""A handle built for a full batch runs every smaller batch with the variants chosen for the full one."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [B.F32, B.F16, B.BF16])
def test_every_smaller_batch(orc, dtype):
    """VGG-16 built (and timed) for 9 images: 1, 2, 5 and 8 of them give the full batch's logits."""
    net = synth.vgg16(10, 32)
    params = synth.layer_params(net, 71)
    x = synth.net_input(net, 71, 9)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, 9, dtype, tune=True)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    for n in (1, 2, 5, 8, 9):
        for graph in (False, True):
            out = handle.forward(xd[:n].contiguous(), use_graph=graph)
            torch.cuda.synchronize()
            check(out.float().cpu().numpy(), ref[:n], dtype, f"batch {n} of 9, graph {graph}")
    handle.close()


@pytest.mark.parametrize("tune", [True, False])
@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_smaller_batches_choose_their_own_tiles(orc, dtype, tune):
    """ResNet-18 on 32x32 images, built for 24: whatever a smaller batch runs, and in whatever order batches come, its logits
    are the full batch's."""
    net = synth.resnet18(10, 32, cifar_stem=True)
    params = synth.layer_params(net, 72)
    x = synth.net_input(net, 72, 24)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    B.cprune_clear_tile_cache()
    handle = pipeline.build_net(net, layers, 24, dtype, tune=tune)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    for n in (1, 24, 3, 11, 21, 1, 23, 24):
        out = handle.forward(xd[:n].contiguous(), use_graph=n == 3)
        torch.cuda.synchronize()
        check(out.float().cpu().numpy(), ref[:n], dtype, f"batch {n} of 24, tune {tune}")
    handle.close()


def _rows_layer(full):
    """One 3x3 layer of 32 channels (a single chunk of the row-strip kernel, whose variants then all add in one order) on 56x56."""
    gen = torch.Generator().manual_seed(5)
    net = synth.NetSpec("rows_at_batch", 32, 56, 56)
    net.add(synth.Layer("conv", -1, 32, 128, k=3, stride=1, pad=1, act=synth.ACT_RELU, name="c"))
    layers = [{"w": (torch.randn(128, 32, 3, 3, generator=gen) / 12.0).cuda(), "b": torch.zeros(128, device="cuda")}]
    return net, layers, torch.randn(full, 32, 56, 56, generator=gen).cuda()


def test_row_strips_at_every_smaller_batch():
    """A handle whose layer runs the fp32 row-strip kernel at its full batch has no other packed copy: every smaller batch runs
    that kernel too, which shows in the bits (the general kernel's fp32 instruction gives others)."""
    net, layers, x = _rows_layer(12)
    B.cprune_clear_tile_cache()
    handle = pipeline.build_net(net, layers, 12, B.F32, tune=False)
    rows = [v for v in range(B.cprune_num_tile_variants()) if B.cprune_tile_variant_name(v, True, B.F32) == "conv_split_rows_kernel<8, 1>"]
    handle.set_layer_variant(0, 0)
    general = handle.forward(x).clone()
    done = 0
    for v in rows:
        try:
            handle.set_layer_variant(0, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        want = handle.forward(x).clone()
        assert not torch.equal(want, general)
        for n in range(1, 13):
            assert torch.equal(handle.forward(x[:n].contiguous()), want[:n]), n
        done += 1
    assert done == 1
    handle.close()
    # likewise where the full batch's choice was not timed, down to sizes where the split kernel would be the choice if it were there
    handle = pipeline.build_net(net, layers, 12, B.F32, tune=False)
    assert "conv_split_rows" in B.cprune_tile_variant_name(handle.layer_variant(0), True, B.F32)
    for n in range(1, 13):
        assert torch.equal(handle.forward(x[:n].contiguous()), want[:n]), n
    handle.close()
    # at any batch as the full one
    for full in (7, 8, 9):
        handle = pipeline.build_net(net, layers, full, B.F32, tune=False)
        ok = 0
        for v in rows:
            try:
                handle.set_layer_variant(0, v)
                ok += 1
            except B.CPruneError as e:
                assert e.status == B.ERR_UNSUPPORTED
        handle.close()
        assert ok == 1, full


def test_one_image_does_not_run_the_tiles_of_many():
    """One 224x224 image through a timed handle for 32 (365 us on the full batch's tiles, 212 on its own) against an untimed
    handle for one (198 us)."""
    net = synth.resnet18(1000, 224)
    params = pipeline.upload_params(synth.layer_params(net, 73))
    layers, _ = pipeline.prune_net(net, params, B.F32)
    x = torch.randn(1, 3, 224, 224, device="cuda")

    def replay_us(max_batch, tune):
        B.cprune_clear_tile_cache()
        handle = pipeline.build_net(net, layers, max_batch, B.F32, tune=tune)
        best = float("inf")
        for _ in range(4):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            handle.forward(x, use_graph=True)
            start.record()
            for _ in range(10):
                handle.forward(x, use_graph=True)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end) * 100.0)
        handle.close()
        return best

    small = replay_us(1, False)
    large = replay_us(32, True)
    assert large < 1.4 * small, (large, small)
