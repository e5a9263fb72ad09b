"""The row-strip kernel (3x3 / stride 1 / pad 1, 16-bit data, inside a handle) at the sizes where its strips can go wrong: one
strip of 16 columns, one column more, ragged rows, two and four images side by side with the last one missing, one chunk of
channels and fewer chunks than wavefronts, filter tiles of one to four blocks with a partial last block; with and without a
fused 2x2 max-pool and a shortcut.  Every variant that accepts the layer, against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import nmax

pytestmark = pytest.mark.gpu


def _rows_variants(dtype):
    return [v for v in range(B.cprune_num_tile_variants()) if "conv_rows" in B.cprune_tile_variant_name(v, True, dtype)]


@pytest.mark.parametrize("dtype", [B.F16, B.BF16])
@pytest.mark.parametrize("cfg", [
    # c_in, c_out, hw, batch, pool, shortcut
    (32, 16, 16, 1, False, False),     # one strip, one chunk, one block
    (33, 17, 17, 2, False, True),      # one column into the second strip, a channel into the second chunk
    (40, 50, 31, 1, False, False),     # edge columns on both sides, ragged rows
    (72, 33, 33, 2, False, True),      # three strips
    (130, 48, 7, 3, False, True),      # two images per strip, one missing; five chunks
    (260, 70, 8, 5, False, False),     # eight columns: the images of a strip touch
    (70, 65, 4, 6, False, True),       # four images per strip, two missing
    (300, 20, 3, 3, False, False),     # three columns of four lanes
    (48, 40, 32, 2, True, False),      # pool, two strips
    (64, 30, 18, 1, True, False),      # pool, ragged strip
    (96, 36, 8, 3, True, False),       # pool, two images
    (160, 24, 4, 5, True, False),      # pool, four images
    (20, 24, 6, 3, True, False),
])
def test_rows_variants(orc, cfg, dtype):
    c_in, c_out, hw, batch, pool, shortcut = cfg
    print(cfg, dtype, flush=True)
    net = synth.NetSpec(f"rows_{c_in}_{c_out}_{hw}_{pool}", 3, hw, hw)
    a = net.add(synth.Layer("conv", -1, 3, c_in, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    r = net.add(synth.Layer("conv", -1, 3, c_out, k=1, act=synth.ACT_NONE, bn=True, name="r")) if shortcut else None
    b = net.add(synth.Layer("conv", a, c_in, c_out, k=3, stride=1, pad=1, act=synth.ACT_RELU, bn=True, residual=r, name="b"))
    if pool:
        p = net.add(synth.Layer("maxpool", b, c_out, c_out, k=2, stride=2, name="p"))
        net.add(synth.Layer("conv", p, c_out, 8, k=1, act=synth.ACT_NONE, bn=True, name="c"))
    params = synth.layer_params(net, 80)
    x = synth.net_input(net, 80, batch)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    ran = 0
    assert handle.layer_variant(b) in _rows_variants(dtype)          # the untimed choice
    for v in _rows_variants(dtype):
        try:
            handle.set_layer_variant(b, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        out = handle.forward(xd)
        torch.cuda.synchronize()
        err = nmax(out.float().cpu().numpy(), ref)
        assert err < 2e-2, (B.cprune_tile_variant_name(v, True, dtype), err)
        ran += 1
    assert ran >= 5
    handle.close()


@pytest.mark.parametrize("hw,batch", [(8, 2), (4, 4), (17, 1)])
def test_rows_neighbours_do_not_leak(hw, batch):
    """An infinity in one image of a strip leaves the others bit for bit, and one pixel reaches its 3x3 neighbours only."""
    net = synth.NetSpec(f"rowsleak_{hw}", 16, hw, hw)
    a = net.add(synth.Layer("conv", -1, 16, 40, k=1, act=synth.ACT_NONE, bn=True, name="a"))
    net.add(synth.Layer("conv", a, 40, 24, k=3, stride=1, pad=1, act=synth.ACT_NONE, bn=True, name="b"))
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(synth.layer_params(net, 81)), B.BF16)
    handle = pipeline.build_net(net, layers, batch, B.BF16, tune=False)
    x = torch.from_numpy(synth.net_input(net, 81, batch)).cuda().to(torch.bfloat16)
    for v in _rows_variants(B.BF16):
        try:
            handle.set_layer_variant(1, v)
        except B.CPruneError:
            continue
        want = handle.forward(x).clone()
        for px in ((0, 0), (hw - 1, hw - 1), (hw // 2, min(15, hw - 1))):
            xb = x.clone()
            xb[batch - 1, :, px[0], px[1]] = float("inf")
            got = handle.forward(xb)
            torch.cuda.synchronize()
            near = torch.zeros(got.shape, dtype=torch.bool, device="cuda")
            near[batch - 1, :, max(0, px[0] - 1):px[0] + 2, max(0, px[1] - 1):px[1] + 2] = True
            assert torch.equal(got[~near], want[~near]), (v, px)
    handle.close()


@pytest.mark.parametrize("cfg", [
    # c_in, c_out, hw, batch, pool, shortcut
    (32, 16, 16, 1, False, False),     # one strip, one chunk, one block
    (33, 17, 17, 2, False, True),      # one column into the second strip, a channel into the second chunk
    (40, 50, 30, 1, False, False),     # strips of 14 new columns: two exactly
    (24, 20, 31, 2, False, True),      # and one column more, ragged rows
    (130, 48, 7, 3, False, True),      # two images per strip, one missing; five chunks
    (260, 70, 8, 5, False, False),     # eight columns: the images of a strip touch
    (70, 65, 4, 6, False, True),       # four images per strip, two missing
    (300, 20, 3, 3, False, False),     # three columns of four lanes, eight wavefronts share a strip
    (48, 40, 28, 2, True, False),      # pool: strips of 12 new columns, two exactly
    (64, 30, 30, 1, True, False),      # pool, two columns more
    (40, 24, 18, 2, True, False),      # pool, ragged strip
    (96, 36, 8, 3, True, False),       # pool, two images
    (160, 24, 4, 5, True, False),      # pool, four images
    (20, 24, 6, 3, True, False),       # pool, six of eight lanes
])
def test_split_rows_variants(orc, cfg):
    """The fp32 kernel, whose strips overlap where a map is wider than 16.  Its sums of at most 2700 terms are off by less than 1e-6
    of their largest; 1e-5 leaves room for the layers around it."""
    c_in, c_out, hw, batch, pool, shortcut = cfg
    print(cfg, flush=True)
    net = synth.NetSpec(f"rows3_{c_in}_{c_out}_{hw}_{pool}", 3, hw, hw)
    a = net.add(synth.Layer("conv", -1, 3, c_in, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    r = net.add(synth.Layer("conv", -1, 3, c_out, k=1, act=synth.ACT_NONE, bn=True, name="r")) if shortcut else None
    b = net.add(synth.Layer("conv", a, c_in, c_out, k=3, stride=1, pad=1, act=synth.ACT_RELU, bn=True, residual=r, name="b"))
    if pool:
        p = net.add(synth.Layer("maxpool", b, c_out, c_out, k=2, stride=2, name="p"))
        net.add(synth.Layer("conv", p, c_out, 8, k=1, act=synth.ACT_NONE, bn=True, name="c"))
    params = synth.layer_params(net, 82)
    x = synth.net_input(net, 82, batch)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params))
    handle = pipeline.build_net(net, layers, batch, tune=False)
    xd = torch.from_numpy(x).cuda()
    ran = []
    for v in range(B.cprune_num_tile_variants()):
        if "conv_split_rows" not in B.cprune_tile_variant_name(v, True, B.F32):
            continue
        try:
            handle.set_layer_variant(b, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        out = handle.forward(xd)
        torch.cuda.synchronize()
        err = nmax(out.cpu().numpy(), ref)
        assert err < 1e-5, (B.cprune_tile_variant_name(v, True, B.F32), err)
        ran.append(v)
    assert len(ran) >= 2, ran        # tall and low strips, more with wavefronts that share a strip
    handle.close()


@pytest.mark.parametrize("dtype", [B.F32, B.F16, B.BF16])
@pytest.mark.parametrize("c_out", [45, 46, 48])
def test_a_dense_map_of_logits_is_written_filter_by_filter(orc, c_out, dtype):
    """A network that ends in a 3x3 layer on a 1x1 map has its logits written without padding: a kernel that stores four filters at
    a time takes it only where a multiple of four filters is left.  Nothing behind the logits is touched."""
    batch = 5
    net = synth.NetSpec(f"rows_logits_{c_out}", 3, 1, 1)
    a = net.add(synth.Layer("conv", -1, 3, 24, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    b = net.add(synth.Layer("conv", a, 24, c_out, k=3, stride=1, pad=1, act=synth.ACT_NONE, bn=True, name="b"))
    params = synth.layer_params(net, 83)
    x = synth.net_input(net, 83, batch)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    taken = []
    for v in [-1] + list(range(B.cprune_num_tile_variants())):
        if v >= 0:
            if "_rows_kernel" not in B.cprune_tile_variant_name(v, True, dtype):
                continue
            try:
                handle.set_layer_variant(b, v)
            except B.CPruneError as e:
                assert e.status == B.ERR_UNSUPPORTED
                continue
            taken.append(v)
            if c_out % 4:
                continue                 # (must not be reached; not run)
        out = torch.full((batch * c_out + 64,), 7.0, dtype=B.TORCH_DTYPE[dtype], device="cuda")
        handle.forward(xd, logits=out)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy()
        assert (got[batch * c_out:] == 7.0).all(), v
        assert nmax(got[:batch * c_out].reshape(ref.shape), ref) < (1e-5 if dtype == B.F32 else 2e-2), v
    assert bool(taken) == (c_out % 4 == 0), taken
    handle.close()


@pytest.mark.parametrize("c_in,runs", [(1, False), (2, True)])
def test_split_rows_need_as_many_terms_as_the_split_kernel(c_in, runs):
    """Three parts are for fp32 sums of at least 16 terms: nine (one channel that is left) stay with the fp32 instruction, timed or
    not, and sums of 18 are as exact in parts (2-norm error against 64 bits at most 1.1 times the instruction's, or half a unit)."""
    gen = torch.Generator().manual_seed(c_in)
    net = synth.NetSpec(f"rows_terms_{c_in}", 16, 56, 56)
    a = net.add(synth.Layer("conv", -1, 16, c_in, k=1, act=synth.ACT_NONE, name="a"))
    b = net.add(synth.Layer("conv", a, c_in, 128, k=3, stride=1, pad=1, act=synth.ACT_NONE, name="b"))
    wa, wb = torch.randn(c_in, 16, 1, 1, generator=gen), torch.randn(128, c_in, 3, 3, generator=gen)
    layers = [{"w": wa.cuda(), "b": torch.zeros(c_in).cuda()}, {"w": wb.cuda(), "b": torch.zeros(128).cuda()}]
    x = torch.randn(48, 16, 56, 56, generator=gen).cuda()
    B.cprune_clear_tile_cache()
    for tune in (False, True):
        handle = pipeline.build_net(net, layers, 48, B.F32, tune=tune)
        if not runs:
            assert "rows_kernel" not in B.cprune_tile_variant_name(handle.layer_variant(b), True, B.F32)
        if not tune:
            handle.set_layer_variant(b, 0)
            base = handle.forward(x).double().cpu()
            mid = handle.activation(a, 48, (c_in, 56, 56))
            ref = torch.nn.functional.conv2d(mid.double().cpu(), wb.double(), None, 1, 1)
            e_base = float((base - ref).norm() / ref.norm())
            took = 0
            for v in range(B.cprune_num_tile_variants()):
                if "conv_split_rows" not in B.cprune_tile_variant_name(v, True, B.F32):
                    continue
                try:
                    handle.set_layer_variant(b, v)
                except B.CPruneError as e:
                    assert e.status == B.ERR_UNSUPPORTED
                    continue
                e = float((handle.forward(x).double().cpu() - ref).norm() / ref.norm())
                assert e <= max(1.1 * e_base, 2.0 ** -24), (v, e, e_base)
                took += 1
            assert bool(took) == runs
        handle.close()


@pytest.mark.parametrize("cfg", [
    # batch, c_in, h, w, c_out: two images side by side, the last alone; four, two missing; three columns of four lanes; strips that
    # overlap, ragged rows; one column into the second strip; several chunks for wavefronts that share a strip
    (3, 20, 8, 8, 24), (6, 70, 4, 4, 40), (5, 130, 3, 3, 17), (1, 40, 31, 44, 20), (2, 33, 9, 17, 33), (2, 260, 7, 7, 48),
])
def test_split_rows_second_pass(cfg):
    """What three parts do not hold is multiplied again on the fp32 instruction: numbers around 1e-30, as exact as that instruction
    (its least exact variant and 10 %); one infinity, which reaches its 3x3 neighbours of the same image with the sign of the
    weight and leaves everything else (of the same wavefront as well) as exact as before."""
    n, c_in, h, w, c_out = cfg
    gen = torch.Generator().manual_seed(c_in)
    net = synth.NetSpec(f"second_{c_in}_{h}", c_in, h, w)
    net.add(synth.Layer("conv", -1, c_in, c_out, k=3, stride=1, pad=1, act=synth.ACT_NONE, name="a"))
    wt = torch.randn(c_out, c_in, 3, 3, generator=gen) / (4.5 * c_in) ** 0.5
    x = torch.randn(n, c_in, h, w, generator=gen)
    handle = pipeline.build_net(net, [{"w": wt.cuda(), "b": torch.zeros(c_out, device="cuda")}], n, B.F32, tune=False)
    small = x * 1e-30
    bad = []
    for img, py, px in ((n - 1, 0, 0), (0, h - 1, w - 1), (n // 2, h // 2, min(w - 1, 15)), (0, 0, min(w - 1, 13))):
        b = x.clone()
        b[img, c_in // 2, py, px] = float("inf")
        bad.append((b, torch.nn.functional.conv2d(b.double(), wt.double(), None, 1, 1)))
    ref = torch.nn.functional.conv2d(small.double(), wt.double(), None, 1, 1)
    errors, rows = {}, []
    for v in range(B.cprune_num_tile_variants()):
        name = B.cprune_tile_variant_name(v, True, B.F32)
        if "conv_split" in name and "rows" not in name:
            continue
        try:
            handle.set_layer_variant(0, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        print(cfg, name, flush=True)
        y = handle.forward(small.cuda()).double().cpu()
        errors[v] = float((y - ref).norm() / ref.norm())
        if "rows" not in name:
            continue
        rows.append(v)
        for b, want in bad:
            got = handle.forward(b.cuda()).double().cpu()
            inf = want.isinf()
            assert not want.isnan().any() and torch.equal(got[inf], want[inf]), name
            assert float((got[~inf] - want[~inf]).norm() / want[~inf].norm()) < 1e-6, name
    base = max(e for v, e in errors.items() if v not in rows)
    assert len(rows) >= 2
    for v in rows:
        assert errors[v] <= 1.1 * base, (v, errors[v], base)
    handle.close()
