"""The row-strip kernel in the boundary's layout through cprune_conv2d_bn_relu, every variant: maps of one pixel up, one to three strips
across, two and four images side by side, part-filled chunks and filter blocks, odd channel counts, 16-bit weights off a 4-byte boundary,
shortcuts; numbers that three parts do not hold; graph replay."""
import pytest
import torch

from paper_2207_01260_amd import binding as B

pytestmark = pytest.mark.gpu
DT = {"f32": B.F32, "f16": B.F16, "bf16": B.BF16}
# fp32: sums rounded once per 32 terms.  16-bit outputs are rounded to nearest: at most half a unit in the last place, 2^-11 (fp16: 11
# significant bits) or 2^-8 (bf16: 8) of an element, and with it of the 2-norm; the sums themselves add less than 1e-5
REL = {"f32": 1e-6, "f16": 2.0 ** -11 + 1e-5, "bf16": 2.0 ** -8 + 1e-5}


def _variants(dtype):
    return [v for v in range(B.cprune_num_tile_variants()) if "conv_rows_nchw" in B.cprune_tile_variant_name(v, False, dtype)]


def _runs(v, dtype, c):
    """Whether a variant runs a layer of c channels: a chunk of 32 for each wavefront that shares a strip, and in fp32 one filter block,
    at most six rows and two wavefronts."""
    blocks, rows, waves = (int(q) for q in B.cprune_tile_variant_name(v, False, dtype).rstrip(">").split(", ")[1:])
    return (waves == 1 or waves <= (c + 31) // 32) and (dtype != B.F32 or (blocks == 1 and rows <= 6 and waves <= 2))


@pytest.mark.parametrize("dtype", sorted(DT))
@pytest.mark.parametrize("cfg", [
    # images, c_in, filters, height, width, shortcut, activation
    (1, 2, 1, 1, 1, False, B.ACT_NONE), (5, 3, 17, 4, 3, True, B.ACT_RELU), (3, 33, 16, 7, 8, False, B.ACT_RELU6),
    (2, 64, 45, 32, 32, False, B.ACT_RELU), (1, 31, 33, 9, 17, True, B.ACT_NONE), (2, 70, 20, 5, 31, False, B.ACT_RELU),
    (9, 129, 50, 3, 4, False, B.ACT_NONE), (1, 200, 36, 14, 14, True, B.ACT_RELU), (2, 97, 83, 13, 45, False, B.ACT_RELU6),
])
def test_every_variant(cfg, dtype):
    n, c, o, h, w, residual, act = cfg
    dt, td = DT[dtype], B.TORCH_DTYPE[DT[dtype]]
    gen = torch.Generator().manual_seed(c * o + h)
    x = torch.randn(n, c, h, w, generator=gen).to(td)
    wt = (torch.randn(o, c, 3, 3, generator=gen) * (2.0 / (9 * c)) ** 0.5).to(td)
    bias = torch.randn(o, generator=gen)
    res = torch.randn(n, o, h, w, generator=gen).to(td) if residual else None
    ref = torch.nn.functional.conv2d(x.double(), wt.double(), bias.double(), 1, 1)
    ref = ref if res is None else ref + res.double()
    ref = ref if act == B.ACT_NONE else ref.clamp(0, 6) if act == B.ACT_RELU6 else ref.clamp(min=0)
    xd, bd, rd = x.cuda(), bias.cuda(), None if res is None else res.cuda()
    room = torch.empty(wt.numel() + 1, device="cuda", dtype=td)
    d = B.conv_desc(x.shape, wt.shape, 1, 1, 1, dt, act, residual)
    for shift in (0, 1):                             # the weights on an odd element, too
        wd = room[shift:shift + wt.numel()].view(wt.shape)
        wd.copy_(wt)
        for v in _variants(dt):
            try:
                y = B.cprune_conv2d_bn_relu(d, xd, wd, bd, rd, v)
            except B.CPruneError as e:
                assert e.status == B.ERR_UNSUPPORTED and not _runs(v, dt, c), v
                continue
            assert _runs(v, dt, c), v
            err = float((y.double().cpu() - ref).norm() / ref.norm())
            assert err < REL[dtype], (B.cprune_tile_variant_name(v, False, dt), shift, err)


@pytest.mark.parametrize("dtype", sorted(DT))
def test_untimed_choice_and_graph_replay(dtype):
    dt, td = DT[dtype], B.TORCH_DTYPE[DT[dtype]]
    x, wt = torch.randn(2, 40, 20, 24, device="cuda").to(td), torch.randn(30, 40, 3, 3, device="cuda").to(td)
    d = B.conv_desc(x.shape, wt.shape, 1, 1, 1, dt, B.ACT_RELU)
    B.cprune_clear_tile_cache()
    for _ in range(2):
        assert "conv_rows_nchw" in B.cprune_tile_variant_name(B.cprune_cached_tile(d)[0], False, dt)
    y = torch.empty(B.out_shape(d), device="cuda", dtype=td)
    B.cprune_conv2d_bn_relu(d, x, wt, y=y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.cprune_conv2d_bn_relu(d, x, wt, y=y)
    for _ in range(3):
        x.copy_(torch.randn(x.shape, device="cuda").to(td))
        want = B.cprune_conv2d_bn_relu(d, x, wt)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


def test_numbers_three_parts_do_not_hold():
    gen = torch.Generator().manual_seed(8)
    c, o, h = 70, 40, 11
    x = torch.randn(3, c, h, h, generator=gen)
    x[0, 3, 4, 4], x[0, 60, 9, 2] = float("inf"), 3.39e38
    x[1] *= 2.0 ** -118
    wt = torch.randn(o, c, 3, 3, generator=gen).cuda()
    d = B.conv_desc(x.shape, wt.shape, 1, 1, 1, B.F32, B.ACT_NONE)
    want = B.cprune_conv2d_bn_relu(d, x.cuda(), wt, tile_variant=0).double().cpu()      # the fp32 instruction
    assert not want[0].isfinite().all() and want[1:].isfinite().all()
    ran = 0
    for v in _variants(B.F32):
        try:
            got = B.cprune_conv2d_bn_relu(d, x.cuda(), wt, tile_variant=v).double().cpu()
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED and not _runs(v, B.F32, c), v
            continue
        ran += 1
        assert torch.equal(got.isfinite(), want.isfinite()), v
        for n in range(3):
            ok = want[n].isfinite()
            # 630 terms in fp32, in other orders
            assert float((got[n][ok] - want[n][ok]).norm() / want[n][ok].norm()) < 2e-6, (v, n)
    assert ran == 5                                  # one block; 2 and 4 rows alone or shared by two, 6 rows
