"""Numbers that three bf16 parts do not hold (infinities, both ends of the range), in inputs and in weights: the split
kernel answers as the fp32 instruction does, in the boundary's layout and inside a handle."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu

SHAPES = [(1, 20, 12, 12, 24, 3, 1), (3, 33, 9, 7, 100, 3, 2), (2, 64, 8, 8, 17, 1, 1)]   # n, c_in, h, w, c_out, k, stride


def _data(cfg, x_scale=1.0, w_scale=1.0):
    n, c_in, h, w, c_out, k, _ = cfg
    gen = torch.Generator().manual_seed(c_in)
    x = (torch.randn(n, c_in, h, w, generator=gen, dtype=torch.float64) * x_scale).clamp(-3.4028e38, 3.4028e38).float()
    wt = (torch.randn(c_out, c_in, k, k, generator=gen, dtype=torch.float64) * (w_scale * (2.0 / (c_in * k * k)) ** 0.5)).float()
    return x, wt


def _outputs(cfg, x, wt, layout):
    """{variant: output}: every split variant that runs the layer, and one variant of the general kernel (key None)."""
    n, c_in, h, w, c_out, k, stride = cfg
    xd, wd, bd = x.cuda(), wt.cuda(), torch.zeros(c_out, device="cuda")
    d = B.conv_desc(x.shape, wt.shape, stride, k // 2, 1, B.F32, B.ACT_NONE, False)
    splits = [v for v in range(B.cprune_num_tile_variants())
              if "conv_split" in B.cprune_tile_variant_name(v, layout == "handle", B.F32)]
    out, handle = {}, None
    if layout == "handle":
        net = synth.NetSpec("one", c_in, h, w)
        net.add(synth.Layer("conv", -1, c_in, c_out, k=k, stride=stride, pad=k // 2, act=synth.ACT_NONE, name="c"))
        handle = pipeline.build_net(net, [{"w": wd, "b": bd}], n, B.F32, tune=False)
    for v in [0] + splits:
        try:
            if handle:
                handle.set_layer_variant(0, v)
                y = handle.forward(xd)
            else:
                y = B.cprune_conv2d_bn_relu(d, xd, wd, bd, None, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED and v
            continue
        torch.cuda.synchronize()
        out[v or None] = y.cpu().reshape(B.out_shape(d))
    if handle:
        handle.close()
    assert len(out) >= 5, sorted(out, key=str)
    return out


@pytest.mark.parametrize("layout", ["boundary", "handle"])
@pytest.mark.parametrize("cfg", SHAPES)
@pytest.mark.parametrize("what", ["inputs", "weights", "tiny weights", "nan weights"])
def test_infinities(cfg, what, layout):
    x, w = _data(cfg)
    inf = float("inf")
    w[3, 4] = 1.0
    if what == "inputs":
        x[0, 4, 5, 5], x[-1, 7, 2, 1] = inf, float("nan")
    elif what == "weights":
        w[2, 4, -1, 0], w[11, 9, 0, -1] = inf, -inf
        x[0, 4, :3], x[0, 9, 1:4] = 1.0, 0.5             # parts that are zero
        x[0, 4, 6] = 1.00390625                          # parts of different sign
    elif what == "tiny weights":
        w[5, 4], w[6, 4], w[7, 4] = 2.0 ** -105, -2.0 ** -125, 1e-40
        x[0, 4, 5, 5] = inf
    else:
        w[8, 3, 0, 0] = float("nan")
    ys = _outputs(cfg, x, w, layout)
    want = ys.pop(None)
    odd = ~torch.isfinite(want)
    assert odd.any() and not odd.all()
    for v, y in ys.items():
        assert torch.equal(torch.isnan(y), torch.isnan(want)), v
        assert torch.equal(torch.isinf(y), torch.isinf(want)) and torch.equal(y[torch.isinf(y)], want[torch.isinf(want)]), v
        assert float((y - want)[~odd].norm() / want[~odd].norm()) < 1e-6, v


@pytest.mark.parametrize("layout", ["boundary", "handle"])
@pytest.mark.parametrize("cfg", SHAPES)
@pytest.mark.parametrize("x_scale,w_scale", [(1e-25, 1.0), (1e-33, 1.0), (1e-36, 1.0), (1.0, 1e-34), (1e-18, 1e-18), (1e30, 1.0),
                                             (1.5e38, 1e-4), (1e-4, 1.5e38), (1e-36, 1e10), (1e10, 1e-36)])
def test_both_ends_of_the_range(cfg, x_scale, w_scale, layout):
    """2-norm error against 64 bits: no larger than 1.1 times the fp32 instruction's own (10 % for the spread between two
    orders of one sum), or half a unit in the last place, which short sums reach in either form.  A number that loses bits
    times one of 1e10 is inside the stated range (2^59 over the terms of a sum: 1e15 for these)."""
    x, w = _data(cfg, x_scale, w_scale)
    if x_scale == 1e-36:
        x[..., :4] = 0.0                                  # sums that are exactly zero beside the small ones
    ref = torch.nn.functional.conv2d(x.double(), w.double(), None, cfg[6], cfg[5] // 2)
    ys = _outputs(cfg, x, w, layout)
    base = float((ys.pop(None).double() - ref).norm() / ref.norm())
    for v, y in ys.items():
        e = float((y.double() - ref).norm() / ref.norm())
        assert e <= max(1.1 * base, 2.0 ** -24), (v, e, base)


@pytest.mark.parametrize("layout", ["boundary", "handle"])
def test_small_numbers_beside_ordinary_ones(layout):
    """A corner of the map 1e34 times smaller than the rest keeps its own relative accuracy."""
    cfg = (1, 40, 12, 12, 48, 3, 1)
    x, w = _data(cfg)
    x[..., :6, :6] *= 1e-34
    ref = torch.nn.functional.conv2d(x.double(), w.double(), None, 1, 1)[..., :5, :5]
    ys = _outputs(cfg, x, w, layout)
    base = float((ys.pop(None).double()[..., :5, :5] - ref).norm() / ref.norm())
    for v, y in ys.items():
        e = float((y.double()[..., :5, :5] - ref).norm() / ref.norm())
        assert e <= max(1.1 * base, 2.0 ** -24), (v, e, base)


@pytest.mark.parametrize("layout", ["boundary", "handle"])
def test_what_is_left_out_of_a_product(layout):
    """One term per sum: the rounding of the result (2.53e-8 in the 2-norm over random numbers) and the parts left out (5.7e-9
    with both operands cut by rounding, 1.8e-8 with one cut by truncation) make 2.6e-8, by truncation 3.1e-8."""
    cfg = (4, 32, 32, 32, 64, 1, 1)
    x, w = _data(cfg)
    x *= torch.nn.functional.one_hot(torch.arange(4 * 32 * 32) % 32, 32).reshape(4, 32, 32, 32).permute(0, 3, 1, 2)
    ref = torch.nn.functional.conv2d(x.double(), w.double())
    for v, y in _outputs(cfg, x, w, layout).items():
        assert float((y.double() - ref).norm() / ref.norm()) < 2.75e-8, v


@pytest.mark.parametrize("layout", ["boundary", "handle"])
@pytest.mark.parametrize("c_in,k", [(2, 3), (16, 1), (17, 1), (24, 1), (3, 3), (4, 3), (32, 1), (1, 5), (40, 1)])
def test_short_sums(c_in, k, layout):
    """Sums of 16 to 40 terms: no less exact than on the fp32 instruction."""
    if layout == "handle" and c_in <= 4:
        pytest.skip("a handle reads at most four input channels in the caller's layout")
    cfg = (4, c_in, 28, 28, 64, k, 1)
    x, w = _data(cfg)
    ref = torch.nn.functional.conv2d(x.double(), w.double(), None, 1, k // 2)
    ys = _outputs(cfg, x, w, layout)
    base = float((ys.pop(None).double() - ref).norm() / ref.norm())
    for v, y in ys.items():
        e = float((y.double() - ref).norm() / ref.norm())
        print(cfg, layout, v, f"{e:.3e} against {base:.3e}", flush=True)
        assert e <= base, (v, e, base)


@pytest.mark.parametrize("c_in,k", [(1, 1), (2, 1), (3, 1), (5, 1), (8, 1), (15, 1), (1, 3)])
def test_shorter_sums_stay_on_the_fp32_instruction(c_in, k):
    x, w = _data((1, c_in, 16, 16, 32, k, 1))
    d = B.conv_desc(x.shape, w.shape, 1, k // 2, 1, B.F32, B.ACT_NONE, False)
    for v in range(B.cprune_num_tile_variants()):
        if "conv_split" in B.cprune_tile_variant_name(v, False, B.F32):
            with pytest.raises(B.CPruneError) as e:
                B.cprune_conv2d_bn_relu(d, x.cuda(), w.cuda(), None, None, v)
            assert e.value.status == B.ERR_UNSUPPORTED
