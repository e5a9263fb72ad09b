"""The 1x1 kernel on the 16-bit matrix cores (layers of a handle; fp32 on three parts), every variant: one to many rounds and chunks of the reduction, a part-filled
last round, pixels and filters past the last tile, stride 2, shortcuts; numbers that three parts do not hold."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu


DT = {"f32": B.F32, "f16": B.F16, "bf16": B.BF16}
# 2-norm of the difference over that of the result.  fp32: sums of c terms, rounded once per 32, of three parts: under 1e-6 up to 1000 terms.
# 16-bit outputs are rounded to nearest: at most half a unit in the last place, 2^-11 (fp16: 11 significant bits) or 2^-8 (bf16: 8) of an
# element, and the shortcut, itself such an output, adds as much
REL = {"f32": 1e-6, "f16": 2.0 ** -11 + 1e-5, "bf16": 2.0 ** -8 + 1e-5}


def _variants():
    return [v for v in range(B.cprune_num_tile_variants()) if "conv_pw3" in B.cprune_tile_variant_name(v, True, B.F32)]


def _handle(c, o, h, w, stride, residual, act, batch, wts, bias, dtype=B.F32):
    """identity 1x1 layer (the input, channels-last; a second one for the shortcut) -> the layer under test"""
    net = synth.NetSpec("pw3", c, h, w)
    a = net.add(synth.Layer("conv", -1, c, c, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="a"))
    layers = [{"w": torch.eye(c, device="cuda").view(c, c, 1, 1).to(B.TORCH_DTYPE[dtype]), "b": torch.zeros(c, device="cuda")}]
    res = None
    if residual:
        res = net.add(synth.Layer("conv", a, c, o, k=1, stride=stride, pad=0, act=synth.ACT_NONE, name="r"))
        layers.append({"w": wts[1], "b": torch.zeros(o, device="cuda")})
    net.add(synth.Layer("conv", a, c, o, k=1, stride=stride, pad=0, act=act, residual=res, name="b"))
    layers.append({"w": wts[0], "b": bias})
    return pipeline.build_net(net, layers, batch, dtype, tune=False)


@pytest.mark.parametrize("dtype", sorted(DT))
@pytest.mark.parametrize("cfg", [
    # c_in, filters, height, width, stride, batch, shortcut, activation
    (16, 1, 1, 1, 1, 1, False, synth.ACT_NONE), (18, 48, 4, 3, 1, 2, False, synth.ACT_NONE), (17, 33, 5, 7, 1, 3, False, synth.ACT_RELU),
    (32, 64, 8, 4, 1, 1, True, synth.ACT_NONE), (33, 65, 13, 13, 2, 2, False, synth.ACT_RELU6),
    (64, 130, 7, 7, 1, 3, True, synth.ACT_RELU), (68, 16, 9, 11, 2, 4, True, synth.ACT_NONE),
    (97, 385, 14, 14, 1, 2, False, synth.ACT_RELU), (160, 129, 3, 5, 1, 1, False, synth.ACT_NONE),
    (829, 40, 7, 7, 1, 2, True, synth.ACT_RELU), (200, 257, 16, 16, 2, 5, False, synth.ACT_RELU),
])
def test_every_variant(cfg, dtype):
    c, o, h, w, stride, batch, residual, act = cfg
    dt, td = DT[dtype], B.TORCH_DTYPE[DT[dtype]]
    gen = torch.Generator().manual_seed(c * o)
    x = torch.randn(batch, c, h, w, generator=gen).to(td)
    wts = [(torch.randn(o, c, 1, 1, generator=gen) * (2.0 / c) ** 0.5).to(td) for _ in range(2)]
    bias = torch.randn(o, generator=gen)
    conv = lambda q: torch.nn.functional.conv2d(x.double(), q.double(), None, stride)
    ref = conv(wts[0]) + bias.double().view(1, -1, 1, 1)
    if residual:
        ref += conv(wts[1])
    ref = ref if act == synth.ACT_NONE else ref.clamp(0, 6) if act == synth.ACT_RELU6 else ref.clamp(min=0)
    handle = _handle(c, o, h, w, stride, residual, act, batch, [q.cuda() for q in wts], bias.cuda(), dt)
    last = 2 if residual else 1
    runnable = 0
    for v in _variants():
        try:
            handle.set_layer_variant(last, v)
        except B.CPruneError as e:              # a variant of the other types, or a dense 1x1 output whose filters are no multiple of four
            assert e.status == B.ERR_UNSUPPORTED
            continue
        runnable += 1
        for n in {batch, (batch + 1) // 2}:
            y = handle.forward(x[:n].cuda()).double().cpu()
            bound = REL[dtype] * (2 if residual else 1)
            assert float((y - ref[:n]).norm() / ref[:n].norm()) < bound, (v, n)
            assert float((y - ref[:n]).abs().max()) < 10 * bound * float(ref.abs().max()), (v, n)
    assert runnable >= 4 or (h * w == 1 and o % 4)
    handle.close()


def test_numbers_three_parts_do_not_hold():
    gen = torch.Generator().manual_seed(5)
    c, o, hw = 80, 72, 6
    x = torch.randn(3, c, hw, hw, generator=gen)
    x[0, 3, 2, 2], x[0, 70, 5, 5] = float("inf"), 3.39e38
    x[1] *= 2.0 ** -118
    wts = torch.randn(o, c, 1, 1, generator=gen)
    wts[7] *= 2.0 ** -60
    # the identity in front of the layer multiplies infinities by zero: the shortcut-free layer on the input itself
    net = synth.NetSpec("pw3r", c, hw, hw)
    net.add(synth.Layer("conv", -1, c, o, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="a"))
    handle = pipeline.build_net(net, [{"w": wts.cuda(), "b": torch.zeros(o, device="cuda")}], 3, B.F32, tune=False)
    handle.set_layer_variant(0, 0)               # the fp32 instruction
    want = handle.forward(x.cuda()).double().cpu()
    assert not want[0].isfinite().all() and want[1:].isfinite().all()
    ran = 0
    for v in _variants():
        try:
            handle.set_layer_variant(0, v)
        except B.CPruneError as e:               # built for 16-bit data only
            assert e.status == B.ERR_UNSUPPORTED
            continue
        ran += 1
        got = handle.forward(x.cuda()).double().cpu()
        assert torch.equal(got.isfinite(), want.isfinite()), v
        for n in range(3):
            ok = want[n].isfinite()
            assert float((got[n][ok] - want[n][ok]).norm() / want[n][ok].norm()) < 2e-6, (v, n)
            tiny = want[n, 7][ok[7]]
            if n == 1:                           # 2^-178: zero on either
                assert not got[n, 7].any() and not tiny.any()
                continue
            assert float((got[n, 7][ok[7]] - tiny).norm() / tiny.norm()) < 2e-6, (v, n)
    assert ran == 6
    handle.close()
