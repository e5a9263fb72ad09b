"""The row-strip kernel at stride 2, every variant, alone and with the 1x1 / stride 2 layer beside it in the same launch: odd maps, one to
three strips across, two and four images side by side, part-filled chunks and filter blocks; numbers that three parts do not hold."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu
DT = {"f32": B.F32, "f16": B.F16, "bf16": B.BF16}
# 2-norm of the difference over that of the result: sums rounded once per 32 terms in fp32; 16-bit outputs are rounded to nearest, which
# moves an element by at most half a unit in the last place, 2^-11 (fp16: 11 significant bits) or 2^-8 (bf16: 8) of its size, and with
# it the 2-norm; the sums themselves, and activations under fp16's normal range, add less than 1e-5
REL = {"f32": 1e-6, "f16": 2.0 ** -11 + 1e-5, "bf16": 2.0 ** -8 + 1e-5}


def _name(v, dtype):
    return B.cprune_tile_variant_name(v, True, dtype)


def _variants(dtype):
    return [v for v in range(B.cprune_num_tile_variants()) if "conv_rows_s2" in _name(v, dtype)]


def _rel(y, ref):
    return float((y.double().cpu() - ref).norm() / ref.norm())


def _data(c, o, o1, h, w, batch, dtype, seed):
    gen = torch.Generator().manual_seed(seed)
    td = B.TORCH_DTYPE[dtype]
    x = torch.randn(batch, c, h, w, generator=gen).to(td)
    w3 = (torch.randn(o, c, 3, 3, generator=gen) * (2.0 / (9 * c)) ** 0.5).to(td)
    w1 = (torch.randn(o1, c, 1, 1, generator=gen) * (2.0 / c) ** 0.5).to(td)
    return x, w3, w1, torch.randn(o, generator=gen), torch.randn(o1, generator=gen)


def _net(c, o, o1, h, w):
    """identity 1x1 (the input, channels-last) -> 1x1 / stride 2 and 3x3 / stride 2 on it -> a last 1x1 on the latter"""
    net = synth.NetSpec("s2", c, h, w)
    a = net.add(synth.Layer("conv", -1, c, c, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="a"))
    if o1:
        net.add(synth.Layer("conv", a, c, o1, k=1, stride=2, pad=0, act=synth.ACT_RELU6, name="p"))
    q = net.add(synth.Layer("conv", a, c, o, k=3, stride=2, pad=1, act=synth.ACT_RELU, name="q"))
    net.add(synth.Layer("conv", q, o, 8, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="z"))
    return net, q


def _build(net, c, o, w3, w1, b3, b1, batch, dtype, o1):
    td = B.TORCH_DTYPE[dtype]
    layers = [{"w": torch.eye(c, device="cuda").view(c, c, 1, 1).to(td), "b": torch.zeros(c, device="cuda")}]
    if o1:
        layers.append({"w": w1.cuda(), "b": b1.cuda()})
    layers += [{"w": w3.cuda(), "b": b3.cuda()}, {"w": torch.ones(8, o, 1, 1, device="cuda").to(td), "b": torch.zeros(8, device="cuda")}]
    B.cprune_clear_tile_cache()
    return pipeline.build_net(net, layers, batch, dtype, tune=False)


CASES = [
    # c_in, filters, filters of the 1x1 layer (0: none), height, width, batch
    (16, 16, 0, 2, 2, 1), (40, 33, 20, 7, 7, 5), (64, 67, 128, 13, 15, 3), (33, 90, 17, 28, 31, 2), (130, 20, 70, 34, 62, 1),
    (96, 48, 0, 9, 97, 2), (260, 40, 64, 5, 8, 9), (130, 158, 300, 14, 14, 2),
]


@pytest.mark.parametrize("dtype", sorted(DT))
@pytest.mark.parametrize("cfg", CASES)
def test_every_variant(cfg, dtype):
    c, o, o1, h, w, batch = cfg
    dt = DT[dtype]
    x, w3, w1, b3, b1 = _data(c, o, o1 or 1, h, w, batch, dt, c + o)
    conv = torch.nn.functional.conv2d
    ref3 = conv(x.double(), w3.double(), b3.double(), 2, 1).clamp(min=0)
    ref1 = conv(x.double(), w1.double(), b1.double(), 2, 0).clamp(0, 6)
    net, q = _net(c, o, o1, h, w)
    handle = _build(net, c, o, w3, w1, b3, b1, batch, dt, o1)
    if o1 and dt != B.F32:
        assert handle.layer_fused(q - 1) and handle.layer_variant(q - 1) == -1 and handle.layer_variant(q) in _variants(dt)
    ran = 0
    for v in _variants(dt):
        try:
            handle.set_layer_variant(q, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        ran += 1
        for n in {batch, (batch + 1) // 2}:
            handle.forward(x[:n].cuda(), use_graph=n == batch)
            y3 = handle.activation(q, n, ref3.shape[1:])
            assert _rel(y3, ref3[:n]) < REL[dtype], (_name(v, dt), n)
            if o1:
                assert _rel(handle.activation(q - 1, n, ref1.shape[1:]), ref1[:n]) < REL[dtype], (_name(v, dt), n)
    assert ran >= 1                                  # (one chunk of channels: only variants of one wavefront per strip)
    if o1 and dt != B.F32:
        assert handle.layer_fused(q - 1)             # still one launch
        both = handle.activation(q, batch, ref3.shape[1:]).clone() if batch == 1 else None
        handle.set_layer_variant(q - 1, 0)
        assert not handle.layer_fused(q - 1) and handle.layer_variant(q - 1) == 0
        handle.forward(x.cuda())
        assert _rel(handle.activation(q, batch, ref3.shape[1:]), ref3) < REL[dtype]
        assert _rel(handle.activation(q - 1, batch, ref1.shape[1:]), ref1) < REL[dtype]
        assert both is None or torch.equal(both, handle.activation(q, 1, ref3.shape[1:]))
    handle.close()


@pytest.mark.parametrize("dtype", sorted(DT))
def test_untimed_pairs_are_small_layers(dtype):
    """One launch up to 0.3 GFLOP in fp32 and 0.6 in 16-bit data, two above: the same activations."""
    c, o, o1, h = 160, 40, 64, 28                     # 26.6 MFLOP an image
    dt = DT[dtype]
    conv = torch.nn.functional.conv2d
    for batch, small in ((4, True), (11 if dtype == "f32" else 22, True), (12 if dtype == "f32" else 23, False), (32, False)):
        x, w3, w1, b3, b1 = _data(c, o, o1, h, h, batch, dt, 5)
        net, q = _net(c, o, o1, h, h)
        handle = _build(net, c, o, w3, w1, b3, b1, batch, dt, o1)
        assert bool(handle.layer_fused(q - 1)) == small and (handle.layer_variant(q - 1) == -1) == small, batch
        handle.forward(x.cuda())
        ref3 = conv(x.double(), w3.double(), b3.double(), 2, 1).clamp(min=0)
        ref1 = conv(x.double(), w1.double(), b1.double(), 2, 0).clamp(0, 6)
        assert _rel(handle.activation(q, batch, ref3.shape[1:]), ref3) < REL[dtype]
        assert _rel(handle.activation(q - 1, batch, ref1.shape[1:]), ref1) < REL[dtype]
        handle.close()


@pytest.mark.parametrize("dtype", sorted(DT))
def test_a_timed_handle(dtype):
    """Layers apart or in one launch, whichever was the faster, and a smaller batch: the same activations."""
    c, o, o1, h, w, batch = 64, 70, 128, 28, 28, 16
    dt = DT[dtype]
    x, w3, w1, b3, b1 = _data(c, o, o1, h, w, batch, dt, 3)
    conv = torch.nn.functional.conv2d
    ref3 = conv(x.double(), w3.double(), b3.double(), 2, 1).clamp(min=0)
    ref1 = conv(x.double(), w1.double(), b1.double(), 2, 0).clamp(0, 6)
    net, q = _net(c, o, o1, h, w)
    _build(net, c, o, w3, w1, b3, b1, batch, dt, o1).close()
    td = B.TORCH_DTYPE[dt]
    layers = [{"w": torch.eye(c, device="cuda").view(c, c, 1, 1).to(td), "b": torch.zeros(c, device="cuda")},
              {"w": w1.cuda(), "b": b1.cuda()}, {"w": w3.cuda(), "b": b3.cuda()},
              {"w": torch.ones(8, o, 1, 1, device="cuda").to(td), "b": torch.zeros(8, device="cuda")}]
    form = None
    for _ in range(2):                                # timed, then from what was remembered
        handle = pipeline.build_net(net, layers, batch, dt, tune=True)
        assert form is None or form == (handle.layer_fused(q - 1), handle.layer_variant(q))
        form = (handle.layer_fused(q - 1), handle.layer_variant(q))
        for n in (batch, 3, 1, batch):
            handle.forward(x[:n].cuda())
            assert _rel(handle.activation(q, n, ref3.shape[1:]), ref3[:n]) < REL[dtype]
            assert _rel(handle.activation(q - 1, n, ref1.shape[1:]), ref1[:n]) < REL[dtype]
        times = handle.layer_times(x.cuda())
        assert (times[q - 1] == 0) == bool(form[0]) and times[q] > 0
        handle.close()
    B.cprune_clear_tile_cache()


def test_numbers_three_parts_do_not_hold():
    gen = torch.Generator().manual_seed(8)
    c, o, h = 70, 40, 11
    x = torch.randn(3, c, h, h, generator=gen)
    x[0, 3, 4, 4], x[0, 60, 9, 2] = float("inf"), 3.39e38
    x[1] *= 2.0 ** -118
    w3 = torch.randn(o, c, 3, 3, generator=gen)
    net = synth.NetSpec("s2r", c, h, h)
    net.add(synth.Layer("conv", -1, c, o, k=3, stride=2, pad=1, act=synth.ACT_NONE, name="a"))
    handle = pipeline.build_net(net, [{"w": w3.cuda(), "b": torch.zeros(o, device="cuda")}], 3, B.F32, tune=False)
    handle.set_layer_variant(0, 0)                   # the fp32 instruction
    want = handle.forward(x.cuda()).double().cpu()
    assert not want[0].isfinite().all() and want[1:].isfinite().all()
    ran = 0
    for v in _variants(B.F32):
        try:
            handle.set_layer_variant(0, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        ran += 1
        got = handle.forward(x.cuda()).double().cpu()
        assert torch.equal(got.isfinite(), want.isfinite()), v
        for n in range(3):
            ok = want[n].isfinite()
            # 630 terms in fp32, in other orders
            assert float((got[n][ok] - want[n][ok]).norm() / want[n][ok].norm()) < 2e-6, (v, n)
    assert ran == 3                                  # one block, three chunks: 4 rows alone or shared by two, 2 shared by two
    handle.close()


def _in_use():
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def test_copies_of_a_pair_that_loses_are_given_back():
    """fp32, 32 images, layers that run faster apart: a handle that found so by timing holds no more than one that remembers it (packed
    for the pair the two layers' weights are 15.7 MB)."""
    c, o, o1, h, batch = 512, 512, 512, 28, 32
    gen = torch.Generator().manual_seed(4)
    layers = [{"w": torch.eye(c).view(c, c, 1, 1).cuda(), "b": torch.zeros(c, device="cuda")},
              {"w": torch.randn(o1, c, 1, 1, generator=gen).cuda(), "b": torch.zeros(o1, device="cuda")},
              {"w": torch.randn(o, c, 3, 3, generator=gen).cuda(), "b": torch.zeros(o, device="cuda")},
              {"w": torch.randn(8, o, 1, 1, generator=gen).cuda(), "b": torch.zeros(8, device="cuda")}]
    net, _ = _net(c, o, o1, h, h)
    pipeline.build_net(net, layers, batch, B.F32, tune=True).close()      # (what the first handle of a process leaves behind)
    used = []
    for remembered in (False, True):
        if not remembered:
            B.cprune_clear_tile_cache()
        before = _in_use()
        handle = pipeline.build_net(net, layers, batch, B.F32, tune=True)
        used.append(_in_use() - before)
        handle.close()
    B.cprune_clear_tile_cache()
    assert used[0] - used[1] < 8 << 20, used


@pytest.mark.parametrize("dtype", sorted(DT))
@pytest.mark.parametrize("tune", [False, True])
def test_layers_of_a_pair_that_ends(dtype, tune):
    """Either layer pinned to a kernel of its own: the other runs the variant it has, from its own copy of the weights."""
    c, o, o1, h, batch = 130, 20, 70, 16, 2
    dt = DT[dtype]
    x, w3, w1, b3, b1 = _data(c, o, o1, h, h, batch, dt, 6)
    conv = torch.nn.functional.conv2d
    ref3 = conv(x.double(), w3.double(), b3.double(), 2, 1).clamp(min=0)
    ref1 = conv(x.double(), w1.double(), b1.double(), 2, 0).clamp(0, 6)
    net, q = _net(c, o, o1, h, h)
    td = B.TORCH_DTYPE[dt]
    layers = [{"w": torch.eye(c, device="cuda").view(c, c, 1, 1).to(td), "b": torch.zeros(c, device="cuda")},
              {"w": w1.cuda(), "b": b1.cuda()}, {"w": w3.cuda(), "b": b3.cuda()},
              {"w": torch.ones(8, o, 1, 1, device="cuda").to(td), "b": torch.zeros(8, device="cuda")}]
    for pinned in (q, q - 1):
        B.cprune_clear_tile_cache()
        handle = pipeline.build_net(net, layers, batch, dt, tune=tune)
        assert tune or handle.layer_fused(q - 1)
        for graph in (False, True):
            handle.forward(x.cuda(), use_graph=graph)
            if not graph:
                handle.set_layer_variant(pinned, 0)
                assert not handle.layer_fused(q - 1) and handle.layer_variant(pinned) == 0
                assert handle.layer_variant(2 * q - 1 - pinned) >= 0
        for n in (batch, 1):
            handle.forward(x[:n].cuda())
            assert _rel(handle.activation(q, n, ref3.shape[1:]), ref3[:n]) < REL[dtype]
            assert _rel(handle.activation(q - 1, n, ref1.shape[1:]), ref1[:n]) < REL[dtype]
        handle.close()
    B.cprune_clear_tile_cache()


@pytest.mark.parametrize("dtype", sorted(DT))
def test_a_pinned_variant_outlives_the_pair(dtype):
    c, o, o1, h, batch = 130, 20, 70, 16, 2
    dt = DT[dtype]
    x, w3, w1, b3, b1 = _data(c, o, o1, h, h, batch, dt, 7)
    ref3 = torch.nn.functional.conv2d(x.double(), w3.double(), b3.double(), 2, 1).clamp(min=0)
    net, q = _net(c, o, o1, h, h)
    pinned = 0
    for v in _variants(dt):
        handle = _build(net, c, o, w3, w1, b3, b1, batch, dt, o1)
        assert handle.layer_fused(q - 1)
        try:
            handle.set_layer_variant(q, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
        else:
            pinned += 1
            handle.set_layer_variant(q - 1, 0)
            assert handle.layer_variant(q) == v and handle.layer_variant(q - 1) == 0
            handle.forward(x.cuda())
            assert _rel(handle.activation(q, batch, ref3.shape[1:]), ref3) < REL[dtype]
        handle.close()
    assert pinned >= 2


@pytest.mark.parametrize("dtype", sorted(DT))
@pytest.mark.parametrize("batch", [2, 32])
def test_choices_of_a_timed_handle_applied_to_another(dtype, batch):
    """Both forms of a layer pair too large to be paired untimed, and of a small one: the variants a handle reports, set on an untimed one."""
    c, o, o1, h = 160, 72, 64, 28
    dt = DT[dtype]
    x, w3, w1, b3, b1 = _data(c, o, o1, h, h, batch, dt, 8)
    conv = torch.nn.functional.conv2d
    ref3 = conv(x.double(), w3.double(), b3.double(), 2, 1).clamp(min=0)
    ref1 = conv(x.double(), w1.double(), b1.double(), 2, 0).clamp(0, 6)
    net, q = _net(c, o, o1, h, h)
    strips = next(v for v in _variants(dt) if _name(v, dt).endswith(" 1, 4, 1>"))
    pw = next(v for v in range(B.cprune_num_tile_variants()) if "conv_pw3" in _name(v, dt) and _name(v, dt).endswith("1, 2, true>"))
    for choices, fused in (([-1, strips], True), ([pw, strips], False), ([pw, 0], False)):
        handle = _build(net, c, o, w3, w1, b3, b1, batch, dt, o1)
        for layer, v in zip((q - 1, q), choices):
            if v >= 0:
                handle.set_layer_variant(layer, v)
        assert handle.layer_fused(q - 1) == fused
        assert [handle.layer_variant(q - 1), handle.layer_variant(q)] == choices
        for graph in (False, True):
            handle.forward(x.cuda(), use_graph=graph)
            assert _rel(handle.activation(q, batch, ref3.shape[1:]), ref3) < REL[dtype]
            assert _rel(handle.activation(q - 1, batch, ref1.shape[1:]), ref1) < REL[dtype]
        handle.close()
    # a timed handle's own, whatever they are
    td = B.TORCH_DTYPE[dt]
    layers = [{"w": torch.eye(c, device="cuda").view(c, c, 1, 1).to(td), "b": torch.zeros(c, device="cuda")},
              {"w": w1.cuda(), "b": b1.cuda()}, {"w": w3.cuda(), "b": b3.cuda()},
              {"w": torch.ones(8, o, 1, 1, device="cuda").to(td), "b": torch.zeros(8, device="cuda")}]
    B.cprune_clear_tile_cache()
    timed = pipeline.build_net(net, layers, batch, dt, tune=True)
    want = [(timed.layer_variant(i), timed.layer_fused(i)) for i in range(4)]
    outputs = []
    for handle in (timed, _build(net, c, o, w3, w1, b3, b1, batch, dt, o1)):
        for i, (v, _) in enumerate(want):
            if v >= 0 and handle is not timed:
                handle.set_layer_variant(i, v)
        assert [(handle.layer_variant(i), handle.layer_fused(i)) for i in range(4)] == want
        handle.forward(x.cuda())
        outputs.append([handle.activation(i, batch, ref.shape[1:]).clone() for i, ref in ((q, ref3), (q - 1, ref1))])
        handle.close()
    assert all(torch.equal(a, b) for a, b in zip(*outputs))


@pytest.mark.parametrize("dtype", sorted(DT))
def test_one_1x1_layer_between_two(dtype):
    """Two 3x3 layers on the input of one 1x1 layer: it runs in one launch at most, whichever 3x3 layer is given a variant of that kernel."""
    c, o, o1, h, batch = 130, 20, 70, 16, 2
    dt = DT[dtype]
    x, w3, w1, b3, b1 = _data(c, o, o1, h, h, batch, dt, 9)
    conv = torch.nn.functional.conv2d
    ref3 = conv(x.double(), w3.double(), b3.double(), 2, 1).clamp(min=0)
    ref1 = conv(x.double(), w1.double(), b1.double(), 2, 0).clamp(0, 6)
    net = synth.NetSpec("s2two", c, h, h)
    a = net.add(synth.Layer("conv", -1, c, c, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="a"))
    p = net.add(synth.Layer("conv", a, c, o1, k=1, stride=2, pad=0, act=synth.ACT_RELU6, name="p"))
    qs = [net.add(synth.Layer("conv", a, c, o, k=3, stride=2, pad=1, act=synth.ACT_RELU, name=f"q{i}")) for i in range(2)]
    net.add(synth.Layer("conv", qs[1], o, 8, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="z"))
    td = B.TORCH_DTYPE[dt]
    three = {"w": w3.cuda(), "b": b3.cuda()}
    layers = [{"w": torch.eye(c, device="cuda").view(c, c, 1, 1).to(td), "b": torch.zeros(c, device="cuda")}, {"w": w1.cuda(), "b": b1.cuda()},
              three, three, {"w": torch.ones(8, o, 1, 1, device="cuda").to(td), "b": torch.zeros(8, device="cuda")}]
    B.cprune_clear_tile_cache()
    handle = pipeline.build_net(net, layers, batch, dt, tune=False)
    strips = next(v for v in _variants(dt) if _name(v, dt).endswith(" 1, 4, 1>"))
    for order in (qs, qs[::-1], [p]):
        for layer in order:
            handle.set_layer_variant(layer, strips if layer != p else 0)
        handle.forward(x.cuda())
        assert _rel(handle.activation(p, batch, ref1.shape[1:]), ref1) < REL[dtype]
        for q in qs:
            assert handle.layer_variant(q) == strips
            assert _rel(handle.activation(q, batch, ref3.shape[1:]), ref3) < REL[dtype]
        times = handle.layer_times(x.cuda())
        assert all(times[q] > 0 for q in qs) and bool(handle.layer_fused(p)) == (order != [p]) == (times[p] == 0)
    handle.close()


@pytest.mark.parametrize("dtype,c,o,h,batch,strips", [
    # fp32: over 1 GFLOP 16.8 us on the kernel before, 24.1 on strips; a chain of 22 chunks under 0.2 GFLOP 14.1 and 17.2
    ("f32", 181, 265, 20, 14, False), ("f32", 683, 94, 14, 1, False), ("f32", 223, 127, 28, 4, True), ("f32", 446, 363, 7, 9, True),
    ("bf16", 181, 265, 20, 14, True), ("bf16", 683, 94, 14, 1, True),
])
def test_untimed_layers_on_strips(dtype, c, o, h, batch, strips):
    dt = DT[dtype]
    _, w3, w1, b3, b1 = _data(c, o, 1, h, h, batch, dt, 10)
    net, q = _net(c, o, 0, h, h)
    handle = _build(net, c, o, w3, w1, b3, b1, batch, dt, 0)
    assert (handle.layer_variant(q) in _variants(dt)) == strips
    handle.close()
