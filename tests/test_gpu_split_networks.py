"""The split kernel inside a handle: with a pool in its epilogue, and over whole networks against the fp32 instruction."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

pytestmark = pytest.mark.gpu


def _splits():
    return [v for v in range(B.cprune_num_tile_variants()) if "conv_split" in B.cprune_tile_variant_name(v, True, B.F32)]


@pytest.mark.parametrize("scale", [1.0, 1e-30])      # the second: every block is multiplied again on the fp32 instruction
@pytest.mark.parametrize("cfg", [(2, 20, 16, 14, 24), (5, 64, 8, 8, 90), (1, 33, 4, 6, 130), (3, 130, 28, 28, 48)])
def test_pool_in_the_epilogue(cfg, scale):
    """3x3 convolution + ReLU + 2x2 max-pool: every split variant that runs it is no less exact than the fp32-instruction
    variants are in the middle (those that cut the reduction into eight slices round less often)."""
    n, c_in, h, w, c_out = cfg
    gen = torch.Generator().manual_seed(c_in)
    net = synth.NetSpec("pooled", c_in, h, w)
    a = net.add(synth.Layer("conv", -1, c_in, c_out, k=3, stride=1, pad=1, act=synth.ACT_RELU, name="a"))
    p = net.add(synth.Layer("maxpool", a, c_out, c_out, k=2, stride=2, pad=0, name="p"))
    net.add(synth.Layer("conv", p, c_out, 8, k=1, stride=1, pad=0, act=synth.ACT_NONE, name="b"))
    wa, wb = torch.randn(c_out, c_in, 3, 3, generator=gen) / (4.5 * c_in) ** 0.5, torch.randn(8, c_out, 1, 1, generator=gen)
    ba, x = torch.randn(c_out, generator=gen) * 0.1 * scale, torch.randn(n, c_in, h, w, generator=gen) * scale
    layers = [{"w": wa.cuda(), "b": ba.cuda()}, {}, {"w": wb.cuda(), "b": torch.zeros(8, device="cuda")}]
    ref = torch.nn.functional.max_pool2d(torch.relu(torch.nn.functional.conv2d(x.double(), wa.double(), ba.double(), 1, 1)), 2)
    handle = pipeline.build_net(net, layers, n, B.F32, tune=False)
    errors, splits = {}, set(_splits())
    for v in range(B.cprune_num_tile_variants()):
        try:
            handle.set_layer_variant(0, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        handle.forward(x.cuda())
        y = handle.activation(1, n, ref.shape[1:]).double().cpu()
        errors[v] = float((y - ref).norm() / ref.norm())
    handle.close()
    fp32 = sorted(e for v, e in errors.items() if v not in splits)
    # (one chain of the fp32 instruction per sum, when multiplied again: as the least exact of those variants)
    base = fp32[len(fp32) // 2] if scale == 1.0 else 1.1 * fp32[-1]
    ran = [v for v in errors if v in splits]
    assert len(ran) >= 5, sorted(errors)
    for v in ran:
        assert errors[v] <= base, (v, errors[v], base)


def _logits64(net, layers, x):
    F, acts = torch.nn.functional, []
    for L, q in zip(net.layers, layers):
        src = x.double() if L.input < 0 else acts[L.input]
        if L.kind == "conv":
            y = F.conv2d(src, q["w"].double().cpu(), q["b"].double().cpu(), L.stride, L.pad)
            y = y if L.residual is None else y + acts[L.residual]
            y = y.clamp(min=0) if L.act else y
        elif L.kind == "maxpool":
            y = F.max_pool2d(src, L.k, L.stride, L.pad)
        elif L.kind == "gavgpool":
            y = src.mean((2, 3), keepdim=True)
        else:
            y = F.linear(src.flatten(1), q["w"].double().cpu().flatten(1), q["b"].double().cpu())
        acts.append(y)
    return acts[-1].flatten(1)


@pytest.mark.parametrize("name", ["vgg16", "resnet18"])
def test_logits_are_no_less_exact(name):
    """Logits against 64 bits, mean of four sets of weights and images: every layer that can on the split kernel, against
    the same layers on the first variant with the fp32 instruction."""
    net = synth.vgg16(10, 32) if name == "vgg16" else synth.resnet18(10, 32, cifar_stem=True)
    errors = {"split": [], "fp32": []}
    for seed in (81, 82, 83, 84):
        params = synth.layer_params(net, seed)
        layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), B.F32)
        x = torch.from_numpy(synth.net_input(net, seed, 8))
        ref = _logits64(net, layers, x)
        B.cprune_clear_tile_cache()
        handle = pipeline.build_net(net, layers, 8, B.F32, tune=False)
        took = []
        for i in range(handle.n_layers):
            for v in _splits():
                try:
                    handle.set_layer_variant(i, v)
                    took.append(i)
                    break
                except B.CPruneError:
                    continue
        assert len(took) >= 8, took
        for kind in ("split", "fp32"):
            for i in took if kind == "fp32" else ():
                assert any(_pins(handle, i, v) for v in range(B.cprune_num_tile_variants()) if v not in _splits())
            y = handle.forward(x.cuda()).double().cpu()
            errors[kind].append(float((y - ref).norm() / ref.norm()))
        handle.close()
    print(name, {k: ["%.2e" % e for e in v] for k, v in errors.items()}, flush=True)
    assert sum(errors["split"]) <= sum(errors["fp32"]), errors


def _pins(handle, layer, v):
    try:
        handle.set_layer_variant(layer, v)
        return True
    except B.CPruneError:
        return False
