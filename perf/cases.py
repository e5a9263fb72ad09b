"""The work a user of this framework has it do, as a list of cases that can be timed.

Three kinds, all through the public entry points:

* ``net``    one forward pass of a channel-pruned network through an inference handle
             (``pipeline.build_net`` once, ``Net.forward`` per batch): what the method runs and times
             for every candidate model, and what serves the model afterwards;
* ``conv``   one pruned conv + folded batch-norm + activation through the single-layer entry point
             (``cprune_conv2d_bn_relu``): the layer-level call of the C ABI;
* ``prune``  the pruning stage of a whole network (``PrunePlan.run``: L1 scores, kept lists, gathered
             and folded weights): what every iteration of the search does before it builds a handle.

``listed()`` gives fixed cases, ``draw(rng)`` more of the same ranges, ``prepare(case, seed)`` what a
program has in hand before the call, ``run(state)`` one pass, ``work(case)`` the bytes and operations the
pass cannot do without, ``tolerance(case)`` how far another correct implementation may be off and
``exact(case, seed)`` the result in 64 bits.

Channel counts after pruning belong to the case (``keep_seed``); the values of weights, batch-norm
vectors and inputs, and with them which filters survive, come from the seed.
"""
import math
import random

import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth

DTYPES = {"f32": B.F32, "f16": B.F16, "bf16": B.BF16}

# the evaluated networks: builder, and the largest batch a drawn case takes (so that none costs more than
# the largest listed one)
NETS = {
    "vgg16": (lambda: synth.vgg16(10, 32), 64),
    "resnet18_cifar": (lambda: synth.resnet18(10, 32, cifar_stem=True), 64),
    "resnet18": (lambda: synth.resnet18(1000, 224), 32),
    "mobilenetv2": (lambda: synth.mobilenetv2(1000, 224), 64),
    "mnasnet": (lambda: synth.mnasnet(1000, 224), 48),
}


def _net_case(name, net, batch, dtype, keep_seed, max_batch=None, tune=True, graph=False):
    return {"name": name, "kind": "net", "net": net, "batch": batch, "max_batch": max_batch or batch, "dtype": dtype,
            "tune": tune, "graph": graph, "keep_seed": keep_seed}


def _conv_case(name, n, c_in, c_out, hw, dtype, k=3, stride=1, act=1, residual=False, tuned=True):
    return {"name": name, "kind": "conv", "n": n, "c_in": c_in, "c_out": c_out, "hw": hw, "k": k, "stride": stride,
            "dtype": dtype, "act": act, "residual": residual, "tuned": tuned}


def listed():
    return [
        # one pruned layer of a network on a 32x32 map, one image: the shortest call (launches and host work)
        _conv_case("conv_64to45_32_b1_f32", 1, 64, 45, 32, "f32", tuned=False),
        # a point of the channel-count sweep: odd filter count, a shape timed beforehand
        _conv_case("conv_128to83_56_b8_f32", 8, 128, 83, 56, "f32"),
        # the pruning stage between two candidates of a search
        {"name": "prune_vgg16_f32", "kind": "prune", "net": "vgg16", "dtype": "f32", "shortcuts": False, "keep_seed": 2},
        # latency of a single image, replayed as a graph
        _net_case("vgg16_b1_f32_graph", "vgg16", 1, "f32", 2, graph=True),
        # the headline workload: a batch of 64
        _net_case("vgg16_b64_f32", "vgg16", 64, "f32", 2),
        _net_case("vgg16_b64_f16", "vgg16", 64, "f16", 2),
        # the last, smaller batch of a data set through the handle built for full batches
        _net_case("vgg16_37of64_f16", "vgg16", 37, "f16", 5, max_batch=64),
        # a single 224x224 image, eager launches
        _net_case("resnet18_b1_bf16", "resnet18", 1, "bf16", 3),
        # 224x224 images, batch 32, both precisions (the largest case)
        _net_case("resnet18_b32_f32", "resnet18", 32, "f32", 3),
        _net_case("resnet18_b32_bf16", "resnet18", 32, "bf16", 3),
        # inverted residuals: pruned 1x1 layers and 3x3 depthwise layers at batch 64
        _net_case("mobilenetv2_b64_f32", "mobilenetv2", 64, "f32", 4),
        # 5x5 depthwise layers, a middle-sized batch in 16-bit data
        _net_case("mnasnet_b16_bf16", "mnasnet", 16, "bf16", 6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["net"] * 6 + ["conv"] * 3 + ["prune"])
    if kind == "net":
        net = rng.choice(sorted(NETS))
        tune = rng.random() < 0.85
        cap = NETS[net][1] if tune else NETS[net][1] // 4   # an untimed choice of programs may be slower
        batch = _log_int(rng, 1, cap)
        max_batch = batch if rng.random() < 0.7 else rng.randint(batch, cap)
        dtype = rng.choice(sorted(DTYPES))
        if net == "mnasnet" and dtype == "f16":
            dtype = "bf16"      # plain ReLU and no trained scales: its activations leave the range of fp16
        case = _net_case("", net, batch, dtype, rng.randrange(1 << 30), max_batch, tune,
                         graph=batch <= 4 and rng.random() < 0.5)
    elif kind == "conv":
        k, stride = rng.choice([(3, 1), (3, 1), (3, 1), (3, 2), (1, 1), (1, 2), (5, 1), (7, 2)])
        while True:
            n, hw = _log_int(rng, 1, 32), _log_int(rng, 7, 112)
            c_in, c_out = _log_int(rng, 3, 512), _log_int(rng, 3, 512)
            flops = 2.0 * n * c_out * c_in * k * k * (hw / stride) ** 2
            if 1e6 <= flops <= 2e10 and n * hw * hw * max(c_in, c_out) <= 1 << 27:
                break
        case = _conv_case("", n, c_in, c_out, hw, rng.choice(sorted(DTYPES)), k, stride, act=rng.choice([0, 1, 1, 2]),
                          residual=rng.random() < 0.25, tuned=rng.random() < 0.7)
    else:
        net = rng.choice(["vgg16", "resnet18", "resnet18_cifar"])
        case = {"name": "", "kind": "prune", "net": net, "dtype": rng.choice(sorted(DTYPES)),
                "shortcuts": net != "vgg16" and rng.random() < 0.5, "keep_seed": rng.randrange(1 << 30)}
    del case["name"]
    return case


# ---- networks and their parameters --------------------------------------------------------------

def _spec(case):
    if case["kind"] == "prune" and case["shortcuts"]:
        if case["net"] == "resnet18":
            return synth.resnet18(1000, 224, prune_shortcuts=True)
        return synth.resnet18(10, 32, cifar_stem=True, prune_shortcuts=True)
    return NETS[case["net"]][0]()


def _kept_counts(net, keep_seed):
    """Filters every pruned layer keeps: a ratio drawn from the network's own range."""
    rng = random.Random(keep_seed)
    return {i: synth.keep_count(rng.uniform(net.keep_lo, net.keep_hi), L.c_out)
            for i, L in enumerate(net.layers) if L.prune_out == "own"}


def _device_params(net, keep, gen):
    """Raw weights and batch-norm vectors with the distributions of synth.layer_params, made on the device."""
    def normal(n, std):
        return torch.randn(n, device="cuda", generator=gen) * std

    def uniform(n, lo, hi):
        return lo + (hi - lo) * torch.rand(n, device="cuda", generator=gen)

    out = []
    for i, L in enumerate(net.layers):
        p = {}
        if L.kind == "conv":
            cpg = L.c_in // L.groups
            p["w"] = normal((L.c_out, cpg, L.k, L.k), math.sqrt(2.0 / (cpg * L.k * L.k)))
            if L.bn:
                p.update(gamma=uniform(L.c_out, 0.5, 1.5), beta=normal(L.c_out, 0.1), mean=normal(L.c_out, 0.1),
                         var=uniform(L.c_out, 0.5, 1.5))
        elif L.kind == "fc":
            p["w"], p["b"] = normal((L.c_out, L.c_in), math.sqrt(2.0 / L.c_in)), normal(L.c_out, 0.1)
        if i in keep:
            p["keep"] = keep[i]
        out.append(p)
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = DTYPES[case["dtype"]]
    tdt = B.TORCH_DTYPE[dtype]
    if case["kind"] == "conv":
        k, hw = case["k"], case["hw"]
        x = torch.randn((case["n"], case["c_in"], hw, hw), device="cuda", generator=gen).to(tdt)
        w = (torch.randn((case["c_out"], case["c_in"], k, k), device="cuda", generator=gen)
             * math.sqrt(2.0 / (case["c_in"] * k * k))).to(tdt)
        bias = torch.randn(case["c_out"], device="cuda", generator=gen) * 0.1
        d = B.conv_desc(x.shape, w.shape, case["stride"], k // 2, 1, dtype, case["act"], case["residual"])
        res = torch.randn(B.out_shape(d), device="cuda", generator=gen).to(tdt) if case["residual"] else None
        if case["tuned"] and not B.cprune_cached_tile(d)[1]:
            B.cprune_select_tile(d, x, w, bias, res)
        return {"kind": "conv", "d": d, "x": x, "w": w, "bias": bias, "res": res}
    net = _spec(case)
    keep = _kept_counts(net, case["keep_seed"])
    params = _device_params(net, keep, gen)
    if case["kind"] == "prune":
        return {"kind": "prune", "plan": pipeline.prune_plan(net, params, dtype)}
    layers, _ = pipeline.prune_net(net, params, dtype)
    handle = pipeline.build_net(net, layers, case["max_batch"], dtype, tune=case["tune"])
    x = torch.randn((case["batch"], net.in_c, net.in_h, net.in_w), device="cuda", generator=gen).to(tdt)
    return {"kind": "net", "handle": handle, "x": x, "graph": case["graph"]}


def run(state):
    if state["kind"] == "conv":
        return B.cprune_conv2d_bn_relu(state["d"], state["x"], state["w"], state["bias"], state["res"])
    if state["kind"] == "prune":
        plan = state["plan"]
        plan.run()
        return [plan.kept, plan.w_out, plan.bias_out]
    return state["handle"].forward(state["x"], use_graph=state["graph"])


def work(case):
    es = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "conv":
        k, s, hw, n = case["k"], case["stride"], case["hw"], case["n"]
        ho = (hw + 2 * (k // 2) - k) // s + 1
        out = n * case["c_out"] * ho * ho
        moved = n * case["c_in"] * hw * hw + case["c_out"] * case["c_in"] * k * k + out * (2 if case["residual"] else 1)
        return {"bytes": es * moved + 4 * case["c_out"], "flops": 2.0 * out * case["c_in"] * k * k}
    net = _spec(case)
    keep = _kept_counts(net, case["keep_seed"])
    shp = synth.shapes(net, keep)
    if case["kind"] == "prune":
        # the raw weights of every layer once, the folded weights of the surviving filters and channels once;
        # one absolute value and one addition per weight ranked, one product per weight kept
        ranked = set(keep).union(*[set(L.score_with or []) for L in net.layers])
        read = written = flops = 0
        for i, L in enumerate(net.layers):
            if L.kind not in ("conv", "fc"):
                continue
            per = (L.c_in // L.groups) * L.k * L.k
            kept_rows, kept_cols = shp[i][1], (1 if L.groups != 1 else shp[i][0])
            read += per * (L.c_out if i in ranked else kept_rows)
            written += kept_rows * kept_cols * L.k * L.k
            flops += (per * L.c_out * 2 if i in ranked else 0) + kept_rows * kept_cols * L.k * L.k
        return {"bytes": 4 * read + es * written, "flops": float(flops)}
    macs, weights = synth.count_macs_params(net, keep)
    moved = case["batch"] * (net.in_c * net.in_h * net.in_w + shp[-1][1] * shp[-1][2] * shp[-1][3]) + weights
    return {"bytes": es * moved, "flops": 2.0 * macs * case["batch"]}


# Relative error (2-norm) another correct implementation shows, measured on these networks: fp32, one choice of
# programs against another (another order of the sums), up to 1.4e-6; 16-bit data, the same comparison and the
# path against itself with fp32 activations between the layers on the same rounded weights and input (a fused
# implementation rounds less often than a layer-by-layer one): up to 1e-3 in fp16 and 7e-3 in bf16, 4.7e-3 and
# 3e-2 on MobileNetV2, whose linear bottlenecks carry every rounding to the end.  Stated: about four times that,
# at most 3e-2.
NET_REL = {"f32": 6e-6, "f16": 4e-3, "bf16": 3e-2}
MOBILE_REL = {"f32": 6e-6, "f16": 2e-2, "bf16": 3e-2}
# one layer against double precision: 3e-7 in fp32 at 1152 terms, half a unit in the last place in 16-bit data
CONV_REL = {"f32": 3e-6, "f16": 1e-3, "bf16": 8e-3}


def tolerance(case):
    if case["kind"] == "prune":
        return "exact"      # scores and folds in double, rounded once: kept lists and weights have one value
    if case["kind"] == "conv":
        return {"rel": CONV_REL[case["dtype"]]}
    return {"rel": (MOBILE_REL if case["net"] in ("mobilenetv2", "mnasnet") else NET_REL)[case["dtype"]]}


# ---- the same in 64 bits --------------------------------------------------------------------------

def _act64(y, act):
    return y if act == 0 else y.clamp(min=0) if act == 1 else y.clamp(0, 6)


def _conv64(x, w, bias, stride, pad, groups):
    """Cross-correlation in double; a depthwise layer as the sum of its shifted taps."""
    if groups == 1:
        return torch.nn.functional.conv2d(x, w, bias, stride, pad)
    k, h, wd = w.shape[2], x.shape[2], x.shape[3]
    ho, wo = (h + 2 * pad - k) // stride + 1, (wd + 2 * pad - k) // stride + 1
    xp = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    y = bias.view(1, -1, 1, 1).expand(x.shape[0], -1, ho, wo).clone()
    for u in range(k):
        for v in range(k):
            y += w[:, 0, u, v].view(1, -1, 1, 1) * xp[:, :, u:u + stride * (ho - 1) + 1:stride,
                                                      v:v + stride * (wo - 1) + 1:stride]
    return y


def _prune64(net, params):
    """Kept lists, and every layer's gathered and folded weights and bias, in double."""
    kept = {}
    for i, L in enumerate(net.layers):
        if L.prune_out == "own":
            score = sum(params[j]["w"].abs().flatten(1).sum(1) for j in [i] + list(L.score_with or []))
            first = torch.sort(score, descending=True, stable=True).indices[:params[i]["keep"]]
            kept[i] = first.sort().values
    layers = []
    for i, (L, p) in enumerate(zip(net.layers, params)):
        if L.kind not in ("conv", "fc"):
            layers.append(None)
            continue
        w = p["w"] if L.kind == "conv" else p["w"][:, :, None, None]
        rows = i if L.prune_out == "own" else L.prune_out if isinstance(L.prune_out, int) else None
        if L.prune_in is not None and L.groups == 1:
            w = w[:, kept[L.prune_in]]
        take = kept[rows] if rows is not None else torch.arange(w.shape[0])
        w, b = w[take], p.get("b")
        if L.kind == "conv" and L.bn:
            s = (p["gamma"] / torch.sqrt(p["var"] + pipeline.BN_EPS))[take]
            w, b = w * s.view(-1, 1, 1, 1), p["beta"][take] - p["mean"][take] * s
        layers.append((w, b))
    return kept, layers


def exact(case, seed):
    """What run() returns for these inputs, in double precision on the CPU, from the same inputs as prepare()."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    tdt = B.TORCH_DTYPE[DTYPES[case["dtype"]]]
    F = torch.nn.functional
    if case["kind"] == "conv":
        state = prepare(dict(case, tuned=False), seed)
        x, w, b, res = (None if state[t] is None else state[t].double().cpu() for t in ("x", "w", "bias", "res"))
        y = _conv64(x, w, b, case["stride"], case["k"] // 2, 1)
        return _act64(y if res is None else y + res, case["act"])
    net = _spec(case)
    dev = _device_params(net, _kept_counts(net, case["keep_seed"]), gen)
    params = [{k: v.double().cpu() if torch.is_tensor(v) else v for k, v in p.items()} for p in dev]
    kept, layers = _prune64(net, params)
    if case["kind"] == "prune":
        return [{i: k.to(torch.int32) for i, k in kept.items()},
                {i: q[0] for i, q in enumerate(layers) if q},
                {i: q[1] for i, q in enumerate(layers) if q and net.layers[i].kind == "conv"}]
    x = torch.randn((case["batch"], net.in_c, net.in_h, net.in_w), device="cuda", generator=gen).to(tdt)
    acts = []
    for L, q in zip(net.layers, layers):
        src = x.double().cpu() if L.input < 0 else acts[L.input]
        if L.kind == "conv":
            y = _conv64(src, q[0], q[1], L.stride, L.pad, 1 if L.groups == 1 else src.shape[1])
            y = _act64(y if L.residual is None else y + acts[L.residual], L.act)
        elif L.kind == "maxpool":
            y = F.max_pool2d(src, L.k, L.stride, L.pad)
        elif L.kind == "gavgpool":
            y = src.mean((2, 3), keepdim=True)
        else:
            y = _act64(F.linear(src.flatten(1), q[0].flatten(1), q[1]), L.act)
        acts.append(y)
    return acts[-1]
