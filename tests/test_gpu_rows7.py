"""Row strips of seven rows: maps of fewer rows than one strip, of exactly one and two, of one more and one less, strips of one, two and
four images with some missing, fewer chunks of channels than wavefronts, partial filter tiles; with a shortcut; in three types, against
the oracle.  A fused 2x2 max-pool over pairs of rows is refused."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import nmax

pytestmark = pytest.mark.gpu


def _sevens(dtype):
    names = {v: B.cprune_tile_variant_name(v, True, dtype) for v in range(B.cprune_num_tile_variants())}
    return {v: n for v, n in names.items() if n.startswith(("conv_rows_kernel", "conv_split_rows")) and
            int(n.split("<")[1].rstrip(">").split(",")[-2 if n.startswith("conv_rows") else 0]) == 7}


@pytest.mark.parametrize("dtype,tol", [(B.F32, 1e-4), (B.F16, 2e-2), (B.BF16, 2e-2)])     # the bars every other conv test states
@pytest.mark.parametrize("c_in,c_out,hw,batch,shortcut", [
    (33, 20, 7, 3, True),        # one strip of rows, two images a strip, one missing
    (140, 37, 14, 2, False),     # two strips of rows; five chunks of channels
    (70, 16, 15, 1, True),       # one row into a third strip
    (40, 33, 6, 3, True),        # a strip with a row missing
    (65, 50, 4, 5, False),       # four images a strip, three missing
    (32, 17, 17, 1, True),       # a column into a second strip, four rows of a third
    (20, 24, 28, 2, False),
])
def test_seven_rows(orc, dtype, tol, c_in, c_out, hw, batch, shortcut):
    net = synth.NetSpec(f"rows7_{c_in}_{hw}", 3, hw, hw)
    a = net.add(synth.Layer("conv", -1, 3, c_in, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    r = net.add(synth.Layer("conv", -1, 3, c_out, k=1, act=synth.ACT_NONE, bn=True, name="r")) if shortcut else None
    b = net.add(synth.Layer("conv", a, c_in, c_out, k=3, stride=1, pad=1, act=synth.ACT_RELU, bn=True, residual=r, name="b"))
    params = synth.layer_params(net, 84)
    x = synth.net_input(net, 84, batch)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    sevens = _sevens(dtype)
    chunks = (c_in + 31) // 32
    ran = 0
    for v, name in sevens.items():
        print(name, flush=True)
        info = [int(t) for t in name.split("<")[1].rstrip(">").split(",") if t.strip().isdigit()]
        try:
            handle.set_layer_variant(b, v)
        except B.CPruneError as e:
            # two filter tiles a wavefront: 16-bit data only; wavefronts share a strip only while there is a chunk of 32 channels for each
            assert e.status == B.ERR_UNSUPPORTED and (dtype == B.F32 or info[-1] > chunks), name
            continue
        out = handle.forward(xd)
        torch.cuda.synchronize()
        assert nmax(out.float().cpu().numpy(), ref) < tol, name
        ran += 1
    assert ran == (1 if dtype == B.F32 else 2) * sum(ks <= chunks for ks in (1, 2, 4))
    handle.close()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_seven_rows_refuse_a_fused_pool(dtype):
    net = synth.NetSpec("rows7_pool", 3, 14, 14)
    a = net.add(synth.Layer("conv", -1, 3, 40, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    b = net.add(synth.Layer("conv", a, 40, 32, k=3, stride=1, pad=1, act=synth.ACT_RELU, bn=True, name="b"))
    p = net.add(synth.Layer("maxpool", b, 32, 32, k=2, stride=2, name="p"))
    net.add(synth.Layer("conv", p, 32, 8, k=1, act=synth.ACT_NONE, bn=True, name="c"))
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(synth.layer_params(net, 85)), dtype)
    handle = pipeline.build_net(net, layers, 2, dtype, tune=False)
    for v in _sevens(dtype):
        with pytest.raises(B.CPruneError) as e:
            handle.set_layer_variant(b, v)
        assert e.value.status == B.ERR_UNSUPPORTED
    handle.close()
