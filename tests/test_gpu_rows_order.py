"""Row strips whose weights are the larger operand (over 3 MB): the work-groups run filter tile by filter tile.  Grids that are no
multiple of eight, a last work-group with strips missing, a partial last filter tile; every variant, both strides, against the oracle."""
import pytest
import torch

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import pipeline, synth
from parity import nmax

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(B.F32, 1e-4), (B.BF16, 2e-2)])     # the bars every other conv test states
@pytest.mark.parametrize("c_in,c_out,hw,batch,stride", [
    (430, 435, 4, 6, 1),      # four images a strip, two of the last one's missing; 28 filter tiles, the last one of 3 filters
    (421, 449, 7, 3, 1),      # two images a strip
    (440, 417, 9, 1, 1),      # one strip of two (four) rows of strips
    (433, 445, 6, 5, 2),      # stride 2, on its own
])
def test_rows_filter_tiles_slowest(orc, dtype, tol, c_in, c_out, hw, batch, stride):
    net = synth.NetSpec(f"order_{c_in}_{hw}", 3, hw, hw)
    a = net.add(synth.Layer("conv", -1, 3, c_in, k=1, act=synth.ACT_RELU, bn=True, name="a"))
    b = net.add(synth.Layer("conv", a, c_in, c_out, k=3, stride=stride, pad=1, act=synth.ACT_RELU, bn=True, name="b"))
    params = synth.layer_params(net, 83)
    x = synth.net_input(net, 83, batch)
    ref_layers, _ = orc.prune_net(net, params)
    ref = orc.forward(net, ref_layers, x)
    layers, _ = pipeline.prune_net(net, pipeline.upload_params(params), dtype)
    handle = pipeline.build_net(net, layers, batch, dtype, tune=False)
    xd = torch.from_numpy(x).cuda().to(B.TORCH_DTYPE[dtype])
    ran = 0
    for v in range(B.cprune_num_tile_variants()):
        name = B.cprune_tile_variant_name(v, True, dtype)
        if not name.startswith(("conv_rows", "conv_split_rows")):
            continue
        try:
            handle.set_layer_variant(b, v)
        except B.CPruneError as e:
            assert e.status == B.ERR_UNSUPPORTED
            continue
        print(name, flush=True)
        out = handle.forward(xd)
        torch.cuda.synchronize()
        assert nmax(out.float().cpu().numpy(), ref) < tol, name
        ran += 1
    assert ran >= 4
    handle.close()
