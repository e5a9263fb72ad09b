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
