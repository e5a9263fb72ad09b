"""The peak that the report holds a layer's time against is that of the kernel it runs in."""
import pytest

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import report, synth


class _Handle:
    def __init__(self, variants, fused):
        self.layer_variant, self.layer_fused = variants.__getitem__, fused.__getitem__


def _variant(name, dtype):
    return next(v for v in range(B.cprune_num_tile_variants()) if B.cprune_tile_variant_name(v, True, dtype).startswith(name))


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_layers_without_a_variant_of_their_own(dtype):
    net = synth.NetSpec("peaks", 3, 64, 64)
    a = net.add(synth.Layer("conv", -1, 3, 32, k=7, stride=2, pad=3, name="a"))
    b = net.add(synth.Layer("maxpool", a, 32, 32, k=3, stride=2, pad=1, name="b"))
    net.add(synth.Layer("conv", b, 32, 64, k=1, stride=2, pad=0, name="c"))
    net.add(synth.Layer("conv", b, 32, 64, k=3, stride=2, pad=1, name="d"))
    net.add(synth.Layer("conv", 3, 64, 64, k=3, stride=1, pad=1, residual=2, name="e"))
    igemm = _variant("conv_nhwc_kernel", dtype)
    handle = _Handle([-1, -1, -1, _variant("conv_rows_s2", dtype), igemm], [False, False, True, False, False])
    peaks = [report.kernel_peak(k, dtype) for k in report.layer_kernels(net, handle, dtype)]
    if dtype == B.F32:
        parts, whole = report.PEAK_TFLOPS[B.BF16] / 6, report.PEAK_TFLOPS[B.F32]
        assert peaks == [parts, whole, parts, parts, whole]
        assert report.kernel_peak(report.layer_kernels(net, handle, dtype, first_layer_form=0)[0], dtype) == whole
    else:
        assert set(peaks) == {report.PEAK_TFLOPS[dtype]}


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("k,c_out,fused,on_parts", [
    (3, 32, (True, True), (True, True)), (3, 96, (True, True), (True, True)), (3, 97, (True, True), (False, False)),
    (5, 32, (True, True), (False, False)), (3, 32, (False, True), (False, True)), (3, 32, (False, False), (False, False)),
])
@pytest.mark.parametrize("image", [False, True])
def test_blocks_in_one_kernel(dtype, k, c_out, fused, on_parts, image):
    """Expansion (or the network's first layer) and projection around a depthwise layer, as one kernel, with the depthwise layer only, apart."""
    net = synth.NetSpec("blocks", 3, 64, 64)
    a = -1 if image else net.add(synth.Layer("conv", -1, 3, 24, k=1, name="a"))
    e = net.add(synth.Layer("conv", a, 3 if image else 24, 40, k=3 if image else 1, stride=2 if image else 1, pad=1 if image else 0, prune_out="own", name="e"))
    d = net.add(synth.Layer("conv", e, 40, 40, k=k, stride=1, pad=k // 2, groups=40, prune_out=e, name="d"))
    p = net.add(synth.Layer("conv", d, 40, c_out, k=1, name="p"))
    handle = _Handle([-1] * len(net.layers), [False] * (e) + [fused[0], fused[1], False])
    peaks = [report.kernel_peak(name, dtype) for name in report.layer_kernels(net, handle, dtype)]
    parts, whole = report.PEAK_TFLOPS[B.BF16] / 6, report.PEAK_TFLOPS[dtype]
    want = [parts if dtype == B.F32 and on else whole for on in on_parts]
    assert [peaks[e], peaks[p]] == want
    # few terms without an expansion: the fp32 instruction, by what is left of the layer
    few = report.layer_kernels(net, handle, B.F32, kept_counts={e: 15})
    assert (few[p] == "mbrow3_kernel") == (all(fused) and on_parts[1])
