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
