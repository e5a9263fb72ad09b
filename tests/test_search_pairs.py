"""What the search makes of a 1x1 layer that runs in a 3x3 layer's launch."""
import pytest

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import search, synth


def _net():
    net = synth.NetSpec("pairs", 16, 16, 16)
    a = net.add(synth.Layer("conv", -1, 16, 32, k=3, stride=1, pad=1, name="a"))
    net.add(synth.Layer("conv", a, 32, 64, k=3, stride=2, pad=1, name="b"))
    net.add(synth.Layer("conv", a, 32, 128, k=1, stride=2, pad=0, name="c"))
    net.add(synth.Layer("conv", 1, 64, 128, k=3, stride=1, pad=1, residual=2, name="d"))
    net.add(synth.Layer("conv", 3, 128, 128, k=3, stride=2, pad=1, name="e"))
    net.add(synth.Layer("conv", 3, 128, 96, k=1, stride=2, pad=0, name="f"))
    return net


def test_time_and_program_of_a_pair_belong_to_both_layers():
    net = _net()
    shp = synth.shapes(net, {})
    fused, variants, times = [False, False, True, False, False, True], [5, 250, -1, 5, 252, -1], [1.0, 7.0, 0.0, 2.0, 3.9, 0.0]
    pairs = search.paired_layers(net, fused, variants, {250, 252})
    assert pairs == {2: 1, 5: 4}
    got = search.shared_times(net, times, pairs, shp)
    assert got[0] == 1.0 and got[3] == 2.0
    assert got[1] + got[2] == pytest.approx(7.0) and got[2] / got[1] == pytest.approx(128 / (9 * 64))
    assert got[4] + got[5] == pytest.approx(3.9) and got[5] / got[4] == pytest.approx(96 / (9 * 128))
    # layers apart keep what they report
    assert search.paired_layers(net, [False] * 6, [5] * 6, {250, 252}) == {}
    assert search.paired_layers(net, fused, [5, 5, -1, 5, 252, -1], {252}) == {5: 4}


@pytest.mark.gpu
def test_no_task_of_a_residual_network_is_free():
    """ResNet-18 with prunable shortcuts in bf16, where pairs form: every task has a time, a paired layer's is a share of its launch's and
    its step that of the launch's tiles."""
    net = synth.resnet18(10, 64, prune_shortcuts=True)
    params = synth.layer_params(net, 3)
    ds = search.DeviceSearch(net, params, 3, batch=2, dtype=B.BF16, steps=5)
    table, order = ds.tune(ds.initial_model(params))
    assert sorted(map(str, order)) == sorted(map(str, table))
    halving = {i for i, L in enumerate(net.layers) if L.kind == "conv" and L.k == 1 and L.stride == 2}
    assert halving
    for layers, program in table.values():
        assert program["time_ms"] > 0 and program["impact"] > 0, layers
        if halving & set(layers):
            assert program["variant"] >= 0
            assert program["step"] == B.cprune_variant_prune_step(program["variant"], program["c_out"])
