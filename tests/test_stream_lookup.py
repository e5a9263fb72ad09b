"""The caller's stream: torch's own call initialises the device, or says why it cannot; what is asked for afterwards is optional."""
import os
import types

import pytest
import torch

from paper_2207_01260_amd import binding as B


@pytest.fixture()
def calls(monkeypatch):
    made = []

    def current_stream():
        made.append("torch")
        return types.SimpleNamespace(cuda_stream=17)

    def raw(device):
        made.append(("raw", device))
        return 18

    monkeypatch.setattr(B, "_raw_lookup", None)
    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", raw, raising=False)
    return made


def test_the_first_lookup_is_torchs(calls):
    assert B._raw_stream() == 17 and B._raw_stream() == 18 and B._stream().value == 18
    assert calls == ["torch", ("raw", 3), ("raw", 3)]
    assert B._raw_stream(types.SimpleNamespace(cuda_stream=5)) == 5


@pytest.mark.parametrize("name", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_a_torch_without_the_direct_lookup(calls, monkeypatch, name):
    monkeypatch.delattr(torch._C, name)
    assert B._raw_stream() == 17 and B._raw_stream() == 17
    assert calls == ["torch", "torch"]


def test_no_device_is_an_error_as_torch_states_it(calls, monkeypatch):
    def none():
        raise RuntimeError("no device")
    monkeypatch.setattr(torch.cuda, "current_stream", none)
    for _ in range(2):
        with pytest.raises(RuntimeError, match="no device"):
            B._raw_stream()


def test_a_forked_child_asks_torch_again(calls):
    B._raw_stream()
    read, write = os.pipe()
    child = os.fork()
    if child == 0:
        os.write(write, b"%d" % B._raw_stream())
        os._exit(0)
    os.waitpid(child, 0)
    assert os.read(read, 8) == b"17" and B._raw_stream() == 18
