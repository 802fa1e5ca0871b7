"""The binding's way to the current stream, with and without the handle torch keeps under private names."""
import importlib.util
import sys
import types

import torch

import paper_2502_14866_amd.binding as B


def test_the_current_stream_without_torchs_private_names(monkeypatch):
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1234))
    spec = importlib.util.spec_from_file_location("binding_on_another_torch", B.__file__)  # a copy of its own
    module = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(sys.modules, spec.name, module)
    spec.loader.exec_module(module)
    assert module._stream(None) == 0x1234


def test_streams_that_are_handed_in():
    assert B._stream(7) == 7
    assert B._stream(types.SimpleNamespace(cuda_stream=0x77)) == 0x77
