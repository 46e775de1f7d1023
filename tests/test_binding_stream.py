"""The stream that a launch without one goes on, where torch lacks the private
calls that read the current stream's raw handle: the public stream object's."""
import importlib.util
import types

import pytest
import torch

import paper_2509_17542_amd as K


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_without_the_raw_stream_calls(monkeypatch, missing):
    monkeypatch.delattr(torch._C, missing, raising=False)
    spec = importlib.util.spec_from_file_location("kvx_without_raw_stream", K.__file__)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=0x1234))
    assert mod._stream(None) == 0x1234
    assert mod._stream(0x99) == 0x99
