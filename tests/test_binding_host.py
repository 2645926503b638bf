"""The binding's host side, without a GPU."""
import types

import pytest
import torch

from paper_2501_01792_amd import binding


def test_current_stream_without_torchs_own_shortcut(monkeypatch):
    """A build of torch that lacks the undocumented calls for a stream's handle still has torch.cuda.current_stream."""
    monkeypatch.setattr(binding, "_current_stream", None)
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1230))
    assert binding._stream_ptr(None) == 0x1230
    assert binding._stream_ptr(types.SimpleNamespace(cuda_stream=0x4560)) == 0x4560


def test_a_layer_without_its_tensors_is_refused():
    """Before the library is asked: a step over cached tokens alone does not read the layer, and would take null pointers."""
    with pytest.raises(AttributeError):
        binding._params(None, None, None, None)
