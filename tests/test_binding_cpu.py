"""The Python binding where torch's own internal names, which it asks for
speed, are not there: the public calls answer instead."""
import types

import pytest
import torch

import paper_2209_08241_amd as bn


@pytest.mark.parametrize("name", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_internal_names(monkeypatch, name):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 5, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=77))
    assert bn._stream_handle(None) == 5
    monkeypatch.delattr(torch._C, name)
    assert bn._stream_handle(None) == 77


@pytest.mark.parametrize("owner,name", [(torch._C._functorch, "peek_interpreter_stack"),
                                        (torch.autograd.forward_ad, "_current_level"),
                                        (torch._C, "_len_torch_dispatch_stack"),
                                        (torch._C, "_len_torch_function_stack")])
def test_transforms_that_cannot_be_asked_for(monkeypatch, owner, name):
    """What cannot be ruled out keeps the loss on tensor operations."""
    assert bn._eager()
    monkeypatch.delattr(owner, name)
    assert not bn._eager()


def test_storage_that_cannot_be_asked_for(monkeypatch):
    t = torch.zeros(2, 3)
    assert bn._dense(t, torch.float32, t.shape, t.device)
    monkeypatch.delattr(torch._C, "_has_storage")
    assert not bn._dense(t, torch.float32, t.shape, t.device)
