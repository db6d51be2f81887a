"""The stream handle that every call passes on: PyTorch's own where it has one, else the public
Stream object's."""
import torch

import paper_1910_03032_amd as sfem


class _Stream:
    cuda_stream = 77


def test_handle_without_the_raw_call(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda index: _Stream)
    assert sfem._stream_handle(0) == 77


def test_handle_with_the_raw_call(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 10 + index, raising=False)
    assert sfem._stream_handle(3) == 13
