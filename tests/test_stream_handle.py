"""The launch stream's handle, with and without torch's raw-stream call (no GPU)."""
import types

import torch

from paper_2607_14054_amd import sosfilt as S


def test_current_stream_without_the_raw_call(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4321))
    assert S._stream_ptr(None) == 4321


def test_current_stream_with_the_raw_call(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 7)
    assert S._stream_ptr(None) == 107
    assert S._stream_ptr(types.SimpleNamespace(cuda_stream=5)) == 5
