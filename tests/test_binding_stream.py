"""The current stream as a handle, with and without torch's shortcut to it."""
from __future__ import annotations

import types


def test_stream_handle(monkeypatch):
    import torch

    from paper_1709_03708_amd import binding

    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=7))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    assert binding._stream() == 103
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert binding._stream() == 7
