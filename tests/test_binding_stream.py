"""The binding's stream handle where torch has its private raw-stream call and where it does not.  No GPU needed."""
from types import SimpleNamespace

import torch

from paper_2605_22428_amd import binding as B


def test_stream_handle_with_and_without_the_private_call(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(B, "_raw_stream", lambda device: 1000 + device)
    assert B._stream_handle() == 1003
    monkeypatch.setattr(B, "_raw_stream", None)
    assert B._stream_handle() == 77
