"""The handle of the current stream that every call passes on, on the CPU: from
torch's direct accessor, and from the public stream object where a torch build
has none."""
from __future__ import annotations

import types

from paper_2503_01582_amd import api


def test_stream_handle(monkeypatch):
    torch = api.torch
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(api, "_raw_stream", lambda device: 1000 + device)
    assert api._stream() == 1003
    monkeypatch.setattr(api, "_raw_stream", None)
    assert api._stream() == 77
