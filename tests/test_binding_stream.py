"""Which stream a call of the binding runs on: the one it is given, else torch's current one - by its handle where torch tells it, else
through the stream object."""
from types import SimpleNamespace

import torch

from paper_2605_09649_amd import binding


def test_stream_handles(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(binding, "_raw_stream", lambda device: 100 + device)
    assert binding._stream(None) == 103 and binding._stream(SimpleNamespace(cuda_stream=5)) == 5
    monkeypatch.setattr(binding, "_raw_stream", None)
    assert binding._stream(None) == 77 and binding._stream(SimpleNamespace(cuda_stream=5)) == 5
