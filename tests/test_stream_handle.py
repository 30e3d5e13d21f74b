"""The stream handle that the binding passes to the library, with and without
torch's own call for the raw handle."""
import types

import torch

from paper_2311_11700_amd import renderer


def test_stream_handle_without_the_raw_call(monkeypatch):
    monkeypatch.setattr(renderer, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    assert renderer._stream_ptr() == 1234
    assert renderer._stream_ptr(types.SimpleNamespace(cuda_stream=77)) == 77


def test_stream_handle_with_the_raw_call(monkeypatch):
    monkeypatch.setattr(renderer, "_raw_stream", lambda device: 4000 + device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert renderer._stream_ptr() == 4003
