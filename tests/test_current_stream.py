"""The binding finds torch's current stream with and without torch's non-public
raw-handle function (no GPU needed: torch's side is replaced)."""
from types import SimpleNamespace

import torch

from paper_2604_03585_amd import _lib


def test_without_the_raw_handle_function(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(_lib, "_current_raw_stream", None, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: SimpleNamespace(cuda_stream=0x1230))
    assert _lib._stream(None) == 0x1230


def test_with_it(monkeypatch):
    monkeypatch.setattr(_lib, "_current_raw_stream", lambda device: 0x4560 + device)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 2)
    assert _lib._stream(None) == 0x4562


def test_given_streams():
    assert _lib._stream(0x789) == 0x789
    assert _lib._stream(SimpleNamespace(cuda_stream=0x99)) == 0x99
