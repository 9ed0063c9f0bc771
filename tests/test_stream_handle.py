"""The stream that a call without `stream` runs on: torch's current one, also under a torch that does not hand out its bare handle."""
import types

import torch

from paper_2602_05853_amd import binding as bd


def test_current_stream_without_the_raw_handle(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1234))
    assert bd._stream_ptr(None) == 0x1234


def test_raw_handle_is_that_of_the_current_device(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x1000 + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert bd._stream_ptr(None) == 0x1003


def test_a_stream_that_is_given():
    assert bd._stream_ptr(types.SimpleNamespace(cuda_stream=0x77)) == 0x77
