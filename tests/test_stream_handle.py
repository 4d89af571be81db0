"""The stream that the binding hands to the library: a given one, else the current device's current one, with and without the
private torch function that returns its handle."""
import torch

from paper_2605_18643_amd import zeda


class _Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


def test_current_stream_by_handle_or_by_object(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: _Stream(0x55))
    assert zeda._stream(_Stream(0x77)) == 0x77
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x40 + device, raising=False)
    assert zeda._stream(None) == 0x43
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert zeda._stream(None) == 0x55
