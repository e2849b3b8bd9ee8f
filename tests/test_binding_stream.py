"""The stream a call goes to when its caller names none (CPU only)."""
import types

import torch

from paper_2412_11272_amd import binding as wf


def test_callers_stream_comes_first():
    assert wf._raw_stream(0) == 0 and wf._raw_stream(77) == 77


def test_current_stream_by_either_way(monkeypatch):
    """torch's raw handle where it exists, the public Stream object where it does not."""
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    assert wf._raw_stream(None) == 103
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=55))
    assert wf._raw_stream(None) == 55
