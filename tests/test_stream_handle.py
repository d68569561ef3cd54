"""The current stream's handle: from torch's raw call, or from the public one
where a torch has no such call."""
import types

import pytest

import paper_1807_06507_amd as swc

torch = pytest.importorskip("torch")


def test_current_stream_without_the_raw_call(monkeypatch):
    asked = []

    def current_stream(device):
        asked.append(device)
        return types.SimpleNamespace(cuda_stream=0x1234)

    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    device = torch.device("cuda", 1)
    assert swc._stream_handle(None, device) == 0x1234
    assert asked == [device]


def test_current_stream_by_the_raw_call(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 0x5000 + index,
                        raising=False)
    assert swc._stream_handle(None, torch.device("cuda", 2)) == 0x5002


def test_given_stream():
    assert swc._stream_handle(types.SimpleNamespace(cuda_stream=7), None) == 7
