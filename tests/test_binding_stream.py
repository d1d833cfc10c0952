"""The stream that the binding hands on: torch's current one, with and without torch's shortcut to its handle."""
from types import SimpleNamespace

import pytest
import torch

import paper_2006_12575_amd.binding as B


@pytest.mark.parametrize("missing", ["_raw_stream", "_device"])
def test_stream_without_the_shortcut(monkeypatch, missing):
    monkeypatch.setattr(B, missing, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=1234))
    assert B._stream() == 1234


@pytest.mark.gpu
def test_stream_is_the_current_one(monkeypatch):
    s = torch.cuda.Stream()
    for shortcut in (True, False):
        if not shortcut:
            monkeypatch.setattr(B, "_raw_stream", None)
        assert B._stream() == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(s):
            assert B._stream() == s.cuda_stream
