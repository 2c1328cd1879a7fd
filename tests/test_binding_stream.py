"""The binding's stream handle with and without torch's own short way to it (no GPU)."""
from types import SimpleNamespace

import pytest

import paper_2603_13147_amd as llp


@pytest.mark.parametrize("raw", [True, False])
def test_handle(monkeypatch, raw):
    stream = SimpleNamespace(cuda_stream=0x1234)
    torch = SimpleNamespace(
        _C=SimpleNamespace(_cuda_getCurrentRawStream=lambda device: 0x1000 + device) if raw else SimpleNamespace(),
        cuda=SimpleNamespace(current_device=lambda: 3, current_stream=lambda: stream))
    monkeypatch.setattr(llp, "_torch", lambda: torch)
    assert llp._stream().value == (0x1003 if raw else 0x1234)
