"""The Python binding's own decisions (no GPU needed): the current stream's handle, and adapter descriptors."""
import ctypes
from types import SimpleNamespace

import pytest

import paper_2402_15319_amd as vq


def _fake_torch(**private):
    cuda = SimpleNamespace(is_initialized=lambda: True, current_stream=lambda: SimpleNamespace(cuda_stream=77))
    return SimpleNamespace(cuda=cuda, _C=SimpleNamespace(**private))


@pytest.mark.parametrize("private, want", [
    (dict(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda d: 100 + d), 103),
    (dict(_cuda_getDevice=lambda: 3), 77),
    ({}, 77),
], ids=["both", "one", "none"])
def test_current_stream_with_and_without_the_private_functions(monkeypatch, private, want):
    monkeypatch.setattr(vq, "_torch", _fake_torch(**private))
    assert vq._stream(None) == want
    assert vq._stream(5) == 5
