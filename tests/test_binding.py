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


@pytest.mark.parametrize("rank", [8, 64, 0, -8, 2 ** 31, 2 ** 32 + 8, True])
def test_adapter_descriptors_hold_what_a_structure_would(rank):
    got = vq._lora_array([4096, 0], [8192, None], [rank, 16])
    want = (vq.VQLoraDesc * 2)(vq.VQLoraDesc(4096, 8192, rank, 0), vq.VQLoraDesc(0, 0, 16, 0))
    assert bytes(got) == bytes(want) and ctypes.sizeof(got) == 48


def test_a_rank_out_of_range_is_the_library_s_error():
    desc = vq.make_desc(256, 256, 16, 4)
    args = vq.GemvMultiArgs([desc], [1 << 20], [1 << 21], [1 << 22], [1 << 23])
    for rank in (2 ** 31, -8, 12, 72):
        with pytest.raises(vq.VQError):
            vq.vq_gemv_lora_multi(args, [1 << 24], [1 << 25], [rank], 1 << 26, stream=0, workspace_bytes=1 << 16)
    with pytest.raises(TypeError):
        vq.vq_gemv_lora_multi(args, [1 << 24], [1 << 25], [8.0], 1 << 26, stream=0, workspace_bytes=1 << 16)
