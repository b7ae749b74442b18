"""The handle of the current stream: refused where torch refuses the device (a
forked child of a process that uses the GPU), the Stream object's where torch
has no shorter way."""
import types

import pytest
import torch

from paper_1807_02284_amd import level


def test_no_handle_where_torch_refuses_the_device(monkeypatch):
    def refuse():
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")

    monkeypatch.setattr(torch.cuda, "_lazy_init", refuse)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 7, raising=False)
    monkeypatch.setattr(level, "_raw_stream", lambda device: 7, raising=False)
    with pytest.raises(RuntimeError, match="forked"):
        level._stream_handle()


def test_stream_object_without_the_short_way(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 2)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda device=None: types.SimpleNamespace(cuda_stream=100 + device))
    monkeypatch.setattr(level, "_raw_stream", None)
    assert level._stream_handle() == 102
    assert level._stream_handle(types.SimpleNamespace(cuda_stream=5)) == 5


@pytest.mark.gpu
def test_handle_is_the_current_stream():
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    assert level._stream_handle() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert level._stream_handle() == side.cuda_stream
