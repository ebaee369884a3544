"""The handle of the stream that a call without one runs on: torch's current stream, also where torch lacks the private
functions that give it without a Stream object."""
import pytest

from paper_1507_07733_amd import api

PRIVATE = ("_cuda_getCurrentRawStream", "_cuda_getDevice")


@pytest.mark.parametrize("missing", [PRIVATE[:1], PRIVATE[1:], PRIVATE])
def test_without_the_private_functions(monkeypatch, missing):
    import torch

    class Stream:
        cuda_stream = 0x1507

    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream)
    for name in missing:
        monkeypatch.delattr(torch._C, name, raising=False)
    assert api._stream_handle(None).value == 0x1507
    assert api._stream_handle(Stream).value == 0x1507


@pytest.mark.gpu
def test_is_the_current_stream():
    import torch
    torch.cuda.init()
    side = torch.cuda.Stream()
    for s in (torch.cuda.default_stream(), side):
        with torch.cuda.stream(s):
            assert (api._stream_handle(None).value or 0) == s.cuda_stream
