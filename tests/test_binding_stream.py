"""The stream argument of the Python binding, without a GPU: what is no stream is refused before it reaches the
library, and the cached look-up of the current stream leaves none of torch's checks out."""
import ctypes
import os

import pytest

import paper_2609_28519_amd as dct


@pytest.mark.parametrize("stream", ("text", b"bytes", 1.5, ctypes.c_void_p(8), (ctypes.c_int * 2)(), ctypes.byref(ctypes.c_int(0))))
def test_only_handles_are_streams(stream):
    with pytest.raises(TypeError):
        dct._stream(stream)


def test_handles_and_stream_objects():
    class Stream:
        cuda_stream = 4096

    assert dct._stream(Stream()).value == dct._stream(4096).value == 4096
    assert dct._stream(0).value is None  # the null stream


def test_failed_look_up_is_not_cached(monkeypatch):
    import torch

    def refuse():
        raise RuntimeError("no usable GPU in this process")

    monkeypatch.setattr(torch.cuda, "current_stream", refuse)
    monkeypatch.setattr(dct, "_current", None)
    with pytest.raises(RuntimeError):
        dct._stream(None)
    assert dct._current is None


def test_forked_process_asks_again(monkeypatch):
    monkeypatch.setattr(dct, "_current", lambda: 1)
    pid = os.fork()
    if pid == 0:
        os._exit(0 if dct._current is None else 1)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
    assert dct._current is not None
