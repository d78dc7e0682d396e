"""Where the binding takes the stream of a call without a stream argument from.  No device is used: torch's side is replaced."""
import os
import types

import pytest
import torch

from paper_2103_15195_amd import binding as B


@pytest.fixture
def current(monkeypatch):
    """torch.cuda.current_stream() as a program that changes streams sees it."""
    now = types.SimpleNamespace(cuda_stream=42)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: now)
    monkeypatch.setattr(B, "_raw_stream", None)
    return now


def test_raw_lookup(current, monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    assert B._stream_handle(None) == 103 and B._stream_handle(current) == 42 and B._stream_handle(7) == 7


@pytest.mark.parametrize("missing", ["_cuda_getDevice", "_cuda_getCurrentRawStream"])
def test_without_the_raw_lookup(current, monkeypatch, missing):
    """A torch that lacks either function: the public one, asked again in every call."""
    for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
        monkeypatch.setattr(torch._C, name, lambda *a: 0, raising=False)
    monkeypatch.delattr(torch._C, missing)
    assert B._stream_handle(None) == 42
    current.cuda_stream = 43
    assert B._stream_handle(None) == 43


def test_a_forked_child_asks_torch_again(monkeypatch):
    """torch refuses to use a device that the parent process has initialised.  The raw lookup does not, so a child must not
    go on with its parent's."""
    monkeypatch.setattr(B, "_raw_stream", lambda: 42)

    def refuses():
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")
    monkeypatch.setattr(torch.cuda, "current_stream", refuses)
    assert B._stream_handle(None) == 42
    pid = os.fork()
    if pid == 0:
        try:
            B._stream_handle(None)
        except RuntimeError:
            os._exit(0)
        finally:
            os._exit(1)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
