"""The Python binding's own checks, on the CPU: no handle is created, no device is touched."""
import os

import pytest
import torch

import paper_1412_7580_amd as pkg


class NoCalls:
    """Stands in for the library: any call is a mistake."""

    def __getattr__(self, name):
        raise AssertionError(f"{name} was called")


def test_a_handle_in_a_forked_process_is_refused(monkeypatch):
    """As torch's own stream query does: the device must not be touched from a child forked after its initialisation."""
    pkg.load_library()
    h = pkg.Handle.__new__(pkg.Handle)
    h._lib, h._h, h.device, h._stream = NoCalls(), None, 0, 0
    monkeypatch.setattr(pkg, "_forked", True)
    monkeypatch.setattr(torch.cuda, "_initialized", True)
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: True)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 0)
    with pytest.raises(RuntimeError, match="forked subprocess"):
        h._sync_stream()


def test_a_forked_process_knows_that_it_is_one():
    pkg.load_library()
    child = os.fork()
    if child == 0:
        os._exit(7 if pkg._forked else 8)
    assert os.waitstatus_to_exitcode(os.waitpid(child, 0)[1]) == 7
    assert not pkg._forked


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_the_stream_without_the_private_queries(monkeypatch, missing):
    """torch's raw-handle queries are not part of its interface: without them the public one serves."""
    class Stream:
        cuda_stream = 0x1234

    told = []

    class Library(NoCalls):
        def fftconv_set_stream(self, handle, stream):
            told.append(stream.value)
            return 0

    pkg.load_library()
    h = pkg.Handle.__new__(pkg.Handle)
    h._lib, h._h, h.device, h._stream = Library(), None, 0, 0
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    monkeypatch.delattr(torch._C, missing)
    h._sync_stream()
    assert told == [0x1234] and h._stream == 0x1234
