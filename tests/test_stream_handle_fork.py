"""A forked child of a process that has used the GPU is refused with an error, also where the parent has already
looked up how to ask torch for the stream (torch's C layer itself does not check)."""
import types

import pytest

from paper_2302_01382_amd import mpq


def test_a_forked_child_is_refused(monkeypatch):
    forked = [False]

    def init():
        if forked[0]:
            raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")

    c = types.SimpleNamespace(_cuda_getCurrentRawStream=lambda device: 1000 + device, _cuda_getDevice=lambda: 3,
                              _cuda_isInBadFork=lambda: forked[0])
    monkeypatch.setattr(mpq, "_torch", lambda: types.SimpleNamespace(_C=c, cuda=types.SimpleNamespace(init=init)))
    monkeypatch.setattr(mpq, "_raw_stream", None)
    assert mpq._stream() == 1003
    forked[0] = True
    with pytest.raises(RuntimeError, match="forked"):
        mpq._stream()
