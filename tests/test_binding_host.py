"""What the binding keeps between calls: the way to the current stream's handle, and small int32 arrays."""
import os
import sys
import types

import pytest

from paper_2512_17452_amd import binding


class _Stream:
    cuda_stream = 4711


def _fake_torch(monkeypatch, private):
    """A torch whose public call gives stream 4711; private: the functions of torch._C."""
    t = types.ModuleType("torch")
    t._C = types.SimpleNamespace(**private)
    t.inits = 0

    def init():
        t.inits += 1
    t.cuda = types.SimpleNamespace(init=init, current_stream=_Stream)
    monkeypatch.setitem(sys.modules, "torch", t)
    monkeypatch.setattr(binding, "_current_stream", None)
    return t


@pytest.mark.parametrize("private", [{}, {"_cuda_getDevice": lambda: 0}, {"_cuda_getDevice": lambda: 0, "_cuda_getCurrentRawStream": lambda d: 1},
                                     {"_cuda_getDevice": lambda: 3, "_cuda_getCurrentRawStream": lambda d: 4711 if d == 3 else 0}],
                         ids=["none", "one", "disagree", "both"])
def test_stream_with_and_without_torchs_own_names(monkeypatch, private):
    t = _fake_torch(monkeypatch, private)
    assert binding._stream() == 4711 and binding._stream() == 4711 and t.inits == 1


def test_a_forked_child_asks_torch_again(monkeypatch):
    _fake_torch(monkeypatch, {})
    binding._stream()
    assert binding._current_stream is not None
    pid = os.fork()
    if pid == 0:
        os._exit(0 if binding._current_stream is None else 1)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
    assert binding._current_stream is not None


def test_long_lists_are_not_kept():
    kept = binding._kept_array.cache_info().currsize
    for n in range(300, 320):
        assert list(binding._ids(range(n))) == list(range(n))
    assert binding._kept_array.cache_info().currsize == kept
    assert binding._ids([5, 7]) is binding._ids((5, 7))
