"""CPU checks of how Sim's calls find torch's current stream, with stand-ins for torch and the
library: in a forked child of a process that has initialised the GPU, torch refuses GPU work,
and so must a Sim that the child inherited, before anything reaches the library."""
import types

import pytest

from paper_2410_14117_amd import mg


def _sim(monkeypatch, initialised, init):
    calls = []
    cuda = types.SimpleNamespace(is_initialized=lambda: initialised, init=init)
    c = types.SimpleNamespace(_cuda_getDevice=lambda: 0,
                              _cuda_getCurrentRawStream=lambda device: 77 + device)
    lib = types.SimpleNamespace(mg_set_stream=lambda h, s: calls.append((h, s)) or 0)
    monkeypatch.setattr(mg, "_torch", types.SimpleNamespace(cuda=cuda, _C=c))
    monkeypatch.setattr(mg, "_lib", lib)
    sim = mg.Sim.__new__(mg.Sim)
    sim._h = 5
    return sim, calls


def test_the_current_stream_is_bound(monkeypatch):
    def init():
        raise AssertionError("already initialised")
    sim, calls = _sim(monkeypatch, True, init)
    sim._bind_stream()
    sim._h = None                  # nothing to destroy
    assert calls == [(5, 77)]


def test_a_forked_child_is_refused(monkeypatch):
    def init():
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")
    sim, calls = _sim(monkeypatch, False, init)
    try:
        with pytest.raises(RuntimeError, match="forked"):
            sim._bind_stream()
    finally:
        sim._h = None
    assert not calls
