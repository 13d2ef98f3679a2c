"""The array of chain handles that a batched call passes on: from Chain objects
and from bare handles, null ones included (the library refuses those)."""
import ctypes as C

import pytest

import synth
from paper_1712_05012_amd import kcm


def _chain(handle):
    c = object.__new__(kcm.Chain)  # no device block: a handle and nothing else
    c.handle = handle
    return c


def _values(arr):
    return [arr[i] for i in range(len(arr))]


def test_null_and_bare_handles_reach_the_library():
    assert _values(kcm._handles([C.c_void_p(None), C.c_void_p(16)])) == [None, 16]
    c = _chain(C.c_void_p(32))
    assert _values(kcm._handles([c, C.c_void_p(16), C.c_void_p(None)])) == [32, 16, None]
    assert len(kcm._handles([])) == 0
    c.handle = None


def test_handles_follow_a_chain_whose_handle_changes(monkeypatch):
    # a chain in host memory whose handle the library never sees
    pytest.importorskip("torch")
    monkeypatch.setattr(kcm, "kcm_build_chain", lambda *a: C.c_void_p(32))
    monkeypatch.setattr(kcm, "kcm_chain_info", lambda h: (20, 4, 250, kcm.KCM_FP64))
    c = kcm.Chain(synth.sequence(2, 1), synth.residue_types(), device="cpu")
    assert _values(kcm._handles([c])) == [32]
    c.handle = C.c_void_p(48)
    assert _values(kcm._handles([c])) == [48]
    c.handle = None  # released by its owner
    with pytest.raises(AttributeError):
        kcm._handles([c])
