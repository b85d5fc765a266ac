"""The argument marshalling of the module _call, and of ctypes where that has not been built, without a GPU: entry points written in
Python are bound in the library's place and record what they are given."""
import ctypes as C
import os
import types

import numpy as np
import pytest
import torch

from paper_2509_15038_amd import binding as B

VP, I32, I64, F64 = C.c_void_p, C.c_int32, C.c_int64, C.c_double
SIGNATURES = {"scores": [VP, VP, VP, I64, VP, VP], "scores_append": [VP, VP, VP, I64, I64, I64, VP, VP, VP], "normalise": [VP, VP, VP, I64, I64, VP, VP],
              "select": [VP, VP, I64, VP, I32, VP, VP, VP], "compact": [VP, VP, VP, I64, VP, VP, VP, VP, VP],
              "compress": [VP, VP, VP, I64, VP, I32, VP, VP, VP, VP, VP, VP], "compress_adaptive": [VP, VP, VP, I64, I32, I32, F64, VP, VP, VP, VP, VP, VP, VP]}


@pytest.fixture(params=["module", "ctypes"])
def calls(request, monkeypatch):
    L = B.lib()
    seen, kept = [], {}

    def entry(name, types):
        def f(*a):
            seen.append((name, [x or 0 if t is VP else x for x, t in zip(a, types)]))
            return -1 if name == "normalise" else 0
        kept[name] = C.CFUNCTYPE(C.c_int, *types)(f)
        return C.cast(kept[name], VP).value

    addresses = [entry(n, t) for n, t in SIGNATURES.items()]
    by_default = lambda s, usual=B._stream: 77 if s is None else usual(s)
    monkeypatch.setattr(B, "_stream", by_default)
    if request.param == "module":
        if not os.path.exists(B.CALL_PATH):
            pytest.skip("not built for this interpreter")
        B._call.bind(*addresses, B._ptr, by_default)
    else:
        monkeypatch.setattr(B, "_call", B._CtypesCalls(types.SimpleNamespace(**{"curdkv_" + n: f for n, f in kept.items()})))
    yield seen
    monkeypatch.undo()
    B._bind_calls(L)


def test_without_the_module(monkeypatch, tmp_path):
    """A build without Python.h, or for another interpreter: the library loads and is called through ctypes."""
    monkeypatch.setattr(B, "CALL_PATH", str(tmp_path / "_call.none.so"))
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_call", None)
    B.lib()
    assert isinstance(B._call, B._CtypesCalls)
    assert B._call.scores(0, None, None, 1, None, 0) == B.ERR_INVALID_ARG      # (no context: refused before anything is launched)
    assert B.curdkv_sketch_host(B.make_config(1, 1, 1, 128, 4, "fp32", 1, 1), 0, 0).shape == (128, 4)


def test_a_build_without_headers(monkeypatch, tmp_path, capsys):
    from paper_2509_15038_amd import build
    monkeypatch.setattr(build, "CALL", str(tmp_path / "_call.so"))
    (tmp_path / "_call.so").write_bytes(b"of an older source")
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    build._build_call_module("hipcc", False)
    assert not (tmp_path / "_call.so").exists() and "ctypes" in capsys.readouterr().out


def test_every_argument_arrives(calls):
    t = [torch.zeros(8) for _ in range(7)]
    p = [x.data_ptr() for x in t]
    budgets, offsets = np.array([1, 2, 3], np.int32), np.array([0, 1, 3, 6], np.int64)
    b, o = budgets.ctypes.data, offsets.ctypes.data
    m = B._call
    assert m.scores(5, t[0], t[1], 9, t[2], None) == 0
    assert m.scores_append(5, t[0], t[1], np.int64(9), 2 ** 33, np.int32(11), t[2], t[3], 123) == 0
    assert m.normalise(5, t[0], t[1], 9, 8, t[2], None) == -1
    assert m.select(5, t[0], 9, budgets, 4, offsets, t[1], None, 3) == 0
    assert m.compact(5, t[0], t[1], 9, t[2], offsets, t[3], t[4], None, 3) == 0
    assert m.compress(5, t[0], t[1], 9, budgets, 4, offsets, None, t[2], t[3], t[4], None, 3) == 0
    assert m.compress_adaptive(5, t[0], t[1], 9, 7, 4, 0.25, t[2], t[3], t[4], t[5], t[6], 1234, None) == 0
    assert calls == [("scores", [5, p[0], p[1], 9, p[2], 77]), ("scores_append", [5, p[0], p[1], 9, 2 ** 33, 11, p[2], p[3], 123]),
                     ("normalise", [5, p[0], p[1], 9, 8, p[2], 77]), ("select", [5, p[0], 9, b, 4, o, p[1], 77]),
                     ("compact", [5, p[0], p[1], 9, p[2], o, p[3], p[4], 77]), ("compress", [5, p[0], p[1], 9, b, 4, o, 0, p[2], p[3], p[4], 77]),
                     ("compress_adaptive", [5, p[0], p[1], 9, 7, 4, 0.25, p[2], p[3], p[4], p[5], p[6], 1234, 77])]


def test_other_kinds_of_buffers_and_numbers(calls):
    a = np.zeros(4, np.float32)
    stream = type("S", (), {"cuda_stream": 4321})()
    B._call.scores(5, a, 2 ** 64 - 16, 2.9, torch.zeros(2)[1:], stream)
    name, got = calls[0]
    assert got[:4] == [5, a.ctypes.data, 2 ** 64 - 16, 2] and got[5] == 4321
    B._call.compress_adaptive(5, a, a, 9, 2 ** 32 + 3, -1, 1, a, a, a, a, a, a, None)      # 32 bits, as C passes them
    assert calls[1][1][4:7] == [3, -1, 1.0]


@pytest.mark.parametrize("budgets,offsets", [(np.zeros(3, np.int64), np.zeros(4, np.int64)), (np.zeros(3, np.int32), np.zeros(4, np.int32)),
                                             (np.zeros(2, np.int32), np.zeros(4, np.int64)), (np.zeros(3, np.int32), np.zeros(3, np.int64)),
                                             (np.zeros(3, np.float32), np.zeros(4, np.int64)), (np.zeros(3, np.uint32), np.zeros(4, np.int64)),
                                             (np.zeros(3, ">i4"), np.zeros(4, np.int64)), (np.zeros(6, np.int32)[::2], np.zeros(4, np.int64)),
                                             (np.zeros(3, np.int32), np.zeros(4, np.int64)[::-1]), (np.zeros((3, 2), np.int32)[:, 0], np.zeros(4, np.int64))])
def test_host_arrays_of_another_kind_are_refused(calls, budgets, offsets):
    with pytest.raises(AssertionError):
        B._call.select(5, None, 9, budgets, 4, offsets, None, None, 3)
    assert not calls


def test_host_arrays_at_any_address(calls):
    """Views that lie at odd addresses, of two dimensions, or of the other name that 64 bits have."""
    budgets = np.frombuffer(b"\0" * 17, np.uint8)[1:].view(np.int32)
    offsets = np.zeros(5, np.dtype([("kind", "i1"), ("at", "i8")]))["at"].copy()
    odd = np.frombuffer(b"\0" * 41, np.uint8)[1:].view(np.int64)
    for b, o in ((budgets, offsets), (budgets, odd), (np.zeros((2, 2), np.int32), np.zeros(5, np.longlong))):
        B._call.select(5, None, 9, b, 4, o, None, None, 4)
        assert calls[-1][1][3] == b.ctypes.data and calls[-1][1][5] == o.ctypes.data


@pytest.mark.parametrize("args", [(5, None, None, "nine", None, 1), (5, None, None, None, None, 1), (5, object(), None, 9, None, 1), (5, None, None, 9, None),
                                  (5, None, None, 9, None, "x")])
def test_nonsense_is_an_error_and_reaches_nothing(calls, args):
    with pytest.raises((TypeError, ValueError, AttributeError)):
        B._call.scores(*args)
    assert not calls
