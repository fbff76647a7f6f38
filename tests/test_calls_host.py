"""The native module behind the per-step calls of the binding: which
arguments it takes itself, that any other form reaches the ctypes function of
the same name unchanged, and that errors are the same."""
import ctypes
import inspect

import numpy as np
import pytest
import torch

from paper_2607_07388_amd import _calls, tfe

SIG = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32,
                       ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p)


class Stream:
    cuda_stream = 77


@pytest.fixture
def recorder():
    """tfe_head_topk bound to functions that record what arrives natively and
    what is handed on; the real binding afterwards."""
    native, handed = [], []

    @SIG
    def fn(*a):
        native.append(a)
        return -1 if a[2] == 13 else 0

    def slow(*a, **k):
        handed.append((a, k))
        return "slow"

    def check(st):
        raise tfe.TfeError(st, "recorded")

    addr = ctypes.cast(fn, ctypes.c_void_p).value
    _calls.bind(check, {n: (slow, addr) for n in (
        "tfe_lookup_inject", "tfe_lookup_inject_multi", "tfe_prefetch", "tfe_prefetch_scored",
        "tfe_head_topk")})
    yield native, handed
    tfe._bind_calls()


def test_plain_arguments_arrive_natively(recorder):
    native, handed = recorder
    t = torch.zeros(4)
    assert _calls.tfe_head_topk(5, t, 2, 3, None, 9) == 0
    assert _calls.tfe_head_topk(None, t, -2, 3, t, t[1:], Stream()) == 0
    assert _calls.tfe_head_topk(5, 2 ** 63, 2, 3, 0, 9, 11) == 0
    p = t.data_ptr()
    assert native == [(5, p, 2, 3, None, 9, None), (None, p, -2, 3, p, p + 4, 77),
                      (5, 2 ** 63, 2, 3, None, 9, 11)]
    assert handed == []


@pytest.mark.parametrize("args,kw", [
    ((5, 1, 2, 3, 4), {}),                            # too few
    ((5, 1, 2, 3, 4, 5, 6, 7), {}),                   # too many
    ((5, 1, 2, 3, 4, 5), {"stream": None}),           # keywords
    ((5, np.zeros(3), 2, 3, 4, 5), {}),               # a host array
    ((5, "x", 2, 3, 4, 5), {}),                       # no address
    ((5, 1, np.int64(2), 3, 4, 5), {}),               # not an exact int
    ((5, 1, True, 3, 4, 5), {}),
    ((5, 1, 2 ** 31, 3, 4, 5), {}),                   # beyond int32
    ((5, 1, 2.0, 3, 4, 5), {}),
    ((ctypes.c_void_p(5), 1, 2, 3, 4, 5), {}),
    ((5, 1, 2, 3, 4, 5, "stream"), {}),
])
def test_other_forms_are_handed_on(recorder, args, kw):
    native, handed = recorder
    assert _calls.tfe_head_topk(*args, **kw) == "slow"
    assert native == [] and len(handed) == 1
    assert len(handed[0][0]) == len(args) and handed[0][1] == kw
    assert all(x is y for x, y in zip(handed[0][0], args))


def test_processes_that_build_the_module_together(monkeypatch, tmp_path):
    """Ranks that find no module all build it: one that finishes while another
    is still compiling leaves that one's output alone."""
    import subprocess

    from paper_2607_07388_amd import _build
    monkeypatch.setattr(_build, "CALLS", str(tmp_path / "_calls.so"))
    run = subprocess.run
    pid, depth = _build.os.getpid(), []

    def compile_beside_another(*a, **k):
        r = run(*a, **k)
        if not depth:  # the other process starts later and ends first
            depth.append(1)
            monkeypatch.setattr(_build.os, "getpid", lambda: pid + 1)
            _build.build_calls()
            monkeypatch.setattr(_build.os, "getpid", lambda: pid)
        return r

    monkeypatch.setattr(_build.subprocess, "run", compile_beside_another)
    _build.build_calls()
    assert [p.name for p in tmp_path.iterdir()] == ["_calls.so"]
    ctypes.PyDLL(str(tmp_path / "_calls.so")).PyInit__calls


def test_negative_status_raises(recorder):
    with pytest.raises(tfe.TfeError):
        _calls.tfe_head_topk(5, 1, 13, 3, 4, 5)


def test_library_errors_and_signatures():
    with pytest.raises(tfe.TfeError) as e:
        tfe.tfe_lookup_inject(None, None, 1, 0, 1, None, None, None, None, None, 0, 1.0)
    assert e.value.status == tfe.TFE_ERR_INVALID_ARG and "null table" in str(e.value)
    with pytest.raises(tfe.TfeError):
        tfe.tfe_prefetch_scored(None, None, 1, None, None, 1, 1, 1, side_stream=None)
    with pytest.raises(tfe.TfeError):
        tfe.tfe_lookup_inject_multi(None, None, 1, 0, 1, None, None, None, None, 0, 0, 1)
    with pytest.raises(tfe.TfeError):
        tfe.tfe_prefetch(None, None, 1, None, 1, 1)
    with pytest.raises(tfe.TfeError):
        tfe.tfe_head_topk(None, None, 1, 1, None, None)
    assert list(inspect.signature(tfe.tfe_head_topk).parameters) == [
        "head", "hidden", "B", "K", "top_ids", "top_prob", "stream"]
