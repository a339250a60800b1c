"""The native marshalling of torch tensors (the _marshal extension): the
descriptors it hands to a library call equal the ctypes ones field by field,
and what it does not take it leaves to the general path untouched."""
from __future__ import annotations

import ctypes
import os
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2510_15330_amd import _binding as B

P, T = ctypes.c_void_p, ctypes.POINTER(B.Tensor)
# form -> (tensors before the softmax scale, whether a scale and an output follow, options)
FORMS = {B._APPEND: (6, False, False), B._DECODE: (5, True, False), B._DECODE_OPTS: (5, True, True),
         B._STEP: (7, True, True), B._WRITE: (7, False, False), B._PREFILL: (6, True, False)}
PAGES = {B._APPEND: 2, B._DECODE: 1, B._DECODE_OPTS: 1, B._STEP: 3, B._WRITE: 2, B._PREFILL: 1}


def _recorder(form, rc, seen):
    before, scaled, opts = FORMS[form]
    args = [T] * before + ([ctypes.c_float, T] if scaled else []) + ([P] if opts else []) + [P]

    def record(*a):
        a = list(a)
        seen["stream"] = a.pop() or 0
        if opts:
            seen["opts"] = a.pop()
        if scaled:
            seen["scale"] = a.pop(before)
        seen["tensors"] = [bytes(t.contents) for t in a]
        return rc
    return ctypes.CFUNCTYPE(ctypes.c_int, *args)(record)


def test_host_tensors_and_other_objects_are_left():
    B.library()

    def never(*a):
        raise AssertionError("called")
    fn = ctypes.CFUNCTYPE(ctypes.c_int, *([T] * 6), P)(never)
    addr = ctypes.cast(fn, P).value
    t = torch.zeros(2, 2)
    for ts in ([t] * 6, [None] * 6, [1] * 6):
        assert B._native(addr, B._APPEND, 0, 0.0, 0, None, None, *ts) is None
    with pytest.raises(TypeError):
        B._native(addr, B._APPEND, 0, 0.0, 0, None, None, t)
    with pytest.raises(TypeError):
        B._native(addr, 99, 0, 0.0, 0, None, None, *[t] * 6)


@pytest.mark.parametrize("beside", ["nothing", "no extension"])
def test_library_without_the_extension(tmp_path, beside):
    # the library alone: host calls work, device calls keep the general path
    # and its errors
    B.library()
    lib = str(tmp_path / "libbellman.so")
    shutil.copy(B.library_path(), lib)
    if beside != "nothing":
        (tmp_path / "_marshal.so").write_bytes(b"not a library")
    code = """
import warnings, torch, paper_2510_15330_amd as bl
assert bl.version()
t = torch.zeros(2, 2)
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    for _ in range(2):
        try:
            bl.kv_append(t, t, t, t, t, t)
        except ValueError as e:
            assert "device tensors" in str(e)
        else:
            raise AssertionError("accepted")
assert [x for x in w if "_marshal" in str(x.message)].__len__() == 1
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, env=dict(os.environ, BELLMAN_LIBRARY=lib),
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("form", sorted(FORMS))
def test_descriptors_equal_the_ctypes_ones(form):
    B.library()
    before, scaled, opts = FORMS[form]
    dev = "cuda"
    pool = [torch.zeros(3, 5, 7, dtype=torch.bfloat16, device=dev)[:, 1:4, ::2], torch.zeros(4, 0, 3, device=dev),
            torch.zeros(2, 3, 4, 5, 6, dtype=torch.uint8, device=dev), torch.zeros(9, dtype=torch.int32, device=dev)[3:],
            torch.zeros(4, 4, device=dev).to(torch.float8_e4m3fn).t(), torch.tensor(1.0, device=dev),
            torch.zeros(1, 6, dtype=torch.int32, device=dev).expand(4, 6),
            torch.nn.Parameter(torch.zeros(2, 2, device=dev))]
    n = before + (1 if scaled else 0)
    ks, vs = torch.ones(2, 3, device=dev), torch.ones(2, 3, device=dev)
    ev = torch.cuda.Stream()
    for shift in range(len(pool)):
        ts = [pool[(i + shift) % len(pool)] for i in range(n)]
        seen = {}
        fn = _recorder(form, -3, seen)
        with torch.cuda.stream(ev):
            rc = B._native(ctypes.cast(fn, P).value, form, None, 0.1, 77 if opts else 0, ks, vs, *ts)
        assert rc == -3
        want = [bytes(B.desc(t, ks if i == PAGES[form] else vs if i == PAGES[form] + 1 else None))
                for i, t in enumerate(ts)]
        assert seen["tensors"] == want
        assert seen["stream"] == ev.cuda_stream
        if scaled:
            assert seen["scale"] == ctypes.c_float(0.1).value
        if opts:
            assert seen["opts"] == 77
    # what it leaves: types the library has no code for, non-contiguous scales
    seen = {}
    fn = _recorder(form, 0, seen)
    addr = ctypes.cast(fn, P).value
    ok = [pool[3]] * n
    assert B._native(addr, form, 0, 0.1, 0, ks.t(), vs, *ok) is None
    assert B._native(addr, form, 0, 0.1, 0, None, None, *ok[:-1], torch.zeros(2, device=dev, dtype=torch.float64)) is None
    assert B._native(addr, form, 0, 0.1, 0, None, None, *ok[:-1], torch.zeros((1,) * 6, device=dev)) is None
    assert not seen
