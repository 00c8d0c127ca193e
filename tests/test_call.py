"""The CPython function of the decode step's call: what it hands to the entry point, what it refuses, and the call without it (no GPU needed)."""
import ctypes as C
import os
import sys

import numpy as np
import pytest
import torch

from paper_2510_13797_amd import bc


def test_native_call_hands_over_addresses_and_numbers():
    bc.load()
    seen = []
    vp = C.c_void_p
    entry = C.CFUNCTYPE(C.c_int32, *[vp] * 10, C.c_size_t, vp)(lambda *a: seen.append(a) or 5)
    at = C.cast(entry, vp).value
    shape, cache = bc.bc_shape(2, 4, 1, 64, bc.BC_BF16, 0.125), bc.bc_cache()
    t = [torch.zeros(3 + i) for i in range(7)]
    args = [at, shape, cache, *t[:4], None, t[4], t[5], t[6], 1 << 40, 7]
    assert bc._call(*args) == 5
    assert [x or 0 for x in seen[0]] == [C.addressof(shape), C.addressof(cache), *(x.data_ptr() for x in t[:4]), 0,
                                         *(x.data_ptr() for x in t[4:]), 1 << 40, 7]
    for i, bad in ((0, None), (0, 0), (1, 3), (2, None), (3, 4), (11, -1), (11, "8"), (12, None)):
        with pytest.raises((TypeError, ValueError, AttributeError, OverflowError, BufferError)):
            bc._call(*[bad if j == i else x for j, x in enumerate(args)])
    with pytest.raises(TypeError):
        bc._call(*args[:-1])
    assert len(seen) == 1


def _runtime(ws_bytes=40):
    rt = bc.Runtime.__new__(bc.Runtime)
    rt.torch, rt.device, rt.dtype, rt.ws_bytes = torch, torch.device("cpu"), "bf16", ws_bytes
    one = torch.zeros(64, dtype=torch.int32).data_ptr()
    rt.shape = bc.bc_shape(2, 4, 1, 64, bc.BC_BF16, 0.125)
    rt.cache = bc.bc_cache(*[one] * 9, 32, None, 0, 0, 0, 0)
    rt.out, rt.ws = torch.empty(2, 4, 64), torch.empty(64, dtype=torch.uint8)
    k, v, bk, bv = (torch.zeros(2, 1, 64, dtype=torch.bfloat16) for _ in range(4))
    return rt, k, v, torch.zeros(2, 4, 64, dtype=torch.bfloat16), bk, bv


def test_decode_step_by_the_native_call(monkeypatch):
    # what Runtime.decode_step hands over where the module is there
    bc.load()
    assert bc._lib is bc._call_lib
    seen = []
    vp = C.c_void_p
    entry = C.CFUNCTYPE(C.c_int32, *[vp] * 10, C.c_size_t, vp)(lambda *a: seen.append([x or 0 for x in a]) or 0)
    monkeypatch.setattr(bc, "_decode_step_at", C.cast(entry, vp).value)
    monkeypatch.setattr(bc, "_stream_ptr", lambda: 7)
    rt, k, v, q, bk, bv = _runtime()
    out, active = torch.empty(2, 4, 64), torch.ones(2, dtype=torch.uint8)
    at = lambda t: 0 if t is None else t.data_ptr()
    for b in ((None, None), (bk, bv)):
        for a in (None, active):
            for o in (None, out):
                seen.clear()
                want = rt.out if o is None else o
                assert rt.decode_step(k, v, q, *b, a, o) is want
                assert seen == [[C.addressof(rt.shape), C.addressof(rt.cache), at(k), at(v), at(q), at(want), at(b[0]), at(b[1]), at(a), at(rt.ws), 40, 7]]
    seen.clear()
    rt.decode_step(np.zeros((2, 1, 64), np.float32), v, q, None, None, np.ones(2))
    assert seen[0][3:5] == [at(v), at(q)] and seen[0][2] and seen[0][8]
    failing = C.CFUNCTYPE(C.c_int32, *[vp] * 10, C.c_size_t, vp)(lambda *a: bc.BC_ERR_ARG)
    monkeypatch.setattr(bc, "_decode_step_at", C.cast(failing, vp).value)
    with pytest.raises(bc.BcError):
        rt.decode_step(k, v, q)


def test_library_loads_without_the_native_call(monkeypatch):
    # no module for this interpreter: the library loads as before, and a decode step reaches its checks through ctypes
    import paper_2510_13797_amd as package
    monkeypatch.setattr(bc, "_stream_ptr", lambda: 0)
    errors = []
    for there in (True, False):
        with monkeypatch.context() as m:
            if not there:
                bc.load()
                for name in ("_lib", "_call", "_call_lib", "_decode_step_at"):
                    m.setattr(bc, name, None)
                m.delattr(package, "_bc_call", raising=False)
                m.setitem(sys.modules, "paper_2510_13797_amd._bc_call", None)
            assert bc.load() is bc._lib and (bc._call is not None) == there and (bc._call_lib is bc._lib) == there
            assert bc.bc_version() > 0 and bc._lib.bc_prefill_attn.restype is C.c_int32
            rt, k, v, q, bk, bv = _runtime(ws_bytes=16)
            with pytest.raises(bc.BcError) as e:
                rt.decode_step(k, v, q, bk, bv)
            errors.append(str(e.value))
    assert errors[0] == errors[1] and str(bc.BC_ERR_WORKSPACE) in errors[0]


def test_build_without_a_compiler_or_headers_leaves_no_old_module(monkeypatch, tmp_path, capsys):
    import __graft_entry__ as G
    lib = tmp_path / "_bc_call.so"
    monkeypatch.setattr(G, "CALL_LIB", str(lib))
    for name, value in (("which", lambda *a: None), ("exists", lambda p, real=os.path.exists: not p.endswith("Python.h") and real(p))):
        lib.write_bytes(b"old")
        with monkeypatch.context() as m:
            m.setattr(G.shutil if name == "which" else G.os.path, name, value)
            assert G.build_call_module() is False
        assert not lib.exists() and "ctypes" in capsys.readouterr().out
