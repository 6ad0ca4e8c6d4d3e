"""The C-ABI library loads and exports every symbol include/hack.h declares (no compute calls)."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2504_09261_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "hack.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(hack_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    lib = binding.load_library()
    names = _declared()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None
    raw = ctypes.CDLL(binding.LIB_PATH)
    for n in names:
        assert hasattr(raw, n), n


def test_status_strings_and_null_handling():
    lib = binding.load_library()
    assert lib.hack_strerror(0) == b"ok"
    assert lib.hack_strerror(-1) == b"invalid argument"
    assert lib.hack_strerror(-2) == b"capacity exceeded"
    assert lib.hack_last_error(None) == b"NULL context"
    # argument validation that needs no device: NULL config / unsupported head_dim
    ctx = ctypes.c_void_p()
    assert lib.hack_create(ctypes.byref(ctx), None) == -1
    cfg = binding.hack_config(0, 16, 96, 0, 16, 128, 16, 32)
    assert lib.hack_create(ctypes.byref(ctx), ctypes.byref(cfg)) == -1 and not ctx.value
    cfg = binding.hack_config(0, 16, 64, 0, 16, 128, 16, 33)
    assert lib.hack_create(ctypes.byref(ctx), ctypes.byref(cfg)) == -1
    rows = ctypes.c_int64()
    cap = (ctypes.c_int32 * 3)(5, 8, 9)
    assert lib.hack_kvcache_rows_required(3, cap, ctypes.byref(rows)) == 0 and rows.value == 2 * (8 + 8 + 16)
    cap[1] = 0
    assert lib.hack_kvcache_rows_required(3, cap, ctypes.byref(rows)) == -1
    assert lib.hack_kvcache_step_form(None) == 0
    assert lib.hack_score_item_keys(None, 1, cap) == -1


def test_host_arrays_are_typed_pointers():
    """hack_cache holds and hands out typed pointers, and the calls refuse pointers to another type."""
    lib = binding.load_library()
    off, length = (ctypes.c_int64 * 2)(0, 24), (ctypes.c_int32 * 2)(17, 9)
    c = binding.hack_cache(None, None, None, 40, off, ctypes.cast(length, ctypes.POINTER(ctypes.c_int32)))
    assert c.off[1] == 24 and c.len[0] == 17 and c.rows == 40
    rows = ctypes.c_int64()
    for wrong in ((ctypes.c_float * 2)(1, 1), (ctypes.c_int64 * 2)(1, 1), 4096):
        with pytest.raises(ctypes.ArgumentError):
            lib.hack_kvcache_rows_required(2, wrong, ctypes.byref(rows))
    # the library's own arrays, read-only and empty ones among them
    a = np.array([5, 8, 9], np.int32)
    for x in (a, np.frombuffer(a.tobytes(), np.int32)):
        assert lib.hack_kvcache_rows_required(3, binding._p(x, ctypes.c_int32), ctypes.byref(rows)) == 0 and rows.value == 64
    assert lib.hack_kvcache_rows_required(0, binding._p(a[:0], ctypes.c_int32), ctypes.byref(rows)) == -1
    cache = object.__new__(binding.Cache)
    cache.k = cache.v = cache.pos = None
    cache.rows, cache.off, cache.len = 32, np.array([0, 16], np.int64), np.array([3, 4], np.int32)
    st = cache.struct()
    assert isinstance(st, binding.hack_cache) and [st.off[1], st.len[0], st.len[1], st.rows] == [16, 3, 4, 32]
