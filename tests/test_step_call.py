"""The CPython entry to hack_step passes on what ctypes would, checked on the host against a stand-in for the C function."""
import ctypes as C

import numpy as np
import pytest

from paper_2504_09261_amd import binding


class Tensor:
    def __init__(self, ptr, shape=(2, 3, 5, 64), cuda=True, contiguous=True):
        self.ptr, self.shape, self.is_cuda, self.contiguous = ptr, shape, cuda, contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return self.ptr


SEEN = []


@C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_void_p, C.c_int32, C.c_int32, C.c_void_p, C.c_void_p, C.c_void_p, C.POINTER(C.c_uint8),
             C.POINTER(C.c_int32), C.c_int32, C.c_float, C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p)
def stand_in(ctx, cache, B, N_k, q, k, v, types, budget, n_init, scale, out, kept, stride, stream):
    SEEN.append((ctx, cache, B, N_k, q, k, v, types[:3], budget[:6], n_init, scale, out, kept, stride, stream))
    return -4


def call(types=np.array([0, 1, 1], np.uint8), budget=np.arange(6, dtype=np.int32), q=Tensor(2**40), k=Tensor(17), out=Tensor(19),
         kept=None, n_init=5, scale=0.125, ctx=2**47 + 8):
    binding.load_library()
    fn = C.cast(stand_in, C.c_void_p).value
    return binding._step_call(fn, ctx, 33, q, k, Tensor(18), types, budget, n_init, scale, out, kept, 2**33, 0)


def test_arguments_arrive_as_given():
    SEEN.clear()
    assert call() == -4
    assert SEEN.pop() == (2**47 + 8, 33, 2, 5, 2**40, 17, 18, [0, 1, 1], [0, 1, 2, 3, 4, 5], 5, 0.125, 19, None, 2**33, None)
    assert call(kept=Tensor(21), n_init=np.int64(7), scale=1, out=None, ctx=None) == -4     # NULL is the library's to refuse
    assert SEEN.pop() == (None, 33, 2, 5, 2**40, 17, 18, [0, 1, 1], [0, 1, 2, 3, 4, 5], 7, 1.0, None, 21, 2**33, None)
    budget = np.arange(6, dtype=np.int32)
    budget.flags.writeable = False
    assert call(budget=budget) == -4 and SEEN.pop()[8] == [0, 1, 2, 3, 4, 5]


@pytest.mark.parametrize("kw", [
    dict(types=[0, 1, 1]), dict(types=np.array([0, 1, 1])), dict(types=np.array([False, True, True])), dict(budget=list(range(6))),
    dict(budget=np.arange(6)), dict(budget=np.arange(6, dtype=np.float32)), dict(budget=np.arange(12, dtype=np.int32)[::2]),
    dict(budget=np.arange(6, dtype=np.uint32)), dict(types=np.array([0, 1, 1], np.int8)),
])
def test_other_host_arrays_are_left_to_the_caller_to_convert(kw):
    SEEN.clear()
    assert call(**kw) is None and not SEEN


def test_tensors_that_are_refused():
    SEEN.clear()
    for bad in (Tensor(1, cuda=False), Tensor(1, contiguous=False)):
        for name in ("k", "out", "kept"):
            with pytest.raises(AssertionError, match="contiguous CUDA/HIP"):
                call(**{name: bad})
    with pytest.raises(ValueError):
        call(q=Tensor(1, shape=(2, 3, 5)))
    with pytest.raises(AttributeError):
        call(q=None)
    with pytest.raises(TypeError):
        call(scale="x")
    assert not SEEN
