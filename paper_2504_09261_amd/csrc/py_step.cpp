// CPython entry to hack_step / hack_step_final for binding.py: reads the arguments of one step out of torch tensors and host
// arrays and calls the C function.  Issuing the first scales of an image takes longer than running them, and of
// 6.8 us a step 4.8 went into building 17 ctypes arguments; here it is about one.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

namespace {

typedef int (*StepFn)(void* ctx, void* cache, int32_t B, int32_t N_k, const void* q, const void* k_new, const void* v_new,
                      const uint8_t* head_type, const int32_t* budget, int32_t n_init, float scale, void* out, int32_t* kept_idx,
                      int64_t idx_stride, void* stream);

PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_shape;

// Address of a device tensor, NULL of None; an exception is set where false is returned.
bool device_address(PyObject* t, void** p) {
  *p = nullptr;
  if (t == Py_None) return true;
  PyObject* cuda = PyObject_GetAttr(t, s_is_cuda);
  if (!cuda) return false;
  int ok = PyObject_IsTrue(cuda);
  Py_DECREF(cuda);
  if (ok == 1) {
    PyObject* c = PyObject_CallMethodNoArgs(t, s_is_contiguous);
    if (!c) return false;
    ok = PyObject_IsTrue(c);
    Py_DECREF(c);
  }
  if (ok < 0) return false;
  if (!ok) {
    PyErr_SetString(PyExc_AssertionError, "device tensors must be contiguous CUDA/HIP tensors");
    return false;
  }
  PyObject* a = PyObject_CallMethodNoArgs(t, s_data_ptr);
  if (!a) return false;
  *p = PyLong_AsVoidPtr(a);
  Py_DECREF(a);
  return !PyErr_Occurred();
}

// As ctypes converts an int32 argument: higher bits are dropped.
bool int32_arg(PyObject* o, int32_t* v) {
  *v = (int32_t)PyLong_AsUnsignedLongMask(o);
  return !PyErr_Occurred();
}

// The elements of a contiguous host array of the given struct-module type code; false, without an exception, for any other object.
bool host_array(PyObject* o, char code, Py_buffer* b) {
  if (PyObject_GetBuffer(o, b, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
    PyErr_Clear();
    return false;
  }
  if (b->format && b->format[0] == code && b->format[1] == 0) return true;
  PyBuffer_Release(b);
  return false;
}

// step(fn, ctx, cache, q, k_new, v_new, head_type, budget, n_init, scale, out, kept_idx, idx_stride, stream) -> status.
// fn, ctx, cache, stream: addresses.  Returns None, having called nothing, unless head_type and budget are contiguous arrays of uint8
// and int32 (the caller converts them then).
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 14) {
    PyErr_SetString(PyExc_TypeError, "step takes 14 arguments");
    return nullptr;
  }
  auto address = [&](int i) { return a[i] == Py_None ? nullptr : PyLong_AsVoidPtr(a[i]); };
  void *fn = address(0), *ctx = address(1), *cache = address(2), *stream = address(13);
  int32_t n_init, B, N_k;
  const double scale = PyFloat_AsDouble(a[9]);
  const long long stride = PyLong_AsLongLong(a[12]);
  if (PyErr_Occurred() || !int32_arg(a[8], &n_init)) return nullptr;
  PyObject* shape = PyObject_GetAttr(a[3], s_shape);
  if (!shape) return nullptr;
  if (!PyTuple_Check(shape) || PyTuple_GET_SIZE(shape) != 4) {
    Py_DECREF(shape);
    PyErr_SetString(PyExc_ValueError, "q must have four dimensions");
    return nullptr;
  }
  const bool sized = int32_arg(PyTuple_GET_ITEM(shape, 0), &B) && int32_arg(PyTuple_GET_ITEM(shape, 2), &N_k);
  Py_DECREF(shape);
  if (!sized) return nullptr;
  void *q, *k, *v, *out, *kept;
  if (!device_address(a[3], &q) || !device_address(a[4], &k) || !device_address(a[5], &v) || !device_address(a[10], &out) ||
      !device_address(a[11], &kept))
    return nullptr;
  Py_buffer types, budget;
  if (!host_array(a[6], 'B', &types)) Py_RETURN_NONE;
  if (!host_array(a[7], 'i', &budget)) {
    PyBuffer_Release(&types);
    Py_RETURN_NONE;
  }
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = reinterpret_cast<StepFn>(fn)(ctx, cache, B, N_k, q, k, v, static_cast<const uint8_t*>(types.buf),
                                        static_cast<const int32_t*>(budget.buf), n_init, (float)scale, out, static_cast<int32_t*>(kept),
                                        stride, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&types);
  PyBuffer_Release(&budget);
  return PyLong_FromLong(status);
}

PyMethodDef methods[] = {{"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(step)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_step_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__step_call() {
  s_is_cuda = PyUnicode_InternFromString("is_cuda");
  s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_shape = PyUnicode_InternFromString("shape");
  if (!s_is_cuda || !s_is_contiguous || !s_data_ptr || !s_shape) return nullptr;
  return PyModule_Create(&module);
}
