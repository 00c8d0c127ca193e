// The Python decode step's call of the C ABI, as a CPython function: addresses of tensors and structures to the entry point without a Python
// frame or a ctypes conversion for each.  What it gives is host time: the conversions were 2.1 us of a call of 6.7, now 0.9.  (A pass of 16 small steps, called one by
// one, 98 to 109 us, differs from run to run by more than that.)  The entry point's address comes with every call: nothing is kept here.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>
#include <cstdint>

namespace {

using DecodeStep = int32_t (*)(const void*, const void*, const void*, const void*, const void*, float*, const void*, const void*,
                               const uint8_t*, void*, size_t, void*);

PyObject* data_ptr_name;

// Address of a tensor (None: null).  False with a Python error set.
bool tensor_address(PyObject* t, void** at) {
  *at = nullptr;
  if (t == Py_None) return true;
  PyObject* n = PyObject_CallMethodNoArgs(t, data_ptr_name);
  if (n == nullptr) return false;
  *at = PyLong_AsVoidPtr(n);
  Py_DECREF(n);
  return *at != nullptr || PyErr_Occurred() == nullptr;
}

// decode_step(entry point, shape, cache, k, v, q, out, beacon_k, beacon_v, active, workspace, workspace_bytes, stream) -> status
// shape, cache: ctypes structures; k ... workspace: tensors or None; the rest: numbers.
PyObject* decode_step(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 13) return PyErr_Format(PyExc_TypeError, "decode_step takes 13 arguments (%zd given)", n);
  const DecodeStep call = reinterpret_cast<DecodeStep>(PyLong_AsVoidPtr(args[0]));
  if (call == nullptr) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "decode_step: no entry point");
    return nullptr;
  }
  const size_t bytes = PyLong_AsSize_t(args[11]);
  if (bytes == static_cast<size_t>(-1) && PyErr_Occurred()) return nullptr;
  void* stream = PyLong_AsVoidPtr(args[12]);
  if (stream == nullptr && PyErr_Occurred()) return nullptr;
  void* at[8];
  for (int i = 0; i < 8; ++i)
    if (!tensor_address(args[3 + i], &at[i])) return nullptr;
  Py_buffer shape, cache;
  if (PyObject_GetBuffer(args[1], &shape, PyBUF_SIMPLE) != 0) return nullptr;
  if (PyObject_GetBuffer(args[2], &cache, PyBUF_SIMPLE) != 0) {
    PyBuffer_Release(&shape);
    return nullptr;
  }
  int32_t status;
  Py_BEGIN_ALLOW_THREADS      // (as ctypes does)
  status = call(shape.buf, cache.buf, at[0], at[1], at[2], static_cast<float*>(at[3]), at[4], at[5], static_cast<const uint8_t*>(at[6]), at[7],
                bytes, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&cache);
  PyBuffer_Release(&shape);
  return PyLong_FromLong(status);
}

PyMethodDef methods[] = {
    {"decode_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_step)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bc_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bc_call() {
  data_ptr_name = PyUnicode_InternFromString("data_ptr");
  return data_ptr_name == nullptr ? nullptr : PyModule_Create(&module);
}
