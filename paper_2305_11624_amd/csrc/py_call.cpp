// CPython extension `_call`: turns the tensors of a block call into pointers and calls the C ABI.  Host code only.
//
// A small block's kernels take a few microseconds each, so a call's own cost on the host is what such a block waits
// for.  Marshalling fourteen tensors through ctypes (a Python function per tensor, a stream object per call) took
// 5-7 us a call; here it takes well under one.
//
//   call(address, desc, groups, tensors..., ws, stream) -> status
//
// `address` is the entry point's address, `desc` a convbn_desc (any object with the buffer protocol), groups None
// means that the entry point takes none; a tensor is None, a device tensor or an int (a raw address); ws is None or a
// device tensor, passed on as pointer and size (NO_WS: the entry point takes none); stream is None (the current
// stream) or a raw handle.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

#include "../../include/convbn.h"

namespace {

constexpr int kMaxPtr = 16;

PyObject* g_no_ws = nullptr;   // the NO_WS marker

// Torch throws where a tensor has no memory of its own or there is no device; the interpreter's C frames let no C++
// exception through, so it becomes a Python error.
template <typename F>
bool guarded(F&& f) {
  try {
    return f();
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  } catch (...) {
    PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
  }
  return false;
}

// Address of a tensor argument; false (with a Python error set) where it is neither None, an int nor a dense device tensor.
bool pointer_of(PyObject* o, void** out) {
  if (o == Py_None) { *out = nullptr; return true; }
  if (THPVariable_Check(o)) return guarded([&] {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
      PyErr_SetString(PyExc_AssertionError, "device, dense tensors only");
      return false;
    }
    *out = t.data_ptr();
    return true;
  });
  if (PyLong_Check(o)) {
    *out = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
  }
  PyErr_Format(PyExc_TypeError, "expected a tensor, an address or None, got %s", Py_TYPE(o)->tp_name);
  return false;
}

bool stream_of(PyObject* o, void** out) {
  if (o == Py_None) return guarded([&] {
    *out = c10::hip::getCurrentHIPStream().stream();
    return true;
  });
  *out = PyLong_AsVoidPtr(o);
  return !PyErr_Occurred();
}

template <typename... A>
int invoke(void* f, A... a) { return reinterpret_cast<int (*)(A...)>(f)(a...); }

// desc [, groups], n pointers [, ws, bytes], stream
#define P4 p[0], p[1], p[2], p[3]
#define P8 P4, p[4], p[5], p[6], p[7]
#define P12 P8, p[8], p[9], p[10], p[11]
template <typename... T>
int dispatch(void* f, int n, void* const* p, bool* known, const void* d, T... tail) {
  switch (n) {
    case 3: return invoke(f, d, p[0], p[1], p[2], tail...);
    case 4: return invoke(f, d, P4, tail...);
    case 8: return invoke(f, d, P8, tail...);
    case 9: return invoke(f, d, P8, p[8], tail...);
    case 11: return invoke(f, d, P8, p[8], p[9], p[10], tail...);
    case 13: return invoke(f, d, P12, p[12], tail...);
  }
  *known = false;
  return 0;
}
template <typename... T>
int dispatch_groups(void* f, int n, void* const* p, bool* known, const void* d, int groups, T... tail) {
  switch (n) {
    case 9: return invoke(f, d, groups, P8, p[8], tail...);
    case 13: return invoke(f, d, groups, P12, p[12], tail...);
  }
  *known = false;
  return 0;
}

PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  const Py_ssize_t n = nargs - 5;   // tensors
  if (n < 1 || n > kMaxPtr) {
    PyErr_SetString(PyExc_TypeError, "call(address, desc, groups, tensors..., ws, stream)");
    return nullptr;
  }
  void* f = PyLong_AsVoidPtr(args[0]);
  const bool has_groups = args[2] != Py_None;
  const long groups = has_groups ? PyLong_AsLong(args[2]) : 0;
  if (PyErr_Occurred()) return nullptr;
  void* p[kMaxPtr];
  for (Py_ssize_t i = 0; i < n; ++i)
    if (!pointer_of(args[3 + i], &p[i])) return nullptr;
  PyObject* ws_o = args[3 + n];
  const bool has_ws = ws_o != g_no_ws;
  void* ws = nullptr;
  size_t ws_bytes = 0;
  if (has_ws) {
    if (!pointer_of(ws_o, &ws)) return nullptr;
    if (THPVariable_Check(ws_o) && !guarded([&] { ws_bytes = THPVariable_Unpack(ws_o).nbytes(); return true; })) return nullptr;
  }
  void* stream = nullptr;
  if (!stream_of(args[4 + n], &stream)) return nullptr;
  Py_buffer d;
  if (PyObject_GetBuffer(args[1], &d, PyBUF_SIMPLE) != 0) return nullptr;
  if (d.len != (Py_ssize_t)sizeof(convbn_desc)) {
    PyBuffer_Release(&d);
    PyErr_SetString(PyExc_TypeError, "expected a convbn_desc");
    return nullptr;
  }
  bool known = true;
  int st = 0;
  Py_BEGIN_ALLOW_THREADS
  if (has_groups) st = dispatch_groups(f, (int)n, p, &known, d.buf, (int)groups, ws, ws_bytes, stream);
  else if (has_ws) st = dispatch(f, (int)n, p, &known, d.buf, ws, ws_bytes, stream);
  else st = dispatch(f, (int)n, p, &known, d.buf, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&d);
  if (!known) {
    PyErr_SetString(PyExc_TypeError, "no entry point takes this number of tensors");
    return nullptr;
  }
  return PyLong_FromLong(st);
}

// pointer(tensor) -> address or None, stream(None or handle) -> handle: for the entry points that take no descriptor.
PyObject* pointer(PyObject*, PyObject* o) {
  void* p = nullptr;
  if (!pointer_of(o, &p)) return nullptr;
  if (!p) Py_RETURN_NONE;
  return PyLong_FromVoidPtr(p);
}
PyObject* stream(PyObject*, PyObject* o) {
  void* p = nullptr;
  if (!stream_of(o, &p)) return nullptr;
  return PyLong_FromVoidPtr(p);
}

PyMethodDef methods[] = {
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL, nullptr},
    {"pointer", pointer, METH_O, nullptr},
    {"stream", stream, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call() {
  PyObject* m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  g_no_ws = PyUnicode_FromString("NO_WS");
  if (!g_no_ws) return nullptr;
  Py_INCREF(g_no_ws);
  if (PyModule_AddObject(m, "NO_WS", g_no_ws) != 0) return nullptr;
  return m;
}
