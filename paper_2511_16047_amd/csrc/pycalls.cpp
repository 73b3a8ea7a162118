// The two calls of the path that a model makes for every layer and scale, amskv_append_scale and amskv_attend, as a
// CPython extension: argument marshalling only, for binding.py (all other calls go through ctypes).  One image through a
// 16-layer stack is 320 of these calls and 160 short launches, and with ctypes and torch's public stream lookup (about
// 3.6 us a call by itself) the host side took longer than the kernels: 1908 us a pass, 719 with this (launches included).
// The library stays behind its C ABI: bind() is given the addresses of the two functions.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <cstdint>

namespace {

typedef int32_t (*Append)(void*, int32_t, int32_t, const void*, const void*, void*);
typedef int32_t (*Attend)(void*, int32_t, int32_t, const void*, void*, void*);
Append append_fn = nullptr;
Attend attend_fn = nullptr;
PyObject* lookup = nullptr;  // asked once, when a call first leaves the stream to torch: (current device, current stream) functions
PyObject *get_device = nullptr, *get_stream = nullptr;  // its answer; None: there is no device
PyObject *name_data_ptr = nullptr, *name_cuda_stream = nullptr;

bool integer(PyObject* o, int32_t* out) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) return false;
  *out = (int32_t)v;
  return true;
}

bool address(PyObject* o, void** out) {
  *out = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLongMask(o));
  return *out != reinterpret_cast<void*>(UINTPTR_MAX) || !PyErr_Occurred();
}

// None, a device address, or a tensor
bool tensor(PyObject* o, void** out) {
  *out = nullptr;
  if (o == Py_None) return true;
  if (PyLong_Check(o)) return address(o, out);
  PyObject* p = PyObject_CallMethodNoArgs(o, name_data_ptr);
  if (!p) return false;
  const bool ok = address(p, out);
  Py_DECREF(p);
  return ok;
}

bool find_stream_functions() {
  PyObject* two = PyObject_CallNoArgs(lookup);
  if (!two) return false;
  PyObject *device, *current;
  const bool ok = PyArg_ParseTuple(two, "OO", &device, &current);
  if (ok) {
    Py_XSETREF(get_device, Py_NewRef(device));
    Py_XSETREF(get_stream, Py_NewRef(current));
  }
  Py_DECREF(two);
  return ok;
}

// None (torch's current stream of the current device), a raw handle, or a stream object
bool stream(PyObject* o, void** out) {
  *out = nullptr;
  if (PyLong_Check(o)) return address(o, out);
  PyObject* p;
  if (o == Py_None) {
    if (!get_stream && !find_stream_functions()) return false;
    if (get_stream == Py_None) return true;
    PyObject* dev = PyObject_CallNoArgs(get_device);
    if (!dev) return false;
    p = PyObject_CallOneArg(get_stream, dev);
    Py_DECREF(dev);
  } else {
    p = PyObject_GetAttr(o, name_cuda_stream);
  }
  if (!p) return false;
  const bool ok = address(p, out);
  Py_DECREF(p);
  return ok;
}

// (cache, layer, s, tensor, tensor, stream) -> status
template <typename F>
PyObject* call(F fn, PyObject* const* args, Py_ssize_t n) {
  int32_t layer, s, status;
  void *cache, *a, *b, *st;
  if (n != 6 || !fn) {
    PyErr_SetString(PyExc_TypeError, "(cache, layer, s, tensor, tensor, stream) expected, after bind()");
    return nullptr;
  }
  if (args[0] == Py_None) cache = nullptr;
  else if (!address(args[0], &cache)) return nullptr;
  if (!integer(args[1], &layer) || !integer(args[2], &s) || !tensor(args[3], &a) || !tensor(args[4], &b) || !stream(args[5], &st))
    return nullptr;
  Py_BEGIN_ALLOW_THREADS  // in the token modes a call may wait for a layer's Eq. 3 test
  status = fn(cache, layer, s, a, b, st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

PyObject* append_scale(PyObject*, PyObject* const* args, Py_ssize_t n) { return call(append_fn, args, n); }
PyObject* attend(PyObject*, PyObject* const* args, Py_ssize_t n) { return call(attend_fn, args, n); }

// bind(address of amskv_append_scale, address of amskv_attend, lookup)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3) {
    PyErr_SetString(PyExc_TypeError, "three arguments expected");
    return nullptr;
  }
  void *f, *g;
  if (!address(args[0], &f) || !address(args[1], &g)) return nullptr;
  append_fn = reinterpret_cast<Append>(f);
  attend_fn = reinterpret_cast<Attend>(g);
  Py_XSETREF(lookup, Py_NewRef(args[2]));
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(bind)), METH_FASTCALL, "function addresses and stream lookup"},
    {"append_scale", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(append_scale)), METH_FASTCALL, "amskv_append_scale"},
    {"attend", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(attend)), METH_FASTCALL, "amskv_attend"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycalls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycalls() {
  name_data_ptr = PyUnicode_InternFromString("data_ptr");
  name_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  return name_data_ptr && name_cuda_stream ? PyModule_Create(&module) : nullptr;
}
