// Calls of the C ABI from Python without ctypes: the entry points that a decoder calls once per step.
//
// A step takes 3 to 5 us on the GPU, and marshalling its ten arguments through ctypes took about 2.2 us of host time
// (a Python-level conversion per device buffer, then ctypes' own) on top of the launch, so the calls were bound by the
// host.  Here the arguments such a caller passes are converted directly: device buffers as None, an int address or
// anything whose data_ptr() is an int, numbers as int and float; the interpreter lock is released during the call, as
// ctypes does.  (0.8 us a call instead of 2.2; greedy steps back to back, B = 32, V = 1024: 5.1 -> 4.0 us.)  A call with
// an argument of any other kind -- numpy scalars, ctypes objects, something wrong -- goes to the ctypes form of the entry
// point as it is, so both accept and refuse the same.  The functions are bound by address to the library that the
// package has loaded, and return its status code.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <tuple>
#include <utility>

#include "pb.h"

namespace {

PyObject* g_data_ptr = nullptr;  // interned method name

// The conversions: false (with or without a Python error set) for an argument that is not of the plain kind.
bool get(PyObject* o, unsigned long long& out) {  // (bits of an int of any size, as ctypes takes them)
  if (!PyLong_Check(o)) return false;
  out = PyLong_AsUnsignedLongLongMask(o);
  return !(out == ~0ull && PyErr_Occurred());
}
template <typename T>
bool get(PyObject* o, T*& out) {
  unsigned long long bits = 0;
  if (o != Py_None && !get(o, bits)) {
    if (PyLong_Check(o)) return false;
    PyObject* r = PyObject_CallMethodNoArgs(o, g_data_ptr);
    const bool ok = r && get(r, bits);
    Py_XDECREF(r);
    if (!ok) return false;
  }
  out = reinterpret_cast<T*>(static_cast<uintptr_t>(bits));
  return true;
}
bool get(PyObject* o, int32_t& out) {
  unsigned long long bits = 0;
  const bool ok = get(o, bits);
  out = static_cast<int32_t>(bits);
  return ok;
}
bool get(PyObject* o, int64_t& out) {
  unsigned long long bits = 0;
  const bool ok = get(o, bits);
  out = static_cast<int64_t>(bits);
  return ok;
}
bool get(PyObject* o, float& out) {
  if (!PyFloat_Check(o) && !PyLong_Check(o)) return false;
  const double d = PyFloat_AsDouble(o);
  out = static_cast<float>(d);
  return !(d == -1.0 && PyErr_Occurred());
}

template <int ID, typename... A>
struct Entry {
  static inline int (*fn)(A...) = nullptr;
  static inline PyObject* other = nullptr;  // the ctypes form
  template <std::size_t... I>
  static bool unpack(PyObject* const* args, std::tuple<A...>& v, std::index_sequence<I...>) {
    return (get(args[I], std::get<I>(v)) && ...);
  }
  static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (!fn) {
      PyErr_SetString(PyExc_RuntimeError, "the entry point is not bound");
      return nullptr;
    }
    std::tuple<A...> v;
    if (n != static_cast<Py_ssize_t>(sizeof...(A)) || !unpack(args, v, std::index_sequence_for<A...>{})) {
      PyErr_Clear();
      return PyObject_Vectorcall(other, args, static_cast<std::size_t>(n), nullptr);
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = std::apply(fn, v);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  }
};
template <int ID, typename... A>
Entry<ID, A...> entry_of(int (*)(A...));

#define PB_ENTRIES(X)                                                                                          \
  X(0, pb_score) X(1, pb_fuse_step) X(2, pb_fuse_frames) X(3, pb_fuse_step_select) X(4, pb_fuse_frames_select) \
  X(5, pb_fuse_frames_ws) X(6, pb_fuse_frames_static) X(7, pb_fuse_step_beam) X(8, pb_score_forest)            \
  X(9, pb_fuse_step_forest) X(10, pb_fuse_frames_forest) X(11, pb_fuse_step_beam_forest)
#define PB_ENTRY(id, name) decltype(entry_of<id>(&name))

// bind(name, address, other): binds an entry point and its ctypes form.
PyObject* bind(PyObject*, PyObject* args) {
  const char* name = nullptr;
  unsigned long long address = 0;
  PyObject* other = nullptr;
  if (!PyArg_ParseTuple(args, "sKO", &name, &address, &other)) return nullptr;
#define PB_BIND(id, f)                                                                             \
  if (PyUnicode_CompareWithASCIIString(PyTuple_GET_ITEM(args, 0), #f) == 0) {                      \
    PB_ENTRY(id, f)::fn = reinterpret_cast<decltype(&f)>(static_cast<uintptr_t>(address));         \
    Py_INCREF(other);                                                                              \
    Py_XSETREF(PB_ENTRY(id, f)::other, other);                                                     \
    Py_RETURN_NONE;                                                                                \
  }
  PB_ENTRIES(PB_BIND)
#undef PB_BIND
  PyErr_Format(PyExc_ValueError, "no entry point %s", name);
  return nullptr;
}

PyMethodDef g_methods[] = {
#define PB_METHOD(id, f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&PB_ENTRY(id, f)::call)), METH_FASTCALL, nullptr},
    PB_ENTRIES(PB_METHOD)
#undef PB_METHOD
    {"bind", bind, METH_VARARGS, "bind(name, address, other): binds an entry point of the loaded library."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_pbcall", "Entry points of libpb.so by address.", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pbcall(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  return g_data_ptr ? PyModule_Create(&g_module) : nullptr;
}
