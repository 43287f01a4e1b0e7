// Python calls of the C ABI's per-step functions (CPython extension
// `_pycall`).
//
// A decode step of a small batch takes the GPU 3-5 us, and marshalling its 14
// to 24 arguments in Python and ctypes took 2.6 us of host time per call, which
// bounded such steps.  Each function here converts its arguments natively and
// calls the library's function of the same name through the address that
// bind() was given (so there is one copy of the library in the process),
// without the interpreter lock.  Pointers are None, integers, or objects with
// a data_ptr() method (torch tensors); the result is the status code.  A call
// with an argument that does not convert goes to the ctypes call that bind() was
// given with the address, which accepts or refuses it as ctypes does.
// Measured per call on one host: 2.6 -> 0.9 us.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "paged_attn.h"

#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

namespace {

PyObject* g_data_ptr = nullptr;   // the interned string "data_ptr"

bool as_pointer(PyObject* o, uintptr_t* out) {
  if (o == Py_None) {
    *out = 0;
    return true;
  }
  PyObject* value = nullptr;
  if (PyLong_CheckExact(o)) {
    value = o;
    Py_INCREF(value);
  } else {
    PyObject* method = PyObject_GetAttr(o, g_data_ptr);
    if (method) {
      value = PyObject_CallNoArgs(method);
      Py_DECREF(method);
    } else if (PyErr_ExceptionMatches(PyExc_AttributeError)) {
      PyErr_Clear();
      value = PyNumber_Long(o);
    }
    if (!value) return false;
  }
  const unsigned long long x = PyLong_AsUnsignedLongLongMask(value);
  Py_DECREF(value);
  if (x == (unsigned long long)-1 && PyErr_Occurred()) return false;
  *out = (uintptr_t)x;
  return true;
}

template <typename T>
bool convert(PyObject* o, T* out) {
  if constexpr (std::is_pointer_v<T>) {
    uintptr_t x = 0;
    if (!as_pointer(o, &x)) return false;
    *out = reinterpret_cast<T>(x);
  } else if constexpr (std::is_floating_point_v<T>) {
    const double x = PyFloat_AsDouble(o);
    if (x == -1.0 && PyErr_Occurred()) return false;
    *out = (T)x;
  } else {
    const unsigned long long x = PyLong_AsUnsignedLongLongMask(o);
    if (x == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *out = (T)x;
  }
  return true;
}

template <int ID, typename F>
struct Call;
template <int ID, typename... A>
struct Call<ID, int (*)(A...)> {
  inline static void* address = nullptr;
  inline static PyObject* plain = nullptr;   // the same call through ctypes (owned)

  template <size_t... I>
  static PyObject* run(PyObject* const* args, std::index_sequence<I...>) {
    std::tuple<A...> v{};
    if (!(convert(args[I], &std::get<I>(v)) && ...)) {
      if (!PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;
      PyErr_Clear();
      return PyObject_Vectorcall(plain, args, sizeof...(A), nullptr);
    }
    int rc = 0;
    Py_BEGIN_ALLOW_THREADS
    rc = reinterpret_cast<int (*)(A...)>(address)(std::get<I>(v)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  }
  static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != (Py_ssize_t)sizeof...(A))
      return PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", (int)sizeof...(A), n);
    if (!address) return PyErr_Format(PyExc_RuntimeError, "bind() has not been called");
    return run(args, std::index_sequence_for<A...>{});
  }
};

struct Entry {
  const char* name;
  PyObject* (*call)(PyObject*, PyObject* const*, Py_ssize_t);
  void** address;
  PyObject** plain;
};
#define PA_ENTRY(id, name)                                                                            \
  {#name, &Call<id, decltype(&name)>::call, &Call<id, decltype(&name)>::address, &Call<id, decltype(&name)>::plain}
const Entry kEntries[] = {
    PA_ENTRY(0, paged_attn_decode),
    PA_ENTRY(1, paged_attn_decode_scheduled),
    PA_ENTRY(2, paged_attn_reduce),
    PA_ENTRY(3, paged_attn_decode_cascade),
    PA_ENTRY(4, paged_attn_decode_cascade_scheduled),
    PA_ENTRY(5, paged_attn_decode_cascade_groups),
    PA_ENTRY(6, paged_attn_reduce_cascade),
    PA_ENTRY(7, paged_attn_reduce_cascade_groups),
    PA_ENTRY(8, paged_attn_append_kv),
    PA_ENTRY(9, paged_attn_decode_append),
    PA_ENTRY(10, paged_attn_decode_cascade_append),
    PA_ENTRY(11, paged_attn_decode_noalloc),
    PA_ENTRY(12, paged_attn_extend),
};
constexpr int kNumEntries = sizeof kEntries / sizeof kEntries[0];

// bind({name: (address, ctypes call)}): every function above must be given.
PyObject* bind(PyObject*, PyObject* calls) {
  if (!PyDict_Check(calls)) return PyErr_Format(PyExc_TypeError, "bind() takes a dict");
  for (const Entry& e : kEntries) {
    PyObject* x = PyDict_GetItemString(calls, e.name);
    if (!x) return PyErr_Format(PyExc_KeyError, "%s", e.name);
    PyObject *address = nullptr, *plain = nullptr;
    if (!PyArg_ParseTuple(x, "OO", &address, &plain)) return nullptr;
    void* p = PyLong_AsVoidPtr(address);
    if (!p) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "%s is NULL", e.name);
    if (!PyCallable_Check(plain)) return PyErr_Format(PyExc_TypeError, "%s is not callable", e.name);
    Py_INCREF(plain);
    Py_XSETREF(*e.plain, plain);
    *e.address = p;
  }
  Py_RETURN_NONE;
}

PyMethodDef g_methods[kNumEntries + 2];
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) {
  for (int i = 0; i < kNumEntries; ++i)
    g_methods[i] = {kEntries[i].name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(kEntries[i].call)),
                    METH_FASTCALL, nullptr};
  g_methods[kNumEntries] = {"bind", bind, METH_O, nullptr};
  g_methods[kNumEntries + 1] = {nullptr, nullptr, 0, nullptr};
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  PyObject* m = g_data_ptr ? PyModule_Create(&g_module) : nullptr;
  if (!m) return nullptr;
  PyObject* names = PyTuple_New(kNumEntries);
  for (int i = 0; names && i < kNumEntries; ++i)
    PyTuple_SET_ITEM(names, i, PyUnicode_FromString(kEntries[i].name));
  if (!names || PyModule_AddObject(m, "NAMES", names) < 0) {
    Py_XDECREF(names);
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
