// The kernel-level entry points as Python calls without ctypes (`_calls`, built beside libcdp.so).
//
// A small layer is a launch of a few microseconds, and converting a dozen arguments through ctypes takes one to two of them.  Here an
// argument is read with one PyLong conversion.  What is accepted is what ctypes accepts for the same prototypes in plain integers: None or 0
// for a null pointer, integers of any size for an int (the low bits, as C would take them).  Anything else makes the call
// return None without doing anything, and the caller goes through ctypes, which converts it or says what is wrong with it.  The interpreter lock
// is released for the call, as ctypes does.
//
// The module is not linked against libcdp.so: `use` is given the addresses of the library that the package loaded.  A library that the
// dynamic linker looks up by path or by name may be another copy's, with its own kernels, scratch memory and last error.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/cdp.h"
#include "../../include/cdp_kernels.h"

namespace {

template <typename T> bool read(PyObject* o, T& v) {
  if constexpr (std::is_pointer_v<T>) {
    if (o == Py_None) {
      v = nullptr;
      return true;
    }
  }
  if (!PyLong_CheckExact(o)) return false;
  const unsigned long long u = PyLong_AsUnsignedLongLongMask(o);
  if constexpr (std::is_pointer_v<T>) v = reinterpret_cast<T>(static_cast<uintptr_t>(u));
  else v = static_cast<T>(u);
  return true;
}

template <typename... A, size_t... I>
PyObject* call(int (*f)(A...), PyObject* const* args, std::index_sequence<I...>) {
  std::tuple<A...> v;
  if (!(read(args[I], std::get<I>(v)) && ...)) Py_RETURN_NONE;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f(std::get<I>(v)...);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}
template <typename... A> PyObject* checked(int (*f)(A...), PyObject* const* args, Py_ssize_t n) {
  if (!f || n != (Py_ssize_t)sizeof...(A)) Py_RETURN_NONE;
  return call(f, args, std::index_sequence_for<A...>{});
}

enum Entry { GEMM, CONV, CONV_WGRAD_STATIC, LAYERNORM, GELU, ATTENTION, ENTRIES };
void* address[ENTRIES];  // null: not told yet

template <int E, typename F> PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return checked(reinterpret_cast<F>(address[E]), args, n);
}
// use(address, ...): of the entry points, in the order of Entry.
PyObject* use(PyObject*, PyObject* const* args, Py_ssize_t n) {
  void* a[ENTRIES];
  if (n != ENTRIES) return PyErr_Format(PyExc_TypeError, "use() takes %d addresses", (int)ENTRIES);
  for (int i = 0; i < ENTRIES; ++i)
    if (!read(args[i], a[i]) || !a[i]) return PyErr_Format(PyExc_TypeError, "use() takes addresses");
  for (int i = 0; i < ENTRIES; ++i) address[i] = a[i];
  Py_RETURN_NONE;
}

PyMethodDef method(const char* name, PyObject* (*f)(PyObject*, PyObject* const*, Py_ssize_t)) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr};
}
// (decltype: the prototypes of the headers, no reference to the functions)
PyMethodDef methods[] = {method("cdp_k_gemm", &entry<GEMM, decltype(&cdp_k_gemm)>),
                         method("cdp_k_conv", &entry<CONV, decltype(&cdp_k_conv)>),
                         method("cdp_k_conv_wgrad_static", &entry<CONV_WGRAD_STATIC, decltype(&cdp_k_conv_wgrad_static)>),
                         method("cdp_k_layernorm", &entry<LAYERNORM, decltype(&cdp_k_layernorm)>),
                         method("cdp_k_gelu", &entry<GELU, decltype(&cdp_k_gelu)>),
                         method("cdp_k_attention", &entry<ATTENTION, decltype(&cdp_k_attention)>),
                         method("use", &use),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
