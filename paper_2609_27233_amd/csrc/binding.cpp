// CPython binding of the C calls in spanmerge.h: argument conversion only.
//
// A decode step is a handful of short launches, and through ctypes the
// conversion of their arguments in Python took longer than the launches (one
// step's rule check, input row and projected append: 36 us of host time for
// four calls, 30 us of kernels).  Every entry here takes the C call's
// arguments in order: a tensor (or None) for a device pointer, the ctypes
// structure for a cache or a rule table, the bytes that merge_params or
// kv_proj_params gave for parameters, an int (or None) for a stream handle,
// plain numbers for the rest; it returns the status.  Values are taken and
// refused as ctypes does for the same prototypes: integers wrap to the C
// type's width, a ctypes number of the argument's own type counts as its
// value, and what does not fit raises ctypes.ArgumentError.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <dlfcn.h>

#include <cstring>
#include <tuple>
#include <type_traits>
#include <utility>

#include "spanmerge.h"

namespace {

// The entries, resolved by open() from the library that the program loaded.
#define SM_ENTRIES(X)                                                                                         \
  X(sm_merge_spans) X(sm_merge_token_table) X(sm_merge_spans_tabled) X(sm_pack_spans) X(sm_kv_rollback)       \
  X(sm_kv_append) X(sm_decode_attention) X(sm_decode_step) X(sm_decode_merge_step)                            \
  X(sm_decode_step_noalloc) X(sm_prefill_attention) X(sm_rules_build) X(sm_rules_lookup) X(sm_match_prompt)   \
  X(sm_match_decode) X(sm_gather_surrogates) X(sm_span_dedupe) X(sm_kv_project) X(sm_kv_append_projected)
#define SM_SLOT(name) decltype(&::name) p_##name;
SM_ENTRIES(SM_SLOT)

PyObject *g_is_cuda, *g_is_contiguous, *g_data_ptr, *g_value;  // interned names

// What setup() is given: the exceptions for unusable tensors and for other
// unusable arguments, the structures, and the C types of plain arguments.
enum { kError, kArgumentError, kPagedCache, kRuleTable, kInt, kInt64, kFloat, kSize, kPointer, kTypes };
PyObject *g_type[kTypes];

bool is_true(PyObject *r, const char *otherwise) {
  if (!r) return false;
  const int v = PyObject_IsTrue(r);
  Py_DECREF(r);
  if (v == 0) PyErr_SetString(g_type[kError], otherwise);
  return v > 0;
}

bool tensor_address(PyObject *t, void **p) {
  *p = nullptr;
  if (t == Py_None) return true;
  if (!is_true(PyObject_GetAttr(t, g_is_cuda), "expected a GPU tensor")) return false;
  if (!is_true(PyObject_CallMethodNoArgs(t, g_is_contiguous), "expected a contiguous tensor")) return false;
  PyObject *r = PyObject_CallMethodNoArgs(t, g_data_ptr);
  if (!r) return false;
  *p = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  return !PyErr_Occurred();
}

template <class T>
constexpr bool is_host_struct = std::is_same_v<T, sm_paged_cache> || std::is_same_v<T, sm_rule_table> ||
                                std::is_same_v<T, sm_merge_params> || std::is_same_v<T, sm_kv_proj_params>;

// the C type that a plain argument (or a stream handle) has in the prototypes
template <class A>
constexpr int plain_type = std::is_same_v<A, hipStream_t>      ? kPointer
                           : std::is_floating_point_v<A>       ? kFloat
                           : std::is_same_v<A, size_t>         ? kSize
                           : sizeof(A) == 8                    ? kInt64
                                                               : kInt;

// a new reference to o, or to its value where o is a ctypes number of type t
PyObject *plain_value(PyObject *o, int t) {
  if (!PyLong_Check(o) && !PyFloat_Check(o) && PyObject_TypeCheck(o, (PyTypeObject *)g_type[t]))
    return PyObject_GetAttr(o, g_value);
  Py_INCREF(o);
  return o;
}

template <class T>
bool get_struct(PyObject *o, T **v) {
  *v = nullptr;
  if (o == Py_None) return true;
  constexpr int t = std::is_same_v<std::remove_cv_t<T>, sm_paged_cache>  ? kPagedCache
                    : std::is_same_v<std::remove_cv_t<T>, sm_rule_table> ? kRuleTable
                                                                         : kTypes;  // the parameters: bytes
  const bool right = t == kTypes ? PyBytes_Check(o) : PyObject_TypeCheck(o, (PyTypeObject *)g_type[t % kTypes]);
  Py_buffer b;
  if (!right) {
    PyErr_SetString(PyExc_TypeError, "wrong structure");
    return false;
  }
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return false;
  const bool whole = b.len >= (Py_ssize_t)sizeof(T);
  *v = (T *)b.buf;  // (the caller's object keeps it for the length of the call)
  PyBuffer_Release(&b);
  if (!whole) PyErr_SetString(PyExc_TypeError, "structure too short");
  return whole;
}

template <class A>
bool get(PyObject *o, A *v) {
  if constexpr (std::is_pointer_v<A> && !std::is_same_v<A, hipStream_t>) {
    if constexpr (is_host_struct<std::remove_cv_t<std::remove_pointer_t<A>>>) {
      return get_struct(o, v);
    } else {
      void *p;
      if (!tensor_address(o, &p)) return false;
      *v = (A)p;
      return true;
    }
  } else {
    PyObject *x = plain_value(o, plain_type<A>);
    if (!x) return false;
    if constexpr (std::is_same_v<A, hipStream_t>) {
      *v = nullptr;
      if (PyLong_Check(x)) *v = (hipStream_t)(uintptr_t)PyLong_AsUnsignedLongLongMask(x);
      else if (x != Py_None) PyErr_SetString(PyExc_TypeError, "expected a stream handle");
    } else if constexpr (std::is_floating_point_v<A>) {
      *v = (A)PyFloat_AsDouble(x);
    } else {
      *v = (A)PyLong_AsUnsignedLongLongMask(x);
    }
    Py_DECREF(x);
    return !PyErr_Occurred();
  }
}

// A TypeError of argument `at` (from 1) as ctypes reports it.
void argument_error(int at) {
  if (!PyErr_ExceptionMatches(PyExc_TypeError)) return;
  PyObject *type, *value, *trace;
  PyErr_Fetch(&type, &value, &trace);
  PyErr_Format(g_type[kArgumentError], "argument %d: %S: %S", at, type, value ? value : Py_None);
  Py_XDECREF(type);
  Py_XDECREF(value);
  Py_XDECREF(trace);
}

template <class... A, size_t... I>
PyObject *call(sm_status (*fn)(A...), PyObject *const *args, Py_ssize_t n, std::index_sequence<I...>) {
  if (n != (Py_ssize_t)sizeof...(A)) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  std::tuple<A...> v;
  int at = 0;
  if (!((++at, get(args[I], &std::get<I>(v))) && ...)) {
    argument_error(at);
    return nullptr;
  }
  sm_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = fn(std::get<I>(v)...);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(st);
}

template <class... A>
PyObject *dispatch(sm_status (*fn)(A...), PyObject *const *args, Py_ssize_t n) {
  return call(fn, args, n, std::index_sequence_for<A...>{});
}

template <auto *Fn>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (!*Fn) {
    PyErr_SetString(g_type[kError], "the library is not open");
    return nullptr;
  }
  return dispatch(*Fn, args, n);
}

// open(path): the entries of the library at `path` (kept loaded)
PyObject *open_library(PyObject *, PyObject *path) {
  PyObject *name;
  if (!PyUnicode_FSConverter(path, &name)) return nullptr;
  void *lib = dlopen(PyBytes_AS_STRING(name), RTLD_NOW | RTLD_LOCAL);
  Py_DECREF(name);
  if (!lib) {
    PyErr_SetString(g_type[kError], dlerror());
    return nullptr;
  }
#define SM_FIND(name)                                                   \
  void *const f_##name = dlsym(lib, #name);                             \
  if (!f_##name) {                                                      \
    PyErr_SetString(g_type[kError], "the library lacks the entry " #name);     \
    return nullptr;                                                     \
  }
  SM_ENTRIES(SM_FIND)
#define SM_STORE(name) p_##name = (decltype(&::name))f_##name;
  SM_ENTRIES(SM_STORE)
  Py_RETURN_NONE;
}

// merge_params(d, h, ln_eps, Q, W_kv, b_kv, g_kv, beta_kv, W_o, b_o, g_o, beta_o): the structure's bytes
PyObject *merge_params(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != 12) {
    PyErr_SetString(PyExc_TypeError, "merge_params takes 12 arguments");
    return nullptr;
  }
  sm_merge_params p;
  std::memset(&p, 0, sizeof p);
  const void **field[9] = {&p.Q, &p.W_kv, &p.b_kv, &p.g_kv, &p.beta_kv, &p.W_o, &p.b_o, &p.g_o, &p.beta_o};
  if (!get(args[0], &p.d) || !get(args[1], &p.h) || !get(args[2], &p.ln_eps)) return nullptr;
  for (int i = 0; i < 9; ++i)
    if (!get(args[3 + i], field[i])) return nullptr;
  return PyBytes_FromStringAndSize((const char *)&p, sizeof p);
}

// kv_proj_params(d, W_k, W_v, rope_theta, rms_eps): the structure's bytes
PyObject *kv_proj_params(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "kv_proj_params takes 5 arguments");
    return nullptr;
  }
  sm_kv_proj_params p;
  std::memset(&p, 0, sizeof p);
  if (!get(args[0], &p.d) || !get(args[1], &p.W_k) || !get(args[2], &p.W_v) || !get(args[3], &p.rope_theta) ||
      !get(args[4], &p.rms_eps))
    return nullptr;
  return PyBytes_FromStringAndSize((const char *)&p, sizeof p);
}

// setup(types): the objects of the enumeration above, in its order
PyObject *setup(PyObject *, PyObject *types) {
  if (!PyTuple_Check(types) || PyTuple_GET_SIZE(types) != kTypes) {
    PyErr_SetString(PyExc_TypeError, "setup takes a tuple of the types");
    return nullptr;
  }
  for (int i = 0; i < kTypes; ++i) {
    PyObject *t = PyTuple_GET_ITEM(types, i);
    if (!PyType_Check(t)) {
      PyErr_SetString(PyExc_TypeError, "setup takes a tuple of the types");
      return nullptr;
    }
    Py_INCREF(t);
    Py_XSETREF(g_type[i], t);
  }
  Py_RETURN_NONE;
}

#define SM_ENTRY(name) {#name, (PyCFunction)(void (*)(void))entry<&p_##name>, METH_FASTCALL, nullptr},
PyMethodDef methods[] = {
    SM_ENTRIES(SM_ENTRY)
    {"merge_params", (PyCFunction)(void (*)(void))merge_params, METH_FASTCALL, nullptr},
    {"kv_proj_params", (PyCFunction)(void (*)(void))kv_proj_params, METH_FASTCALL, nullptr},
    {"setup", setup, METH_O, nullptr},
    {"open", open_library, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  g_is_cuda = PyUnicode_InternFromString("is_cuda");
  g_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  g_value = PyUnicode_InternFromString("value");
  if (!g_is_cuda || !g_is_contiguous || !g_data_ptr || !g_value) return nullptr;
  for (PyObject *&t : g_type) {  // (until setup: no structure or ctypes number is of these types)
    Py_INCREF(PyExc_RuntimeError);
    t = PyExc_RuntimeError;
  }
  return PyModule_Create(&module);
}
