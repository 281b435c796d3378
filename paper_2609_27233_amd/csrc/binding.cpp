// CPython binding of the C calls in spanmerge.h: argument conversion only.
//
// A decode step is a handful of short launches, and through ctypes the
// conversion of their arguments in Python took longer than the launches (one
// step's rule check, input row and projected append: 36 us of host time for
// four calls, 30 us of kernels).  Every entry here takes the C call's
// arguments in order: a tensor (or None) for a device pointer, an object with
// a buffer (a ctypes structure, bytes) for a host structure, an int for a
// stream handle, plain numbers for the rest; it returns the status.
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

PyObject *g_is_cuda, *g_is_contiguous, *g_data_ptr;  // interned names
PyObject *g_error;                                   // the exception for unusable tensors

bool is_true(PyObject *r, const char *otherwise) {
  if (!r) return false;
  const int v = PyObject_IsTrue(r);
  Py_DECREF(r);
  if (v == 0) PyErr_SetString(g_error, otherwise);
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

template <class A>
bool get(PyObject *o, A *v) {
  if constexpr (std::is_same_v<A, hipStream_t>) {
    *v = (hipStream_t)PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
  } else if constexpr (std::is_pointer_v<A>) {
    using T = std::remove_cv_t<std::remove_pointer_t<A>>;
    if constexpr (is_host_struct<T>) {
      *v = nullptr;
      if (o == Py_None) return true;
      Py_buffer b;
      if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return false;
      const bool whole = b.len >= (Py_ssize_t)sizeof(T);
      *v = (A)b.buf;  // (the caller's object keeps it for the length of the call)
      PyBuffer_Release(&b);
      if (!whole) PyErr_SetString(PyExc_ValueError, "structure too short");
      return whole;
    } else {
      void *p;
      if (!tensor_address(o, &p)) return false;
      *v = (A)p;
      return true;
    }
  } else if constexpr (std::is_floating_point_v<A>) {
    *v = (A)PyFloat_AsDouble(o);
    return !PyErr_Occurred();
  } else if constexpr (std::is_same_v<A, size_t>) {
    *v = PyLong_AsSize_t(o);
    return !PyErr_Occurred();
  } else {
    const long long x = PyLong_AsLongLong(o);
    if (PyErr_Occurred()) return false;
    if constexpr (sizeof(A) == 4) {
      if (x != (long long)(int)x) {
        PyErr_SetString(PyExc_OverflowError, "argument does not fit 32 bits");
        return false;
      }
    }
    *v = (A)x;
    return true;
  }
}

template <class... A, size_t... I>
PyObject *call(sm_status (*fn)(A...), PyObject *const *args, Py_ssize_t n, std::index_sequence<I...>) {
  if (n != (Py_ssize_t)sizeof...(A)) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  std::tuple<A...> v;
  if (!(get(args[I], &std::get<I>(v)) && ...)) return nullptr;
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
    PyErr_SetString(g_error, "the library is not open");
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
    PyErr_SetString(g_error, dlerror());
    return nullptr;
  }
#define SM_FIND(name)                                                   \
  void *const f_##name = dlsym(lib, #name);                             \
  if (!f_##name) {                                                      \
    PyErr_SetString(g_error, "the library lacks the entry " #name);     \
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

PyObject *set_error(PyObject *, PyObject *type) {
  Py_INCREF(type);
  Py_XSETREF(g_error, type);
  Py_RETURN_NONE;
}

#define SM_ENTRY(name) {#name, (PyCFunction)(void (*)(void))entry<&p_##name>, METH_FASTCALL, nullptr},
PyMethodDef methods[] = {
    SM_ENTRIES(SM_ENTRY)
    {"merge_params", (PyCFunction)(void (*)(void))merge_params, METH_FASTCALL, nullptr},
    {"kv_proj_params", (PyCFunction)(void (*)(void))kv_proj_params, METH_FASTCALL, nullptr},
    {"set_error", set_error, METH_O, nullptr},
    {"open", open_library, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  g_is_cuda = PyUnicode_InternFromString("is_cuda");
  g_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  if (!g_is_cuda || !g_is_contiguous || !g_data_ptr) return nullptr;
  Py_INCREF(PyExc_RuntimeError);
  g_error = PyExc_RuntimeError;
  return PyModule_Create(&module);
}
