// Calls of libstarattn.so from Python without ctypes: tensors and the shape struct become addresses
// here.  A decode step on a short cache takes the GPU about as long as its call takes the
// host, and of a phase-2 call's 8.5 us on the host 4.2 were eight is_contiguous() / data_ptr() pairs and a
// ctypes call; here they are 0.5 (the two kernel launches are the rest).
// What may be passed, and what is refused, is as with ctypes: tensors that are not
// contiguous raise ValueError, subclasses of torch.Tensor and anything else that has
// is_contiguous() and data_ptr() are asked through Python, None is a null pointer, and the interpreter lock
// is released around the call.
#include <Python.h>

#include <stdexcept>

#include <torch/csrc/autograd/python_variable.h>

#include "../../include/star_attn.h"

namespace {

PyObject* shape_type = nullptr;

// The library's entry points, by position in bind()'s argument.
struct EntryPoints {
  decltype(&star_attn_phase1) phase1;
  decltype(&star_attn_phase1_anchor) phase1_anchor;
  decltype(&star_attn_phase1_rope) phase1_rope;
  decltype(&star_attn_phase2) phase2;
  decltype(&star_attn_phase2_rope) phase2_rope;
  decltype(&star_attn_phase2_static) phase2_static;
  decltype(&star_attn_phase2_partial) phase2_partial;
  decltype(&star_attn_merge) merge;
  decltype(&star_attn_rope) rope;
} lib;

// Reads a call's arguments in order; `ok` is false once a Python error is set.
struct Args {
  PyObject* const* at;
  PyObject* const* end;
  bool ok = true;
  Py_buffer view;
  bool has_view = false;

  Args(PyObject* const* args, Py_ssize_t n, Py_ssize_t want) : at(args), end(args + n) {
    if (n != want) fail(PyExc_TypeError, "wrong number of arguments");
  }
  ~Args() {
    if (has_view) PyBuffer_Release(&view);
  }
  void fail(PyObject* type, const char* what) {
    if (ok) PyErr_SetString(type, what);
    ok = false;
  }
  PyObject* next() { return ok && at < end ? *at++ : nullptr; }

  const star_attn_shape* shape() {
    PyObject* o = next();
    if (!o) return nullptr;
    if (!shape_type || !PyObject_TypeCheck(o, (PyTypeObject*)shape_type)) {
      fail(PyExc_TypeError, "a StarShape is wanted");
      return nullptr;
    }
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) { ok = false; return nullptr; }
    has_view = true;
    if (view.len < (Py_ssize_t)sizeof(star_attn_shape)) { fail(PyExc_TypeError, "a StarShape is wanted"); return nullptr; }
    return (const star_attn_shape*)view.buf;
  }
  int64_t integer() {
    PyObject* o = next();
    if (!o) return 0;
    const int64_t x = (int64_t)PyLong_AsUnsignedLongLongMask(o);      // (wraps, as ctypes does)
    if (x == -1 && PyErr_Occurred()) ok = false;
    return x;
  }
  double real() {
    PyObject* o = next();
    if (!o) return 0;
    const double x = PyFloat_AsDouble(o);
    if (x == -1.0 && PyErr_Occurred()) ok = false;
    return x;
  }
  void* pointer() {
    PyObject* o = next();
    return o ? address(o) : nullptr;
  }
  void* stream() { return (void*)(uintptr_t)integer(); }
  // A tensor's address, with the size of its dimension `dim`, or its bytes (dim = -1).
  void* sized(int dim, int64_t* size) {
    PyObject* o = next();
    *size = 0;
    if (!o) return nullptr;
    void* p = address(o);
    if (ok && o != Py_None) *size = dim < 0 ? bytes(o) : extent(o, dim);
    else if (ok && dim >= 0) fail(PyExc_AttributeError, "'NoneType' object has no attribute 'shape'");
    return p;
  }
  // shape[dim] of the next argument, which is read again as a tensor afterwards.
  int64_t peek_extent(int dim) {
    if (!ok || at >= end) return 0;
    return extent(*at, dim);
  }

 private:
  static const at::Tensor* plain(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }
  int64_t number(PyObject* o) {
    if (!o) { ok = false; return 0; }
    const int64_t x = (int64_t)PyLong_AsUnsignedLongLongMask(o);
    Py_DECREF(o);
    if (x == -1 && PyErr_Occurred()) ok = false;
    return x;
  }
  void* address(PyObject* o) {
    if (o == Py_None) return nullptr;
    const char* strided = "star_attn tensors must be contiguous";
    try {
      if (const at::Tensor* t = plain(o)) {
        if (!t->is_contiguous()) { fail(PyExc_ValueError, strided); return nullptr; }
        return t->data_ptr();
      }
    } catch (const std::exception& e) {
      fail(PyExc_RuntimeError, e.what());
      return nullptr;
    }
    PyObject* c = PyObject_CallMethod(o, "is_contiguous", nullptr);
    if (!c) { ok = false; return nullptr; }
    const int yes = PyObject_IsTrue(c);
    Py_DECREF(c);
    if (yes < 0) { ok = false; return nullptr; }
    if (!yes) { fail(PyExc_ValueError, strided); return nullptr; }
    return (void*)(uintptr_t)number(PyObject_CallMethod(o, "data_ptr", nullptr));
  }
  int64_t extent(PyObject* o, int dim) {
    try {
      if (const at::Tensor* t = plain(o)) {
        if (t->dim() <= dim) { fail(PyExc_IndexError, "tuple index out of range"); return 0; }
        return t->size(dim);
      }
    } catch (const std::exception& e) {
      fail(PyExc_RuntimeError, e.what());
      return 0;
    }
    PyObject* s = PyObject_GetAttrString(o, "shape");
    if (!s) { ok = false; return 0; }
    PyObject* x = PySequence_GetItem(s, dim);
    Py_DECREF(s);
    return number(x);
  }
  int64_t bytes(PyObject* o) {
    try {
      if (const at::Tensor* t = plain(o)) return (int64_t)t->numel() * (int64_t)t->element_size();
    } catch (const std::exception& e) {
      fail(PyExc_RuntimeError, e.what());
      return 0;
    }
    const int64_t n = number(PyObject_CallMethod(o, "numel", nullptr));
    return ok ? n * number(PyObject_CallMethod(o, "element_size", nullptr)) : 0;
  }
};

// What a call returns: the library's status, from outside the interpreter lock.
template <typename Call>
PyObject* finish(Args& a, const void* entry, Call call) {
  if (a.ok && !entry) a.fail(PyExc_RuntimeError, "libstarattn is not loaded");
  if (!a.ok) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

#define FASTCALL(name) PyObject* name(PyObject*, PyObject* const* args, Py_ssize_t n)

// phase1(shape, Q, K, V, O_ctx, LSE_ctx, K_cache, V_cache, workspace, stream)
FASTCALL(phase1) {
  Args a(args, n, 10);
  const star_attn_shape* s = a.shape();
  void *Q = a.pointer(), *K = a.pointer(), *V = a.pointer(), *O = a.pointer(), *L = a.pointer(), *Kc = a.pointer(), *Vc = a.pointer();
  int64_t ws_n;
  void *ws = a.sized(-1, &ws_n), *st = a.stream();
  return finish(a, (const void*)lib.phase1, [&] { return lib.phase1(s, Q, K, V, O, (float*)L, Kc, Vc, ws, (size_t)ws_n, st); });
}
// phase1_anchor(shape, mode, Q, K, V, K_anchor, V_anchor, O_ctx, LSE_ctx, K_cache, V_cache, workspace, stream)
FASTCALL(phase1_anchor) {
  Args a(args, n, 13);
  const star_attn_shape* s = a.shape();
  const int mode = (int)a.integer();
  void *Q = a.pointer(), *K = a.pointer(), *V = a.pointer(), *Ka = a.pointer(), *Va = a.pointer(), *O = a.pointer(), *L = a.pointer(),
       *Kc = a.pointer(), *Vc = a.pointer();
  int64_t ws_n;
  void *ws = a.sized(-1, &ws_n), *st = a.stream();
  return finish(a, (const void*)lib.phase1_anchor,
                [&] { return lib.phase1_anchor(s, mode, Q, K, V, Ka, Va, O, (float*)L, Kc, Vc, ws, (size_t)ws_n, st); });
}
// phase1_rope(shape, theta, pos0, Q, K, V, O_ctx, LSE_ctx, K_cache, V_cache, workspace, stream)
FASTCALL(phase1_rope) {
  Args a(args, n, 12);
  const star_attn_shape* s = a.shape();
  const double theta = a.real();
  const int64_t pos0 = a.integer();
  void *Q = a.pointer(), *K = a.pointer(), *V = a.pointer(), *O = a.pointer(), *L = a.pointer(), *Kc = a.pointer(), *Vc = a.pointer();
  int64_t ws_n;
  void *ws = a.sized(-1, &ws_n), *st = a.stream();
  return finish(a, (const void*)lib.phase1_rope,
                [&] { return lib.phase1_rope(s, theta, pos0, Q, K, V, O, (float*)L, Kc, Vc, ws, (size_t)ws_n, st); });
}
// phase2(shape, cache_len, Qq, Kq, Vq, K_cache, V_cache, O_part, LSE_part, O, workspace, stream)
FASTCALL(phase2) {
  Args a(args, n, 12);
  const star_attn_shape* s = a.shape();
  const int64_t cached = a.integer();
  int64_t q, ws_n;
  void *Q = a.sized(1, &q), *K = a.pointer(), *V = a.pointer(), *Kc = a.pointer(), *Vc = a.pointer(), *Op = a.pointer(),
       *Lp = a.pointer(), *O = a.pointer(), *ws = a.sized(-1, &ws_n), *st = a.stream();
  return finish(a, (const void*)lib.phase2,
                [&] { return lib.phase2(s, cached, q, Q, K, V, Kc, Vc, (float*)Op, (float*)Lp, O, ws, (size_t)ws_n, st); });
}
// phase2_rope(shape, theta, pos0, cache_len, Qq, Kq, Vq, K_cache, V_cache, O_part, LSE_part, O, workspace, stream)
FASTCALL(phase2_rope) {
  Args a(args, n, 14);
  const star_attn_shape* s = a.shape();
  const double theta = a.real();
  const int64_t pos0 = a.integer(), cached = a.integer();
  int64_t q, ws_n;
  void *Q = a.sized(1, &q), *K = a.pointer(), *V = a.pointer(), *Kc = a.pointer(), *Vc = a.pointer(), *Op = a.pointer(),
       *Lp = a.pointer(), *O = a.pointer(), *ws = a.sized(-1, &ws_n), *st = a.stream();
  return finish(a, (const void*)lib.phase2_rope, [&] {
    return lib.phase2_rope(s, theta, pos0, cached, q, Q, K, V, Kc, Vc, (float*)Op, (float*)Lp, O, ws, (size_t)ws_n, st);
  });
}
// phase2_static(shape, cache_len, Qq, Kq, Vq, K_cache, V_cache, O, stream)
FASTCALL(phase2_static) {
  Args a(args, n, 9);
  const star_attn_shape* s = a.shape();
  const int64_t cached = a.integer();
  int64_t q;
  void *Q = a.sized(1, &q), *K = a.pointer(), *V = a.pointer(), *Kc = a.pointer(), *Vc = a.pointer(), *O = a.pointer(),
       *st = a.stream();
  return finish(a, (const void*)lib.phase2_static, [&] { return lib.phase2_static(s, cached, q, Q, K, V, Kc, Vc, O, st); });
}
// phase2_partial(shape, cache_len, Qq, Kq, Vq, K_cache, V_cache, A, LSE, workspace, stream)
FASTCALL(phase2_partial) {
  Args a(args, n, 11);
  const star_attn_shape* s = a.shape();
  const int64_t cached = a.integer();
  int64_t q, ws_n;
  void *Q = a.sized(1, &q), *K = a.pointer(), *V = a.pointer(), *Kc = a.pointer(), *Vc = a.pointer(), *A = a.pointer(),
       *L = a.pointer(), *ws = a.sized(-1, &ws_n), *st = a.stream();
  return finish(a, (const void*)lib.phase2_partial, [&] {
    return lib.phase2_partial(s, cached, q, Q, K, V, Kc, Vc, (float*)A, (float*)L, ws, (size_t)ws_n, st);
  });
}
// merge(shape, A_parts, LSE_parts, O, A, LSE, stream)
FASTCALL(merge) {
  Args a(args, n, 7);
  const star_attn_shape* s = a.shape();
  int64_t parts;
  const int64_t q = a.peek_extent(3);
  void *Ap = a.sized(0, &parts), *Lp = a.pointer(), *O = a.pointer(), *A = a.pointer(), *L = a.pointer(), *st = a.stream();
  return finish(a, (const void*)lib.merge,
                [&] { return lib.merge(s, parts, q, (const float*)Ap, (const float*)Lp, O, (float*)A, (float*)L, st); });
}
// rope(shape, X, Y, theta, pos0, stream)
FASTCALL(rope) {
  Args a(args, n, 6);
  const star_attn_shape* s = a.shape();
  const int64_t tokens = a.peek_extent(1);
  int64_t heads;
  void *X = a.sized(2, &heads), *Y = a.pointer();
  const double theta = a.real();
  const int64_t pos0 = a.integer();
  void* st = a.stream();
  return finish(a, (const void*)lib.rope, [&] { return lib.rope(s, (int32_t)heads, tokens, pos0, theta, X, Y, st); });
}

// bind(StarShape, (addresses of the entry points, in the order of EntryPoints))
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *type, *addresses;
  if (!PyArg_ParseTuple(args, "O!O!", &PyType_Type, &type, &PyTuple_Type, &addresses)) return nullptr;
  void* p[sizeof(EntryPoints) / sizeof(void*)];
  constexpr Py_ssize_t n = sizeof(p) / sizeof(p[0]);
  if (PyTuple_GET_SIZE(addresses) != n) {
    PyErr_SetString(PyExc_ValueError, "wrong number of entry points");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < n; ++i) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
      return nullptr;
    }
  }
  static_assert(sizeof(lib) == sizeof(p), "nothing but function pointers");
  memcpy((void*)&lib, p, sizeof(lib));
  Py_INCREF(type);
  Py_XDECREF(shape_type);
  shape_type = type;
  Py_RETURN_NONE;
}

#define ENTRY(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(phase1), ENTRY(phase1_anchor), ENTRY(phase1_rope), ENTRY(phase2), ENTRY(phase2_rope),
                         ENTRY(phase2_static), ENTRY(phase2_partial), ENTRY(merge), ENTRY(rope),
                         {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "libstarattn's entry points on torch tensors", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
