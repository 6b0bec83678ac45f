// CPython module behind the package's tensor functions: checks the tensors,
// allocates what the caller did not give, and calls the C ABI on the current
// stream.  The host cost of a call bounds every small problem: the launch
// itself takes about 3.5 us, and the same checks and conversions in Python
// with ctypes took another 8 to 10 (per call on the smallest problems, before
// and after: prefill 11.7 and 4.9 us, decode with its output and workspace
// given 12.1 and 3.4, L2 norm 11.9 and 5.1, RMSNorm 13.8 and 6.5).
//
// A call that is not plainly valid (a wrong shape or type, a subclass, a
// stream argument, an unusual scalar) returns None from here, and the Python
// function goes through its own checks, which raise the errors.  A returned
// int is the C ABI's error status.

#include <Python.h>

#include <algorithm>
#include <climits>
#include <cmath>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/attn.h"
#include "../../include/norms.h"

namespace {

// A plain contiguous GPU tensor, or nullptr.
const at::Tensor* plain(PyObject* obj) {
  if (!THPVariable_CheckExact(obj)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(obj);
  return t.layout() == c10::kStrided && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

// Every size fits the C ABI's int arguments.
bool ints(const at::Tensor& t) {
  for (int64_t n : t.sizes())
    if (n > INT_MAX) return false;
  return true;
}

bool number(PyObject* obj, float& x) {
  if (PyFloat_CheckExact(obj)) x = (float)PyFloat_AS_DOUBLE(obj);
  else if (PyLong_CheckExact(obj)) {
    const double d = PyLong_AsDouble(obj);
    if (d == -1.0 && PyErr_Occurred()) {
      PyErr_Clear();
      return false;
    }
    x = (float)d;
  } else return false;
  return true;
}

// A Python int that fits.
bool whole(PyObject* obj, int& x) {
  if (!PyLong_CheckExact(obj)) return false;
  int over = 0;
  const long long v = PyLong_AsLongLongAndOverflow(obj, &over);
  if (over || v < INT_MIN || v > INT_MAX) return false;
  x = (int)v;
  return true;
}

bool truth(PyObject* obj, bool& x) {
  if (!PyBool_Check(obj)) return false;
  x = obj == Py_True;
  return true;
}

hipStream_t stream() { return c10::hip::getCurrentHIPStream().stream(); }

PyObject* none() { Py_RETURN_NONE; }

// Run f (a C ABI call) without the interpreter lock.
template <typename F>
int unlocked(F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return rc;
}

// The given output object, or a new reference to the allocated tensor.
PyObject* result(int rc, PyObject* given, at::Tensor&& made) {
  if (rc != ATTN_OK) return PyLong_FromLong(rc);
  if (given != Py_None) {
    Py_INCREF(given);
    return given;
  }
  return THPVariable_Wrap(std::move(made));
}

struct Attn {
  const at::Tensor *q, *k, *v;
  at::Tensor o;
  const float* slopes = nullptr;
  attn_dtype dtype;
  int B, Hq, Hkv, Lq, Lk, D;
  float scale;
};

// The arguments shared by the attention calls; false if not plainly valid.
bool attn_args(PyObject* q, PyObject* k, PyObject* v, PyObject* o, PyObject* scale, PyObject* slopes, Attn& a) {
  a.q = plain(q);
  a.k = plain(k);
  a.v = plain(v);
  if (!a.q || !a.k || !a.v || a.q->dim() != 4 || a.k->dim() != 4) return false;
  const auto dt = a.q->scalar_type();
  if ((dt != at::kHalf && dt != at::kBFloat16) || a.k->scalar_type() != dt || a.v->scalar_type() != dt) return false;
  if (a.k->sizes() != a.v->sizes() || a.k->size(0) != a.q->size(0) || a.k->size(3) != a.q->size(3)) return false;
  if (!ints(*a.q) || !ints(*a.k)) return false;
  a.dtype = dt == at::kHalf ? ATTN_F16 : ATTN_BF16;
  a.B = (int)a.q->size(0);
  a.Hq = (int)a.q->size(1);
  a.Lq = (int)a.q->size(2);
  a.D = (int)a.q->size(3);
  a.Hkv = (int)a.k->size(1);
  a.Lk = (int)a.k->size(2);
  if (slopes != Py_None) {
    const at::Tensor* s = plain(slopes);
    if (!s || s->scalar_type() != at::kFloat || s->numel() != a.Hq) return false;
    a.slopes = static_cast<const float*>(s->data_ptr());
  }
  if (scale == Py_None) {
    if (a.D < 1) return false;
    a.scale = (float)(1.0 / std::sqrt((double)a.D));
  } else if (!number(scale, a.scale)) return false;
  if (o != Py_None) {
    const at::Tensor* t = plain(o);
    if (!t || t->scalar_type() != dt || t->sizes() != a.q->sizes()) return false;
    a.o = *t;
  } else {
    a.o = at::empty_like(*a.q);
  }
  return true;
}

// (q, k, v, o, causal, scale, alibi_slopes, softcap, window, stream)
PyObject* py_attn_fwd(PyObject*, PyObject* const* x, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Attn a;
  bool causal;
  float cap = 0.f;
  int window = 0;
  if (n != 10 || x[9] != Py_None || !truth(x[4], causal)) return none();
  if (x[8] != Py_None && !whole(x[8], window)) return none();
  if (x[7] != Py_None && !number(x[7], cap)) return none();
  if (!attn_args(x[0], x[1], x[2], x[3], x[5], x[6], a)) return none();
  const void *q = a.q->data_ptr(), *k = a.k->data_ptr(), *v = a.v->data_ptr();
  void* o = a.o.data_ptr();
  // Few rows against many keys: a workspace, which lives on this stream like
  // the call itself (so not for tensors on another device).  Where memory has
  // run out the call does without it.
  at::Tensor ws;
  size_t bytes = 0;
  const int S = attn_fwd_num_splits(a.B, a.Hq, a.Hkv, a.Lq, a.Lk, a.D, causal, window);
  if (S > 1 && a.q->device().index() == c10::hip::getCurrentHIPStream().device_index()) {
    bytes = attn_fwd_workspace_bytes(a.B, a.Hq, a.Lq, a.D, S);
    try {
      ws = at::empty({(int64_t)bytes}, a.q->options().dtype(at::kByte));
    } catch (const c10::OutOfMemoryError&) {
      bytes = 0;
    }
  }
  void* w = bytes ? ws.data_ptr() : nullptr;
  const hipStream_t s = stream();
  const int rc = unlocked([&] {
    return attn_fwd_split(q, k, v, o, a.B, a.Hq, a.Hkv, a.Lq, a.Lk, a.D, causal, a.scale, a.slopes, cap, window, w,
                          bytes, a.dtype, s);
  });
  return result(rc, x[3], std::move(a.o));
  END_HANDLE_TH_ERRORS
}

// (q, k, v, o, scale, alibi_slopes, softcap, num_splits, workspace, stream)
PyObject* py_attn_decode(PyObject*, PyObject* const* x, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Attn a;
  float cap = 0.f;
  int splits;
  if (n != 10 || x[9] != Py_None || !whole(x[7], splits)) return none();
  if (x[6] != Py_None && !number(x[6], cap)) return none();
  at::Tensor ws;
  if (x[8] != Py_None) {
    const at::Tensor* t = plain(x[8]);
    if (!t) return none();
    ws = *t;
  }
  if (!attn_args(x[0], x[1], x[2], x[3], x[4], x[5], a) || a.Lq != 1) return none();
  if (!ws.defined()) {
    const int S = splits ? splits : attn_decode_num_splits(a.B, a.Hq, a.Hkv, a.Lk, a.D);
    const size_t need = attn_decode_workspace_bytes(a.B, a.Hq, a.D, std::max(S, 1));
    ws = at::empty({(int64_t)std::max<size_t>(need, 16)}, a.q->options().dtype(at::kByte));
  }
  const void *q = a.q->data_ptr(), *k = a.k->data_ptr(), *v = a.v->data_ptr();
  void *o = a.o.data_ptr(), *w = ws.data_ptr();
  const size_t bytes = ws.nbytes();
  const hipStream_t s = stream();
  const int rc = unlocked([&] {
    return attn_decode_mod(q, k, v, o, a.B, a.Hq, a.Hkv, a.Lk, a.D, a.scale, a.slopes, cap, splits, w, bytes, a.dtype,
                           s);
  });
  return result(rc, x[3], std::move(a.o));
  END_HANDLE_TH_ERRORS
}

// (q, k, v, o, scale, alibi_slopes, softcap, num_splits, stream)
PyObject* py_attn_decode_noalloc(PyObject*, PyObject* const* x, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Attn a;
  float cap = 0.f;
  int splits;
  if (n != 9 || x[8] != Py_None || !whole(x[7], splits)) return none();
  if (x[6] != Py_None && !number(x[6], cap)) return none();
  if (!attn_args(x[0], x[1], x[2], x[3], x[4], x[5], a) || a.Lq != 1) return none();
  const void *q = a.q->data_ptr(), *k = a.k->data_ptr(), *v = a.v->data_ptr();
  void* o = a.o.data_ptr();
  const hipStream_t s = stream();
  const int rc = unlocked([&] {
    return attn_decode_noalloc(q, k, v, o, a.B, a.Hq, a.Hkv, a.Lk, a.D, a.scale, a.slopes, cap, splits, a.dtype, s);
  });
  return result(rc, x[3], std::move(a.o));
  END_HANDLE_TH_ERRORS
}

struct Norm {
  const at::Tensor* x;
  at::Tensor ws, out, y;
  norm_dtype dtype;
  int N, M, chunks;
};

bool norm_args(PyObject* px, PyObject* pout, PyObject* chunks, PyObject* workspace, bool rms, PyObject* py, Norm& a) {
  a.x = plain(px);
  if (!a.x || a.x->dim() != 2 || !ints(*a.x) || !whole(chunks, a.chunks)) return false;
  const auto dt = a.x->scalar_type();
  if (dt == at::kHalf) a.dtype = NORM_F16;
  else if (dt == at::kBFloat16) a.dtype = NORM_BF16;
  else if (dt == at::kFloat) a.dtype = NORM_F32;
  else return false;
  a.N = (int)a.x->size(0);
  a.M = (int)a.x->size(1);
  if (pout != Py_None) {
    const at::Tensor* t = plain(pout);
    if (!t || t->scalar_type() != at::kFloat || t->numel() != a.N) return false;
    a.out = *t;
  }
  if (rms && py != Py_None) {
    const at::Tensor* t = plain(py);
    if (!t || t->scalar_type() != dt || t->sizes() != a.x->sizes()) return false;
    a.y = *t;
  }
  if (workspace != Py_None) {
    const at::Tensor* t = plain(workspace);
    if (!t) return false;
    a.ws = *t;
  }
  const auto opt = a.x->options();
  if (!a.ws.defined()) {
    const int C = a.chunks ? a.chunks : norm_chunks(rms, a.N, a.M, a.dtype);
    a.ws = at::empty({(int64_t)std::max<size_t>(norm_workspace_bytes(a.N, std::max(C, 1)), 16)}, opt.dtype(at::kByte));
  }
  if (rms && !a.y.defined()) a.y = at::empty_like(*a.x);
  if (!a.out.defined()) a.out = at::empty({(int64_t)a.N}, opt.dtype(at::kFloat));
  return true;
}

// (x, out, chunks, workspace, stream)
PyObject* py_norm_l2(PyObject*, PyObject* const* x, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Norm a;
  if (n != 5 || x[4] != Py_None || !norm_args(x[0], x[1], x[2], x[3], false, nullptr, a)) return none();
  const void* px = a.x->data_ptr();
  float* out = static_cast<float*>(a.out.data_ptr());
  void* w = a.ws.data_ptr();
  const size_t bytes = a.ws.nbytes();
  const hipStream_t s = stream();
  const int rc = unlocked([&] { return norm_l2(px, out, a.N, a.M, a.dtype, a.chunks, w, bytes, s); });
  return result(rc, x[1], std::move(a.out));
  END_HANDLE_TH_ERRORS
}

// (x, y, rowmax, eps, chunks, workspace, stream) -> (y, rowmax)
PyObject* py_rmsnorm_rowmax(PyObject*, PyObject* const* x, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Norm a;
  float eps;
  if (n != 7 || x[6] != Py_None || !number(x[3], eps) || !norm_args(x[0], x[2], x[4], x[5], true, x[1], a))
    return none();
  const void* px = a.x->data_ptr();
  void *y = a.y.data_ptr(), *w = a.ws.data_ptr();
  float* out = static_cast<float*>(a.out.data_ptr());
  const size_t bytes = a.ws.nbytes();
  const hipStream_t s = stream();
  const int rc =
      unlocked([&] { return rmsnorm_rowmax(px, y, out, a.N, a.M, eps, a.dtype, a.chunks, w, bytes, s); });
  if (rc != ATTN_OK) return PyLong_FromLong(rc);
  PyObject* r = PyTuple_New(2);
  if (!r) return nullptr;
  PyTuple_SET_ITEM(r, 0, result(rc, x[1], std::move(a.y)));
  PyTuple_SET_ITEM(r, 1, result(rc, x[2], std::move(a.out)));
  return r;
  END_HANDLE_TH_ERRORS
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyCFunction fast() {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F));
}

PyMethodDef methods[] = {
    {"attn_fwd", fast<py_attn_fwd>(), METH_FASTCALL, nullptr},
    {"attn_decode", fast<py_attn_decode>(), METH_FASTCALL, nullptr},
    {"attn_decode_noalloc", fast<py_attn_decode_noalloc>(), METH_FASTCALL, nullptr},
    {"norm_l2", fast<py_norm_l2>(), METH_FASTCALL, nullptr},
    {"rmsnorm_rowmax", fast<py_rmsnorm_rowmax>(), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
