// Native marshalling for binding.py: the checks, allocations and the call of its usual entry points in one C++ function.
//
// A short call (a decoding step, the training step of a short sequence) is bound by the host: from Python, with its
// attribute reads, tensor constructions and ctypes conversions, a decoding call takes 17.7 us of the host's time, a forward
// call 11.2 and a forward + backward 27.9, where the GPU needs 14.5 for the first and the last. Here they take 9.3, 5.4 and 12.1.
//
// Nothing is decided here that binding.py does not decide. Each function handles the ordinary call, plain tensors of the
// right types and shapes and outputs that it allocates, and returns None for everything else (a subclass, an active
// mode or transform, a wrong shape, an argument of an unusual type, an error from the library): binding.py then goes its own
// way through the same checks and raises its own errors. No state but the addresses that init() is given.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "../../include/fa.h"

namespace {

// ---- the library's entry points, by the order of kNames (binding.py hands their addresses over)
#define FA_HOST_ENTRIES(X)                                                                                            \
  X(fa_fwd) X(fa_bwd) X(fa_bwd_workspace_bytes) X(fa_cross_fwd) X(fa_cross_fwd_f16) X(fa_cross_bwd) X(fa_cross_bwd_f16) \
  X(fa_cross_bwd_workspace_bytes) X(fa_dropout_fwd) X(fa_dropout_fwd_f16) X(fa_dropout_bwd) X(fa_dropout_bwd_f16)       \
  X(fa_local_fwd) X(fa_local_fwd_f16) X(fa_local_bwd) X(fa_local_bwd_f16) X(fa_varlen_fwd) X(fa_varlen_fwd_f16)         \
  X(fa_varlen_bwd) X(fa_varlen_bwd_f16) X(fa_varlen_bwd_workspace_bytes) X(fa_kvcache_fwd) X(fa_kvcache_fwd_f16)        \
  X(fa_splitkv_fwd_workspace_bytes)
struct Entries {
#define X(name) decltype(&::name) name;
  FA_HOST_ENTRIES(X)
#undef X
} lib;
PyObject *get_device, *get_stream, *parameter_type;  // (owned references)
bool ready = false;

// ---- what an ordinary call looks like
bool plain_context() {
  return ready && !c10::impl::TorchDispatchModeTLS::any_modes_set() && at::impl::PythonTorchFunctionTLS::stack_len() == 0 &&
         !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}
// A dense contiguous GPU tensor with memory of its own, or nullptr.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o) && (PyObject*)Py_TYPE(o) != parameter_type) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  using K = c10::DispatchKey;
  if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || !t.has_storage() || t.numel() == 0 || !t.is_contiguous() ||
      t.key_set().has_any(c10::DispatchKeySet({K::Python, K::Negative, K::Conjugate, K::ZeroTensor, K::Functionalize,
                                               K::FuncTorchBatched, K::FuncTorchGradWrapper})))
    return nullptr;
  for (int64_t n : t.sizes())
    if (n > INT_MAX) return nullptr;
  return &t;
}
bool is(const at::Tensor* t, at::ScalarType st, c10::Device dev, at::IntArrayRef shape) {
  return t && t->scalar_type() == st && t->device() == dev && t->sizes() == shape;
}
bool flag(PyObject* o, int& v) {
  if (!PyBool_Check(o)) return false;
  v = o == Py_True;
  return true;
}
bool number(PyObject* o, float& v) {
  if (!PyFloat_CheckExact(o)) return false;
  v = (float)PyFloat_AS_DOUBLE(o);
  return true;
}
bool integer(PyObject* o, int& v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow;
  const long x = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || x > INT_MAX || x < INT_MIN) return false;
  v = (int)x;
  return true;
}
bool current_stream(void*& st) {  // of the current device, as binding.py has it
  PyObject* d = PyObject_CallNoArgs(get_device);
  if (!d) return false;
  PyObject* s = PyObject_CallOneArg(get_stream, d);
  Py_DECREF(d);
  if (!s) return false;
  st = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return !PyErr_Occurred();
}
at::Tensor make(at::IntArrayRef shape, at::ScalarType st, c10::Device dev) {
  return at::empty(shape, at::TensorOptions().dtype(st).device(dev));
}
const void* in(const at::Tensor* t) { return t->const_data_ptr(); }
const float* stat(const at::Tensor* t) { return (const float*)t->const_data_ptr(); }
PyObject* pack(std::initializer_list<at::Tensor> ts) {
  PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
  if (!r) return nullptr;
  Py_ssize_t i = 0;
  for (const at::Tensor& t : ts) {
    PyObject* o = THPVariable_Wrap(t);
    if (!o) {
      Py_DECREF(r);
      return nullptr;
    }
    PyTuple_SET_ITEM(r, i++, o);
  }
  return r;
}
template <class F>
int without_gil(F f) {  // (a launch waits while the queue is full)
  int e;
  Py_BEGIN_ALLOW_THREADS e = f();
  Py_END_ALLOW_THREADS return e;
}

// ---- dense batches: 0 fa_fwd, 1 fa_cross_fwd, 2 fa_dropout_fwd, 3 fa_local_fwd, and their backward passes
struct Dense {
  int kind, B, Nq, Nk, Hq, Hkv, d, causal = 0, left = 0, right = 0;
  float scale, p_drop = 0.f;
  uint64_t seed = 0;
  bool f16;
  c10::Device dev = c10::kCPU;
  at::ScalarType et;
  const at::Tensor *Q, *K, *V;
  // kind, Q, K, V, then at args[opt]: scale and the options of the kind
  bool parse(PyObject* const* args, Py_ssize_t nargs, int opt) {
    if (nargs < opt + 2 || !plain_context() || !integer(args[0], kind)) return false;
    Q = plain(args[1]), K = plain(args[2]), V = plain(args[3]);
    if (!Q || !K || Q->dim() != 4 || K->dim() != 4 || !number(args[opt], scale)) return false;
    et = Q->scalar_type(), dev = Q->device(), f16 = et == at::kHalf;
    if (et != at::kBFloat16 && !(f16 && kind != 0)) return false;
    B = (int)Q->size(0), Nq = (int)Q->size(1), Hq = (int)Q->size(2), d = (int)Q->size(3);
    Nk = (int)K->size(1), Hkv = (int)K->size(2);
    if (kind == 0 && Nk != Nq) return false;
    if (!is(K, et, dev, {B, Nk, Hkv, d}) || !is(V, et, dev, {B, Nk, Hkv, d})) return false;
    if (kind == 3) return nargs == opt + 3 && integer(args[opt + 1], left) && integer(args[opt + 2], right);
    if (!flag(args[opt + 1], causal)) return false;
    if (kind == 2) {
      if (nargs != opt + 4 || !number(args[opt + 2], p_drop) || !PyLong_CheckExact(args[opt + 3])) return false;
      seed = PyLong_AsUnsignedLongLongMask(args[opt + 3]);
      return true;
    }
    return nargs == opt + 2;
  }
};

PyObject* dense_fwd(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  Dense x;
  void* st;
  if (!x.parse(args, nargs, 4)) Py_RETURN_NONE;
  if (!current_stream(st)) return nullptr;
  at::Tensor O = make({x.B, x.Nq, x.Hq, x.d}, x.et, x.dev), L = make({x.B, x.Hq, x.Nq}, at::kFloat, x.dev);
  const void *q = in(x.Q), *k = in(x.K), *v = in(x.V);
  void* o = O.mutable_data_ptr();
  float* l = (float*)L.mutable_data_ptr();
  const int e = without_gil([&] {
    switch (x.kind) {
      case 0: return lib.fa_fwd(q, k, v, o, l, x.B, x.Hq, x.Hkv, x.Nq, x.d, x.scale, x.causal, st);
      case 1: return (x.f16 ? lib.fa_cross_fwd_f16 : lib.fa_cross_fwd)(q, k, v, o, l, x.B, x.Hq, x.Hkv, x.Nq, x.Nk, x.d, x.scale,
                                                                       x.causal, st);
      case 2: return (x.f16 ? lib.fa_dropout_fwd_f16 : lib.fa_dropout_fwd)(q, k, v, o, l, x.B, x.Hq, x.Hkv, x.Nq, x.Nk, x.d,
                                                                           x.scale, x.causal, x.p_drop, x.seed, st);
      case 3: return (x.f16 ? lib.fa_local_fwd_f16 : lib.fa_local_fwd)(q, k, v, o, l, x.B, x.Hq, x.Hkv, x.Nq, x.Nk, x.d, x.scale,
                                                                       x.left, x.right, st);
      default: return -1;
    }
  });
  if (e) Py_RETURN_NONE;
  return pack({O, L});
  END_HANDLE_TH_ERRORS
}

PyObject* dense_bwd(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  Dense x;
  void* st;
  if (!x.parse(args, nargs, 7)) Py_RETURN_NONE;
  const at::Tensor *O = plain(args[4]), *dO = plain(args[5]), *L = plain(args[6]);
  if (!is(O, x.et, x.dev, x.Q->sizes()) || !is(dO, x.et, x.dev, x.Q->sizes()) || !is(L, at::kFloat, x.dev, {x.B, x.Hq, x.Nq}))
    Py_RETURN_NONE;
  if (!current_stream(st)) return nullptr;
  at::Tensor dQ = make(x.Q->sizes(), x.et, x.dev), dK = make(x.K->sizes(), x.et, x.dev), dV = make(x.K->sizes(), x.et, x.dev);
  const size_t nb = x.kind == 0 ? lib.fa_bwd_workspace_bytes(x.B, x.Hq, x.Hkv, x.Nq, x.d)
                                : lib.fa_cross_bwd_workspace_bytes(x.B, x.Hq, x.Hkv, x.Nq, x.Nk, x.d);
  at::Tensor W = make({(int64_t)nb}, at::kByte, x.dev);
  const void *q = in(x.Q), *k = in(x.K), *v = in(x.V), *o = in(O), *g = in(dO);
  const float* l = stat(L);
  void *dq = dQ.mutable_data_ptr(), *dk = dK.mutable_data_ptr(), *dv = dV.mutable_data_ptr(), *w = W.mutable_data_ptr();
  const int e = without_gil([&] {
    switch (x.kind) {
      case 0: return lib.fa_bwd(q, k, v, o, g, l, dq, dk, dv, w, nb, x.B, x.Hq, x.Hkv, x.Nq, x.d, x.scale, x.causal, st);
      case 1: return (x.f16 ? lib.fa_cross_bwd_f16 : lib.fa_cross_bwd)(q, k, v, o, g, l, dq, dk, dv, w, nb, x.B, x.Hq, x.Hkv, x.Nq,
                                                                       x.Nk, x.d, x.scale, x.causal, st);
      case 2: return (x.f16 ? lib.fa_dropout_bwd_f16 : lib.fa_dropout_bwd)(q, k, v, o, g, l, dq, dk, dv, w, nb, x.B, x.Hq, x.Hkv,
                                                                           x.Nq, x.Nk, x.d, x.scale, x.causal, x.p_drop, x.seed, st);
      case 3: return (x.f16 ? lib.fa_local_bwd_f16 : lib.fa_local_bwd)(q, k, v, o, g, l, dq, dk, dv, w, nb, x.B, x.Hq, x.Hkv, x.Nq,
                                                                       x.Nk, x.d, x.scale, x.left, x.right, st);
      default: return -1;
    }
  });
  if (e) Py_RETURN_NONE;
  return pack({dQ, dK, dV});
  END_HANDLE_TH_ERRORS
}

// ---- packed batches
struct Packed {
  int T, Hq, Hkv, d, nseq, longest, causal;
  float scale;
  bool f16;
  c10::Device dev = c10::kCPU;
  at::ScalarType et;
  const at::Tensor *Q, *K, *V, *cu;
  bool parse(PyObject* const* args, Py_ssize_t nargs, int opt) {  // at args[opt]: cu_seqlens, max_seqlen, scale, causal
    if (nargs != opt + 4 || !plain_context()) return false;
    Q = plain(args[0]), K = plain(args[1]), V = plain(args[2]), cu = plain(args[opt]);
    if (!Q || !K || !cu || Q->dim() != 3 || K->dim() != 3) return false;
    if (!integer(args[opt + 1], longest) || !number(args[opt + 2], scale) || !flag(args[opt + 3], causal)) return false;
    et = Q->scalar_type(), dev = Q->device(), f16 = et == at::kHalf;
    if (et != at::kBFloat16 && !f16) return false;
    T = (int)Q->size(0), Hq = (int)Q->size(1), d = (int)Q->size(2), Hkv = (int)K->size(1);
    if (!is(K, et, dev, {T, Hkv, d}) || !is(V, et, dev, {T, Hkv, d})) return false;
    nseq = (int)cu->numel() - 1;
    return cu->scalar_type() == at::kInt && cu->device() == dev && cu->dim() == 1 && nseq >= 1;
  }
};

PyObject* varlen_fwd(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  Packed x;
  void* st;
  if (!x.parse(args, nargs, 3)) Py_RETURN_NONE;
  if (!current_stream(st)) return nullptr;
  at::Tensor O = make(x.Q->sizes(), x.et, x.dev), L = make({x.Hq, x.T}, at::kFloat, x.dev);
  const void *q = in(x.Q), *k = in(x.K), *v = in(x.V);
  const int32_t* cu = (const int32_t*)in(x.cu);
  void* o = O.mutable_data_ptr();
  float* l = (float*)L.mutable_data_ptr();
  const int e = without_gil([&] {
    return (x.f16 ? lib.fa_varlen_fwd_f16 : lib.fa_varlen_fwd)(q, k, v, o, l, cu, x.nseq, x.T, x.longest, x.Hq, x.Hkv, x.d, x.scale,
                                                               x.causal, st);
  });
  if (e) Py_RETURN_NONE;
  return pack({O, L});
  END_HANDLE_TH_ERRORS
}

PyObject* varlen_bwd(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  Packed x;
  void* st;
  if (!x.parse(args, nargs, 6)) Py_RETURN_NONE;
  const at::Tensor *O = plain(args[3]), *dO = plain(args[4]), *L = plain(args[5]);
  if (!is(O, x.et, x.dev, x.Q->sizes()) || !is(dO, x.et, x.dev, x.Q->sizes()) || !is(L, at::kFloat, x.dev, {x.Hq, x.T}))
    Py_RETURN_NONE;
  if (!current_stream(st)) return nullptr;
  at::Tensor dQ = make(x.Q->sizes(), x.et, x.dev), dK = make(x.K->sizes(), x.et, x.dev), dV = make(x.K->sizes(), x.et, x.dev);
  // (binding._packed_bwd_bytes)
  auto d_bytes = [&](long rows) { return (size_t)(4 * rows * x.Hq + 255) / 256 * 256; };
  const size_t nb = x.longest > 0 && x.longest <= x.T
                        ? d_bytes(x.T) - d_bytes(x.longest) + lib.fa_cross_bwd_workspace_bytes(1, x.Hq, x.Hkv, x.longest, x.T, x.d)
                        : lib.fa_varlen_bwd_workspace_bytes(x.T, x.Hq, x.Hkv, x.d);
  at::Tensor W = make({(int64_t)nb}, at::kByte, x.dev);
  const void *q = in(x.Q), *k = in(x.K), *v = in(x.V), *o = in(O), *g = in(dO);
  const float* l = stat(L);
  const int32_t* cu = (const int32_t*)in(x.cu);
  void *dq = dQ.mutable_data_ptr(), *dk = dK.mutable_data_ptr(), *dv = dV.mutable_data_ptr(), *w = W.mutable_data_ptr();
  const int e = without_gil([&] {
    return (x.f16 ? lib.fa_varlen_bwd_f16 : lib.fa_varlen_bwd)(q, k, v, o, g, l, dq, dk, dv, w, nb, cu, x.nseq, x.T, x.longest, x.Hq,
                                                               x.Hkv, x.d, x.scale, x.causal, st);
  });
  if (e) Py_RETURN_NONE;
  return pack({dQ, dK, dV});
  END_HANDLE_TH_ERRORS
}

// ---- key/value caches: Q, Kcache, Vcache, scale, causal, seqlens_k, block_table, max_seqlen_k

// binding._cache_splits, which has the reasons (held to it by a test). All arguments positive.
int cache_splits_of(long B, long Hq, long Hkv, long Nq, long Nk, long d, bool ragged) {
  const long rows = Nq * (Hq / Hkv), units = B * Hkv * ((rows + 255) / 256), blocks = (Nk + 63) / 64;
  auto up = [](long a, long b) { return (a + b - 1) / b; };
  long want, least;
  if (!ragged || rows <= 32) {
    const bool many = ragged && !(B <= 128 && rows <= 32);
    if (d == 64 && rows <= 32 && blocks < 16) return 1;
    if (!many && rows <= 32 && units <= 64 && blocks >= 12) {
      const long fit = 256 / units, eights = blocks / 8;
      auto least_of = [](long a, long b) { return a < b ? a : b; };
      if (eights < up(256, units)) {
        const long small = least_of(least_of(fit, 16), blocks / 2), n = small > eights ? small : eights;
        const long equal = up(blocks, up(blocks, n));
        return (int)(n > 16 ? least_of(n, FA_SPLITKV_MAX_SPLITS) : equal > eights ? equal : eights);
      }
      if (blocks <= (fit >= 5 ? 128 : 63)) return (int)least_of(fit, FA_SPLITKV_MAX_SPLITS);
    }
    want = up(many ? 2048 : 256, units), least = many ? 16 : 8;
  } else {
    want = d == 64 ? 512 / units : up(B > 1 ? 384 : 256, units), least = 16;
  }
  long s = FA_SPLITKV_MAX_SPLITS;
  s = s < blocks / least ? s : blocks / least;
  s = s < want ? s : want;
  return (int)(s > 1 ? s : 1);
}

PyObject* kvcache_fwd(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 8 || !plain_context()) Py_RETURN_NONE;
  const at::Tensor *Q = plain(args[0]), *K = plain(args[1]), *V = plain(args[2]), *lens = nullptr, *table = nullptr;
  float scale;
  int causal, max_k, page = 0, pages = 0;
  void* st;
  if (!Q || !K || Q->dim() != 4 || K->dim() != 4 || !number(args[3], scale) || !flag(args[4], causal) || !integer(args[7], max_k))
    Py_RETURN_NONE;
  const at::ScalarType et = Q->scalar_type();
  const c10::Device dev = Q->device();
  const bool f16 = et == at::kHalf;
  const int B = (int)Q->size(0), Nq = (int)Q->size(1), Hq = (int)Q->size(2), d = (int)Q->size(3), Hkv = (int)K->size(2);
  if ((et != at::kBFloat16 && !f16) || K->size(3) != d || !is(K, et, dev, K->sizes()) || !is(V, et, dev, K->sizes()) || Hq % Hkv)
    Py_RETURN_NONE;
  long Nk = K->size(1);
  if (args[6] == Py_None) {
    if (K->size(0) != B) Py_RETURN_NONE;
  } else {
    table = plain(args[6]);
    if (!table || table->dim() != 2 || !is(table, at::kInt, dev, {B, table->size(1)})) Py_RETURN_NONE;
    page = (int)K->size(1), pages = (int)table->size(1);
    Nk = max_k > 0 ? max_k : (long)page * pages;
    if (Nk > INT_MAX) Py_RETURN_NONE;
  }
  if (args[5] != Py_None) {
    lens = plain(args[5]);
    if (!is(lens, at::kInt, dev, {B})) Py_RETURN_NONE;
  }
  if (!current_stream(st)) return nullptr;
  const int splits = cache_splits_of(B, Hq, Hkv, Nq, Nk, d, lens != nullptr);
  at::Tensor O = make(Q->sizes(), et, dev), L = make({B, Hq, Nq}, at::kFloat, dev);
  const size_t nb = lib.fa_splitkv_fwd_workspace_bytes(B, Hq, Nq, d, splits);
  at::Tensor W = make({(int64_t)nb}, at::kByte, dev);
  const void *q = in(Q), *k = in(K), *v = in(V);
  const int32_t *ln = lens ? (const int32_t*)in(lens) : nullptr, *tb = table ? (const int32_t*)in(table) : nullptr;
  void *o = O.mutable_data_ptr(), *w = W.mutable_data_ptr();
  float* l = (float*)L.mutable_data_ptr();
  const int e = without_gil([&] {
    return (f16 ? lib.fa_kvcache_fwd_f16 : lib.fa_kvcache_fwd)(q, k, v, ln, tb, o, l, w, nb, B, Hq, Hkv, Nq, (int)Nk, d, page, pages,
                                                               scale, causal, splits, st);
  });
  if (e) Py_RETURN_NONE;
  return pack({O, L});
  END_HANDLE_TH_ERRORS
}

PyObject* cache_splits(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  int v[6], ragged;
  for (int i = 0; i < 6; ++i)
    if (nargs != 7 || !integer(args[i], v[i])) Py_RETURN_NONE;
  if (!flag(args[6], ragged)) Py_RETURN_NONE;
  return PyLong_FromLong(cache_splits_of(v[0], v[1], v[2], v[3], v[4], v[5], ragged));
}

PyObject* init(PyObject*, PyObject* args) {  // get_device, get_stream, Parameter, {entry point: address}
  PyObject *dev, *st, *par, *addr;
  if (!PyArg_ParseTuple(args, "OOOO!", &dev, &st, &par, &PyDict_Type, &addr)) return nullptr;
  Entries e;
  PyObject* a;
#define X(name)                                                        \
  a = PyDict_GetItemString(addr, #name);                               \
  if (!a) return PyErr_Format(PyExc_KeyError, "no address of " #name); \
  e.name = (decltype(e.name))PyLong_AsVoidPtr(a);                      \
  if (PyErr_Occurred()) return nullptr;
  FA_HOST_ENTRIES(X)
#undef X
  Py_INCREF(dev);
  Py_INCREF(st);
  Py_INCREF(par);
  Py_XDECREF(get_device);
  Py_XDECREF(get_stream);
  Py_XDECREF(parameter_type);
  get_device = dev, get_stream = st, parameter_type = par, lib = e, ready = true;
  Py_RETURN_NONE;
}

PyObject* entry_names(PyObject*, PyObject*) {
#define X(name) #name,
  const char* names[] = {FA_HOST_ENTRIES(X)};
#undef X
  PyObject* r = PyList_New(0);
  for (const char* n : names) {
    PyObject* s = PyUnicode_FromString(n);
    if (!r || !s || PyList_Append(r, s)) return nullptr;
    Py_DECREF(s);
  }
  return r;
}

#define FAST(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(dense_fwd), FAST(dense_bwd), FAST(varlen_fwd), FAST(varlen_bwd), FAST(kvcache_fwd), FAST(cache_splits),
                         {"init", init, METH_VARARGS, nullptr}, {"entry_names", entry_names, METH_NOARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&module); }
