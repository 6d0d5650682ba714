// Native half of the Python binding (api.py): argument checks, output and
// scratch allocation, and the call into the library, for the ordinary form of
// every entry point.
//
// A call's host work is what bounds the smallest calls: marshalled in Python
// through ctypes, a B1 H2 S128 D64 forward kept the host busy for 17.7 us and a
// backward for 27.2; here 5.4 and 9.2 (one library call is 4 of them), and a
// differentiable forward and backward went from 196 to 99, of which 52 are
// torch's own for an empty function.
//
// Each function takes positional arguments and returns
//   * the call's outputs,
//   * the library's return code, when that is not 0, or
//   * None for anything but plain arguments: a tensor of another type, shape,
//     device or layout than the call needs, a tensor subclass, a transform's
//     or a mode's wrapper, a table not built yet, a value that does not
//     convert.  The caller then marshals the call itself, which raises what
//     there is to raise.
// Nothing is kept between calls.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>

#include "attnfuse.h"
#include "binding.h"

namespace {

using at::Tensor;

struct NotPlain {};   // thrown inside, never past an entry function

// ---------------------------------------------------------------- arguments
struct Args {
  PyObject* const* v;
  Py_ssize_t n, i = 0;
  PyObject* next() {
    if (i >= n) throw NotPlain{};
    return v[i++];
  }
  // A tensor whose memory is its own: exactly torch.Tensor (or Parameter),
  // strided, not wrapped by a transform or a mode.  None: an empty optional.
  const Tensor* tensor() {
    PyObject* o = next();
    if (o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) throw NotPlain{};
    const Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.has_storage()) throw NotPlain{};
    constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                           c10::DispatchKey::Functionalize, c10::DispatchKey::Python,
                                           c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                           c10::DispatchKey::ZeroTensor});
    if (t.key_set().has_any(wrapped)) throw NotPlain{};
    return &t;
  }
  const Tensor& need() {
    const Tensor* t = tensor();
    if (!t) throw NotPlain{};
    return *t;
  }
  double number() {
    PyObject* o = next();
    if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) throw NotPlain{};
    const double x = PyFloat_AsDouble(o);
    if (x == -1.0 && PyErr_Occurred()) {
      PyErr_Clear();
      throw NotPlain{};
    }
    return x;
  }
  long long whole() {
    PyObject* o = next();
    if (o == Py_None) return 0;
    if (!PyLong_CheckExact(o)) throw NotPlain{};
    const long long x = PyLong_AsLongLong(o);
    if (x == -1 && PyErr_Occurred()) {
      PyErr_Clear();
      throw NotPlain{};
    }
    return x;
  }
  int index() {   // an enum's value, or -1 for an unknown name
    const long long x = whole();
    if (x < 0 || x > 2) throw NotPlain{};
    return (int)x;
  }
  int size() {
    const long long x = whole();
    if (x < INT_MIN || x > INT_MAX) throw NotPlain{};
    return (int)x;
  }
  template <class T>
  const T* pointer() {
    return reinterpret_cast<const T*>(static_cast<uintptr_t>(whole()));
  }
  float scale(int64_t D) {
    if (i < n && v[i] == Py_None) {
      ++i;
      return (float)(1.0 / std::sqrt((double)D));
    }
    return (float)number();
  }
};

void same(const Tensor& t, at::IntArrayRef shape, at::ScalarType type, c10::Device dev) {
  if (t.device() != dev || t.scalar_type() != type || t.sizes() != shape || !t.is_contiguous()) throw NotPlain{};
}

Tensor out_or(const Tensor* given, at::IntArrayRef shape, at::ScalarType type, c10::Device dev) {
  if (given) {
    same(*given, shape, type, dev);
    return *given;
  }
  return at::empty(shape, at::TensorOptions().dtype(type).device(dev));
}

int dtype_of(const Tensor& q) {
  if (!q.is_cuda()) throw NotPlain{};
  if (q.scalar_type() == at::kBFloat16) return AF_DTYPE_BF16;
  if (q.scalar_type() == at::kFloat) return AF_DTYPE_FP32;
  throw NotPlain{};
}

// ---------------------------------------------------------------- RoPE table
// The call's cos/sin table: the caller's, or one of the binding's (api._TABLES:
// a dict of (device index, D, theta) -> list of tables).
struct Table {
  const float* ptr = nullptr;
  int rows = 0;
};

Table table_of(Args& a, int rope, double theta, int64_t D, int64_t S, c10::Device dev) {
  const Tensor* given = a.tensor();
  PyObject* tables = a.next();
  Table r;
  if (rope == AF_ROPE_NONE) return r;
  auto take = [&](const Tensor& t) {
    r.ptr = static_cast<const float*>(t.const_data_ptr());
    r.rows = (int)t.size(0);
  };
  if (given) {
    if (given->dim() != 3 || given->size(0) < S || given->size(0) > INT_MAX) throw NotPlain{};
    same(*given, {given->size(0), D / 2, 2}, at::kFloat, dev);
    take(*given);
    return r;
  }
  if (!PyDict_CheckExact(tables)) throw NotPlain{};
  PyObject* key = Py_BuildValue("(iid)", (int)dev.index(), (int)D, (double)(float)theta);
  if (!key) {
    PyErr_Clear();
    throw NotPlain{};
  }
  PyObject* list = PyDict_GetItemWithError(tables, key);   // borrowed
  Py_DECREF(key);
  if (!list || !PyList_CheckExact(list)) {
    PyErr_Clear();
    throw NotPlain{};
  }
  for (Py_ssize_t i = 0; i < PyList_GET_SIZE(list); ++i) {
    PyObject* o = PyList_GET_ITEM(list, i);
    if (!THPVariable_CheckExact(o)) throw NotPlain{};
    const Tensor& t = THPVariable_Unpack(o);
    if (t.size(0) >= S) {
      take(t);
      return r;
    }
  }
  throw NotPlain{};
}

// ---------------------------------------------------------------- calls
struct NoGil {
  PyThreadState* s = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(s); }
};

// f(stream) on dev's current stream, without the interpreter's lock.
template <class F>
int enqueue(c10::Device dev, F f) {
  const c10::DeviceGuard guard(dev);
  void* st = c10::hip::getCurrentHIPStream(dev.index()).stream();
  NoGil unlocked;
  return f(st);
}

const float* slopes_of(const Tensor* s, int64_t H, c10::Device dev) {
  if (!s) return nullptr;
  same(*s, {H}, at::kFloat, dev);
  return static_cast<const float*>(s->const_data_ptr());
}

const void* in(const Tensor& t) { return t.const_data_ptr(); }
void* out(const Tensor& t) { return t.mutable_data_ptr(); }

PyObject* tuple_of(std::initializer_list<const Tensor*> ts) {
  PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
  if (!r) return nullptr;
  Py_ssize_t i = 0;
  for (const Tensor* t : ts) {
    PyObject* o = t && t->defined() ? THPVariable_Wrap(*t) : (Py_INCREF(Py_None), Py_None);
    if (!o) {
      Py_DECREF(r);
      return nullptr;
    }
    PyTuple_SET_ITEM(r, i++, o);
  }
  return r;
}

// q [B, H, S, D], k and v [B, H_kv, S, D], one device, one dtype.
struct Qkv {
  const Tensor &q, &k, &v;
  c10::Device dev;
  int dtype;
  int64_t B, H, Hkv, S, D;
  at::ScalarType type;
  explicit Qkv(Args& a)
      : q(a.need()), k(a.need()), v(a.need()), dev(q.device()), dtype(dtype_of(q)), type(q.scalar_type()) {
    if (q.dim() != 4 || k.dim() != 4) throw NotPlain{};
    B = q.size(0); H = q.size(1); S = q.size(2); D = q.size(3); Hkv = k.size(1);
    for (int64_t x : {B, H, S, D, Hkv}) if (x > INT_MAX) throw NotPlain{};
    same(q, q.sizes(), type, dev);
    same(k, {B, Hkv, S, D}, type, dev);
    same(v, {B, Hkv, S, D}, type, dev);
  }
};

// bias pointer and strides, normalisation (zeros for the plain calls)
struct Bias {
  const float* p;
  long long sb, sh, sq;
  int norm;
  explicit Bias(Args& a) : p(a.pointer<float>()), sb(a.whole()), sh(a.whole()), sq(a.whole()), norm(a.index()) {}
};

// fwd(q, k, v, out, lse, slopes, table, tables, rope, theta, mask, window, scale,
//     bias, sb, sh, sq, norm, q_block_ptr, k_block_idx, blocks) -> (O, LSE)
PyObject* fwd(Args a) {
  Qkv x(a);
  const Tensor *out_ = a.tensor(), *lse = a.tensor(), *slopes = a.tensor();
  Args late = a;            // the table needs the variant, which follows it
  a.i += 2;
  const int rope = a.index();
  const double theta = a.number();
  const int mask = a.index(), window = a.size();
  const float scale = a.scale(x.D);
  const Bias bias(a);
  const int *qp = a.pointer<int>(), *ki = a.pointer<int>();
  const long long blocks = a.whole();
  const Table tab = table_of(late, rope, theta, x.D, x.S, x.dev);
  const float* sl = slopes_of(slopes, x.H, x.dev);
  const bool relu = bias.norm == AF_NORM_RELU;
  const Tensor o = out_or(out_, x.q.sizes(), x.type, x.dev);
  Tensor l;
  if (!relu || lse) l = out_or(lse, {x.B, x.H, x.S}, at::kFloat, x.dev);
  float* lp = l.defined() ? static_cast<float*>(out(l)) : nullptr;
  const int B = (int)x.B, H = (int)x.H, Hkv = (int)x.Hkv, S = (int)x.S, D = (int)x.D;
  Tensor ws;                // keys rotated once, where that is faster
  if (const size_t n = af_fwd_workspace_bytes(B, H, Hkv, S, D, x.dtype, rope, mask, window, bias.norm,
                                              sl || bias.p, blocks)) {
    try {
      ws = at::empty({(int64_t)n}, at::TensorOptions().dtype(at::kByte).device(x.dev));
    } catch (const c10::OutOfMemoryError&) {   // rotated in the loop instead
    }
  }
  const int rc = enqueue(x.dev, [&](void* st) {
    if (ws.defined())
      return af_fwd_ws(in(x.q), in(x.k), in(x.v), out(o), lp, qp, ki, bias.p, bias.sb, bias.sh, bias.sq,
                       bias.norm, out(ws), (size_t)ws.numel(), B, H, Hkv, S, D, x.dtype, rope, (float)theta, tab.ptr,
                       tab.rows, mask, window, sl, scale, st);
    if (qp)
      return attnfuse_fwd_blocksparse(in(x.q), in(x.k), in(x.v), out(o), lp, qp, ki, B, H, Hkv, S, D, x.dtype,
                                      rope, (float)theta, tab.ptr, tab.rows, mask, window, sl, scale, st);
    return attnfuse_fwd_bias_norm(in(x.q), in(x.k), in(x.v), out(o), lp, bias.p, bias.sb, bias.sh, bias.sq,
                                  bias.norm, B, H, Hkv, S, D, x.dtype, rope, (float)theta, tab.ptr, tab.rows, mask,
                                  window, sl, scale, st);
  });
  return rc ? PyLong_FromLong(rc) : tuple_of({&o, &l});
}

// bwd(q, k, v, o, do, lse, dq, dk, dv, workspace, slopes, table, tables, rope, theta, mask, window, scale,
//     bias, sb, sh, sq, norm, q_block_ptr, k_block_idx, k_block_ptr, q_block_idx, longest, tiles) -> (dQ, dK, dV)
PyObject* bwd(Args a) {
  Qkv x(a);
  const Tensor &o = a.need(), &dout = a.need();
  const Tensor *lse = a.tensor(), *dq_ = a.tensor(), *dk_ = a.tensor(), *dv_ = a.tensor(), *ws_ = a.tensor(),
               *slopes = a.tensor();
  Args late = a;
  a.i += 2;
  const int rope = a.index();
  const double theta = a.number();
  const int mask = a.index(), window = a.size();
  const float scale = a.scale(x.D);
  const Bias bias(a);
  const int *qp = a.pointer<int>(), *ki = a.pointer<int>(), *kp = a.pointer<int>(), *qi = a.pointer<int>();
  const int longest = a.size();
  const long long tiles = a.whole();
  const Table tab = table_of(late, rope, theta, x.D, x.S, x.dev);
  const float* sl = slopes_of(slopes, x.H, x.dev);
  same(o, x.q.sizes(), x.type, x.dev);
  same(dout, x.q.sizes(), x.type, x.dev);
  if (lse) same(*lse, {x.B, x.H, x.S}, at::kFloat, x.dev);
  else if (bias.norm != AF_NORM_RELU) throw NotPlain{};
  const float* lp = lse ? static_cast<const float*>(lse->const_data_ptr()) : nullptr;
  const Tensor dq = out_or(dq_, x.q.sizes(), x.type, x.dev), dk = out_or(dk_, x.k.sizes(), x.type, x.dev),
               dv = out_or(dv_, x.k.sizes(), x.type, x.dev);
  const int B = (int)x.B, H = (int)x.H, Hkv = (int)x.Hkv, S = (int)x.S, D = (int)x.D;
  Tensor ws;
  if (ws_) {
    if (ws_->device() != x.dev || !ws_->is_contiguous()) throw NotPlain{};
    ws = *ws_;
  } else {
    ws = at::empty({(int64_t)attnfuse_bwd_workspace_bytes(B, H, Hkv, S, D, rope)},
                   at::TensorOptions().dtype(at::kByte).device(x.dev));
  }
  const size_t n = (size_t)ws.numel() * ws.element_size();
  const int rc = enqueue(x.dev, [&](void* st) {
    if (qp)
      return af_bwd_blocksparse(in(x.q), in(x.k), in(x.v), in(o), in(dout), lp, out(dq), out(dk), out(dv), qp, ki,
                                kp, qi, longest, tiles, out(ws), n, B, H, Hkv, S, D, x.dtype, rope, (float)theta,
                                tab.ptr, tab.rows, mask, window, sl, scale, st);
    return attnfuse_bwd_bias_norm(in(x.q), in(x.k), in(x.v), in(o), in(dout), lp, out(dq), out(dk),
                                  out(dv), bias.p, bias.sb, bias.sh, bias.sq, bias.norm, out(ws), n, B, H, Hkv, S,
                                  D, x.dtype, rope, (float)theta, tab.ptr, tab.rows, mask, window, sl, scale, st);
  });
  return rc ? PyLong_FromLong(rc) : tuple_of({&dq, &dk, &dv});
}

// decode(q, k, v, lens, out, lse, workspace, slopes, table, tables, rope, theta, mask, window, scale, noalloc) -> (O, LSE)
PyObject* decode(Args a) {
  const Tensor &q = a.need(), &k = a.need(), &v = a.need();
  const Tensor *lens = a.tensor(), *out_ = a.tensor(), *lse = a.tensor(), *ws_ = a.tensor(), *slopes = a.tensor();
  Args late = a;
  a.i += 2;
  const int rope = a.index();
  const double theta = a.number();
  const int mask = a.index(), window = a.size();
  const int dtype = dtype_of(q);
  const c10::Device dev = q.device();
  const at::ScalarType type = q.scalar_type();
  if (q.dim() != 3 || k.dim() != 4) throw NotPlain{};
  const int64_t B = q.size(0), H = q.size(1), D = q.size(2), Hkv = k.size(1), S = k.size(2);
  for (int64_t n : {B, H, D, Hkv, S}) if (n > INT_MAX) throw NotPlain{};
  const float scale = a.scale(D);
  const bool noalloc = a.whole() != 0;
  same(q, q.sizes(), type, dev);
  same(k, {B, Hkv, S, D}, type, dev);
  same(v, {B, Hkv, S, D}, type, dev);
  if (lens) same(*lens, {B}, at::kInt, dev);
  const Table tab = table_of(late, rope, theta, D, S, dev);
  const float* sl = slopes_of(slopes, H, dev);
  const Tensor o = out_or(out_, q.sizes(), type, dev), l = out_or(lse, {B, H}, at::kFloat, dev);
  float* lp = static_cast<float*>(out(l));
  const int* ln = lens ? static_cast<const int*>(lens->const_data_ptr()) : nullptr;
  Tensor ws;
  if (!noalloc) {
    if (ws_) {
      if (ws_->device() != dev || !ws_->is_contiguous()) throw NotPlain{};
      ws = *ws_;
    } else {
      ws = at::empty({(int64_t)attnfuse_decode_workspace_bytes((int)B, (int)H, (int)Hkv, (int)S, (int)D)},
                     at::TensorOptions().dtype(at::kByte).device(dev));
    }
  }
  const int rc = enqueue(dev, [&](void* st) {
    if (noalloc)
      return attnfuse_decode_noalloc(in(q), in(k), in(v), ln, out(o), lp, (int)B, (int)H, (int)Hkv, (int)S,
                                     (int)D, dtype, rope, (float)theta, tab.ptr, tab.rows, mask, window, sl, scale, st);
    return attnfuse_decode(in(q), in(k), in(v), ln, out(o), lp, out(ws),
                           (size_t)ws.numel() * ws.element_size(), (int)B, (int)H, (int)Hkv, (int)S, (int)D, dtype,
                           rope, (float)theta, tab.ptr, tab.rows, mask, window, sl, scale, st);
  });
  return rc ? PyLong_FromLong(rc) : tuple_of({&o, &l});
}

// rope(q, k, out_q, out_k, table, tables, rope, theta, inverse) -> (Qr, Kr)
PyObject* rope(Args a) {
  const Tensor& x0 = a.need();
  const Tensor *x1 = a.tensor(), *y0_ = a.tensor(), *y1_ = a.tensor();
  Args late = a;
  a.i += 2;
  const int kind = a.index();
  const double theta = a.number();
  const bool inverse = a.whole() != 0;
  const int dtype = dtype_of(x0);
  const c10::Device dev = x0.device();
  const at::ScalarType type = x0.scalar_type();
  if (x0.dim() != 4 || (!x1 && y1_)) throw NotPlain{};
  const int64_t B = x0.size(0), H = x0.size(1), S = x0.size(2), D = x0.size(3);
  const int64_t Hkv = x1 ? (x1->dim() == 4 ? x1->size(1) : -1) : 1;
  for (int64_t n : {B, H, S, D, Hkv}) if (n > INT_MAX || n < 0) throw NotPlain{};
  same(x0, x0.sizes(), type, dev);
  if (x1) same(*x1, {B, Hkv, S, D}, type, dev);
  const Table tab = table_of(late, kind, theta, D, S, dev);
  const Tensor y0 = out_or(y0_, x0.sizes(), type, dev);
  Tensor y1;
  if (x1) y1 = out_or(y1_, x1->sizes(), type, dev);
  const void* p1 = x1 ? in(*x1) : nullptr;
  void* r1 = x1 ? out(y1) : nullptr;
  const int rc = enqueue(dev, [&](void* st) {
    return (inverse ? attnfuse_rope_bwd : attnfuse_rope)(in(x0), p1, out(y0), r1, (int)B, (int)H, (int)Hkv, (int)S,
                                                         (int)D, dtype, kind, (float)theta, tab.ptr, tab.rows, st);
  });
  return rc ? PyLong_FromLong(rc) : tuple_of({&y0, &y1});
}

template <PyObject* (*F)(Args)>
PyObject* entry(PyObject*, PyObject* const* v, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  try {
    return F(Args{v, n});
  } catch (const NotPlain&) {
    Py_RETURN_NONE;
  }
  END_HANDLE_TH_ERRORS
}

template <PyObject* (*F)(Args)>
constexpr PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<F>)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {method<fwd>("fwd"), method<bwd>("bwd"), method<decode>("decode"), method<rope>("rope"),
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
