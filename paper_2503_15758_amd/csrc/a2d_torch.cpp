// The library's calls on torch tensors: what binding.py and grid.py do per call - checks, strides,
// output tensors, the current stream - as a CPython extension module.  Argument marshalling only, no
// arithmetic of the method.
//
// Why native: through ctypes a call costs 11-19 us of host time (descriptor, argument objects, a
// pointer wrapper per tensor), more than the small tiles' kernels take; here it costs 3-5 us, most of
// it the launch itself.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/HIPGeneratorImpl.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <mutex>
#include <string>
#include <vector>

#include "a2d.h"
#include "a2d_grid.hpp"

namespace {

PyObject* g_error_class = nullptr;            // binding.A2DError(status, detail)

struct Error {
  int status;
  std::string detail;
};
[[noreturn]] void fail(int status, const std::string& detail) { throw Error{status, detail}; }
struct PythonError {};                        // a Python exception is set already

void check(a2d_status st) {
  if (st != A2D_OK) fail(st, a2d_last_error());
}

using Args = PyObject* const*;

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s must be a tensor, not %s", name, Py_TYPE(o)->tp_name);
    throw PythonError();
  }
  return THPVariable_Unpack(o);
}
int64_t integer(PyObject* o) {
  if (PyLong_Check(o)) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PythonError();
    return v;
  }
  PyObject* n = PyNumber_Long(o);
  if (!n) throw PythonError();
  const long long v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw PythonError();
  return v;
}
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw PythonError();
  return v != 0;
}
float scale_of(PyObject* o, int64_t hdim) {
  if (o == Py_None) return (float)(1.0 / std::sqrt((double)hdim));
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw PythonError();
  return (float)v;
}
at::ScalarType dtype_arg(PyObject* o) {
  if (!THPDtype_Check(o)) {
    PyErr_Format(PyExc_TypeError, "out_dtype must be a torch.dtype, not %s", Py_TYPE(o)->tp_name);
    throw PythonError();
  }
  return reinterpret_cast<THPDtype*>(o)->scalar_type;
}
int dtype_code(at::ScalarType t) {
  if (t == at::kFloat) return A2D_F32;
  if (t == at::kBFloat16) return A2D_BF16;
  fail(A2D_ERR_UNSUPPORTED, std::string("dtype ") + c10::toString(t) + " not supported");
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// [heads][rows][H] device tensors (or views) whose rows of H elements are contiguous
void dev3(const at::Tensor& t, const char* name) {
  if (!(t.is_cuda() && t.dim() == 3 && (t.stride(2) == 1 || t.size(2) == 1)))
    fail(A2D_ERR_INVALID_ARG, std::string(name) + " must be a [heads][rows][H] device tensor with contiguous rows");
}
// what the library writes is in the plain layout
void plain(const at::Tensor& t, const char* what) {
  if (!(t.is_cuda() && t.is_contiguous()))
    fail(A2D_ERR_INVALID_ARG, std::string(what) + " must be contiguous device tensors");
}
a2d_layout layout(const at::Tensor& t) {
  if (t.is_contiguous()) return a2d_layout{0, 0};
  const int64_t heads = t.size(0), rows = t.size(1), H = t.size(2);
  const int64_t row = rows > 1 ? t.stride(1) : H;      // a stride over a dimension of extent 1 is arbitrary
  return a2d_layout{heads > 1 ? t.stride(0) : rows * row, row};
}

template <class T>
T* data(const at::Tensor& t) {
  return static_cast<T*>(t.data_ptr());
}

a2d_tile_desc descriptor(const at::Tensor& Q, const at::Tensor& K, const at::Tensor& V, Args a, int flags) {
  // a: q_off, kv_off, causal, scale
  a2d_tile_desc d;
  d.heads = (int32_t)Q.size(0);
  d.nq = (int32_t)Q.size(1);
  d.nkv = (int32_t)K.size(1);
  d.hdim = (int32_t)Q.size(2);
  d.q_off = integer(a[0]);
  d.kv_off = integer(a[1]);
  d.causal = truth(a[2]);
  d.scale = scale_of(a[3], Q.size(2));
  d.dtype = dtype_code(Q.scalar_type());
  d.flags = flags;
  d.lq = layout(Q);
  d.lk = layout(K);
  d.lv = layout(V);
  d.lo = d.ldo = a2d_layout{0, 0};
  return d;
}

// None, or a sequence of (kv_off, rows)
struct Segments {
  std::vector<a2d_kv_segment> v;
  bool given = false;
  explicit Segments(PyObject* o) {
    if (o == Py_None) return;
    given = true;
    PyObject* f = PySequence_Fast(o, "segments must be a sequence of (kv_off, rows)");
    if (!f) throw PythonError();
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(f);
    v.resize(n);
    try {
      for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* e = PySequence_Fast(PySequence_Fast_GET_ITEM(f, i), "segments must be a sequence of (kv_off, rows)");
        if (!e) throw PythonError();
        if (PySequence_Fast_GET_SIZE(e) != 2) {
          Py_DECREF(e);
          PyErr_SetString(PyExc_ValueError, "segments must be a sequence of (kv_off, rows)");
          throw PythonError();
        }
        PyObject *off = PySequence_Fast_GET_ITEM(e, 0), *rows = PySequence_Fast_GET_ITEM(e, 1);
        try {
          v[i].kv_off = integer(off);
          v[i].rows = (int32_t)integer(rows);
          v[i].pad = 0;
        } catch (...) {
          Py_DECREF(e);
          throw;
        }
        Py_DECREF(e);
      }
    } catch (...) {
      Py_DECREF(f);
      throw;
    }
    Py_DECREF(f);
  }
  int n() const { return (int)v.size(); }
  const a2d_kv_segment* ptr() const { return v.empty() ? nullptr : v.data(); }
};

// the caller's output tensors, or new ones; give() returns them as a Python tuple (or the one tensor)
struct Outputs {
  static constexpr int kMost = 3;
  at::Tensor t[kMost];
  PyObject* given[kMost] = {nullptr, nullptr, nullptr};   // new references
  int n = 0;
  ~Outputs() {
    for (int i = 0; i < kMost; ++i) Py_XDECREF(given[i]);
  }
  void take(PyObject* out, int count, const char* what, bool must_be_plain = true) {
    n = count;
    PyObject* f = PySequence_Fast(out, "out must be a sequence of tensors");
    if (!f) throw PythonError();
    if (PySequence_Fast_GET_SIZE(f) != count) {
      Py_DECREF(f);
      PyErr_Format(PyExc_ValueError, "out must hold %d tensors: %s", count, what);
      throw PythonError();
    }
    for (int i = 0; i < count; ++i) {
      given[i] = PySequence_Fast_GET_ITEM(f, i);
      Py_INCREF(given[i]);
    }
    Py_DECREF(f);
    for (int i = 0; i < count; ++i) {
      t[i] = tensor(given[i], what);
      if (must_be_plain) plain(t[i], what);
    }
  }
  void add(at::Tensor x) { t[n++] = std::move(x); }
  PyObject* one(int i) {
    if (given[i]) {
      Py_INCREF(given[i]);
      return given[i];
    }
    return THPVariable_Wrap(t[i]);
  }
  PyObject* give() {
    PyObject* r = PyTuple_New(n);
    if (!r) throw PythonError();
    for (int i = 0; i < n; ++i) {
      PyObject* x = one(i);
      if (!x) {
        Py_DECREF(r);
        throw PythonError();
      }
      PyTuple_SET_ITEM(r, i, x);
    }
    return r;
  }
};

// lists of partials
struct Parts {
  std::vector<const at::Tensor*> t;
  PyObject* f;
  Parts(PyObject* o, const char* name) {
    f = PySequence_Fast(o, "the partials must be a sequence of tensors");
    if (!f) throw PythonError();
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(f);
    t.reserve(n);
    try {
      for (Py_ssize_t i = 0; i < n; ++i) t.push_back(&tensor(PySequence_Fast_GET_ITEM(f, i), name));
    } catch (...) {
      Py_DECREF(f);
      throw;
    }
  }
  ~Parts() { Py_DECREF(f); }
  Parts(const Parts&) = delete;
  int k() const { return (int)t.size(); }
  void all_plain(const char* what) const {
    for (auto* x : t) plain(*x, what);
  }
  std::vector<const float*> ptrs() const {
    std::vector<const float*> p;
    p.reserve(t.size());
    for (auto* x : t) p.push_back(data<float>(*x));
    return p;
  }
};

at::Tensor empty_like_shape(const at::Tensor& like, at::IntArrayRef shape, at::ScalarType t) {
  return at::empty(shape, like.options().dtype(t).requires_grad(false));
}
at::IntArrayRef rows_shape(const at::Tensor& t) { return t.sizes().slice(0, t.dim() - 1); }

void qkv(const at::Tensor& Q, const at::Tensor& K, const at::Tensor& V) {
  dev3(Q, "Q");
  dev3(K, "K");
  dev3(V, "V");
  if (K.sizes() != V.sizes() || K.size(2) != Q.size(2) || K.scalar_type() != Q.scalar_type() ||
      V.scalar_type() != Q.scalar_type())
    fail(A2D_ERR_INVALID_ARG, "Q, K, V shapes / dtypes do not match");
}

// Is the stream being captured by torch?  Its allocator then serves it from a pool that lives as long as the
// graph; a capture begun by other means it knows nothing of.  torch's default generator takes part in torch's
// captures, and on a capturing stream it can be asked for its state (here: moved on by nothing) in those only.
// (Called inside the library's frames: nothing may be thrown through them.)
bool torch_captures(const at::Device& device) noexcept {
  try {
    at::Generator g = at::cuda::detail::getDefaultCUDAGenerator(device.index());
    std::lock_guard<std::mutex> lock(g.mutex());
    g.get<at::CUDAGeneratorImpl>()->philox_cuda_state(0);
    return true;
  } catch (...) {
    return false;
  }
}

// Offers the library memory for the partial results of shared walks while it lives: from torch's allocator (the
// blocks go back when it dies; the allocator orders their reuse on the stream) or, for the static calls, the
// library's own device array.  A foreign capture gets none: its graph would replay into memory that has been
// handed out again.  tell() says it where there was no memory, and the call's sums were added in another order.
class Scratch {
  std::vector<at::Tensor> held_;
  const at::Tensor* like_;                           // NULL: the library's array
  hipStream_t stream_;
  size_t missing_ = 0;
  a2d::ScratchSource source_;

  bool capturable() const {
    hipStreamCaptureStatus now = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream_, &now) != hipSuccess) {
      (void)hipGetLastError();                       // (not an error of the launches to come)
      return false;
    }
    return now == hipStreamCaptureStatusNone || torch_captures(like_->device());
  }
  void* allocate(size_t bytes) {
    if (!capturable()) return nullptr;
    try {
      held_.push_back(at::empty({(int64_t)bytes}, like_->options().dtype(at::kByte).requires_grad(false)));
      return held_.back().data_ptr();
    } catch (...) {
      missing_ = bytes;
      return nullptr;
    }
  }
  static void* get(void* self, size_t bytes) {
    Scratch* s = static_cast<Scratch*>(self);
    if (s->like_) return s->allocate(bytes);
    void* p = a2d::static_partial_sums(bytes);
    if (!p) s->missing_ = bytes;
    return p;
  }
  Scratch(const at::Tensor* like, void* stream)
      : like_(like), stream_(static_cast<hipStream_t>(stream)), source_{&Scratch::get, this} {
    a2d::scratch_offer(&source_);
  }

 public:
  Scratch(const at::Tensor& like, void* stream) : Scratch(&like, stream) {}
  explicit Scratch(void* stream) : Scratch(nullptr, stream) {}
  ~Scratch() { a2d::scratch_offer(nullptr); }
  Scratch(const Scratch&) = delete;
  void tell() const {
    if (missing_ && PyErr_WarnFormat(PyExc_RuntimeWarning, 1,
                                     "no memory for partial results (%zu bytes): the call did not share its walks among "
                                     "workgroups, its sums are added in another order", missing_) != 0)
      throw PythonError();
  }
};

// runs f with the GIL released
template <class F>
a2d_status unlocked(F&& f) {
  a2d_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return st;
}

// Q, K, V, q_off, kv_off, causal, scale, out, segments, accumulate
PyObject* partial_fwd(Args a) {
  const at::Tensor &Q = tensor(a[0], "Q"), &K = tensor(a[1], "K"), &V = tensor(a[2], "V");
  qkv(Q, K, V);
  const a2d_tile_desc d = descriptor(Q, K, V, a + 3, 0);
  const Segments segs(a[8]);
  const bool acc = truth(a[9]);
  Outputs o;
  if (a[7] == Py_None) {
    if (acc) fail(A2D_ERR_INVALID_ARG, "accumulate needs out=(O_part, m, l)");
    o.add(empty_like_shape(Q, Q.sizes(), at::kFloat));
    o.add(empty_like_shape(Q, rows_shape(Q), at::kFloat));
    o.add(empty_like_shape(Q, rows_shape(Q), at::kFloat));
  } else {
    o.take(a[7], 3, "out=(O_part, m, l)");
  }
  void* s = stream();
  const void *q = Q.data_ptr(), *k = K.data_ptr(), *v = V.data_ptr();
  float *N = data<float>(o.t[0]), *m = data<float>(o.t[1]), *l = data<float>(o.t[2]);
  const int kvh = (int)K.size(0);
  const Scratch scratch(Q, s);
  check(unlocked([&] {
    if (kvh != d.heads)                                // grouped queries: K, V hold fewer heads than Q
      return a2d_partial_fwd_gqa(&d, kvh, segs.n(), segs.ptr(), acc ? A2D_TILE_ACCUMULATE : 0, q, k, v, N, m, l, nullptr,
                                 0, s);
    if (acc) return a2d_partial_fwd_acc(&d, segs.n(), segs.ptr(), q, k, v, N, m, l, nullptr, 0, s);
    if (segs.given) return a2d_partial_fwd_seg(&d, segs.n(), segs.ptr(), q, k, v, N, m, l, nullptr, 0, s);
    return a2d_partial_fwd(&d, q, k, v, N, m, l, nullptr, 0, s);
  }));
  scratch.tell();
  return o.give();
}

// Q, K, V, q_off, kv_off, causal, scale, out, segments
PyObject* partial_fwd_norm(Args a) {
  const at::Tensor &Q = tensor(a[0], "Q"), &K = tensor(a[1], "K"), &V = tensor(a[2], "V");
  qkv(Q, K, V);
  const a2d_tile_desc d = descriptor(Q, K, V, a + 3, 0);
  const Segments segs(a[8]);
  Outputs o;
  if (a[7] == Py_None) {
    o.add(empty_like_shape(Q, Q.sizes(), Q.scalar_type()));
    o.add(empty_like_shape(Q, rows_shape(Q), at::kFloat));
  } else {
    o.take(a[7], 2, "out=(O_norm, lse)");
  }
  void* s = stream();
  const void *q = Q.data_ptr(), *k = K.data_ptr(), *v = V.data_ptr();
  void* O = o.t[0].data_ptr();
  float* lse = data<float>(o.t[1]);
  const int kvh = (int)K.size(0);
  const Scratch scratch(Q, s);
  check(unlocked([&] {
    if (kvh != d.heads)
      return a2d_partial_fwd_gqa(&d, kvh, segs.n(), segs.ptr(), A2D_TILE_NORMALISED, q, k, v, O, lse, nullptr, nullptr, 0,
                                 s);
    return a2d_partial_fwd_norm(&d, segs.n(), segs.ptr(), q, k, v, O, lse, nullptr, 0, s);
  }));
  scratch.tell();
  return o.give();
}

// Q, K, V, O, dO, lse: checked as the backward calls need them
struct Saved {
  const at::Tensor &Q, &K, &V, &O, &dO, &lse;
  explicit Saved(Args a)
      : Q(tensor(a[0], "Q")), K(tensor(a[1], "K")), V(tensor(a[2], "V")), O(tensor(a[3], "O")), dO(tensor(a[4], "dO")),
        lse(tensor(a[5], "lse")) {
    dev3(Q, "Q");
    dev3(K, "K");
    dev3(V, "V");
    dev3(O, "O");
    dev3(dO, "dO");
  }
  bool match() const {
    return O.sizes() == Q.sizes() && dO.sizes() == Q.sizes() && O.scalar_type() == Q.scalar_type() &&
           dO.scalar_type() == Q.scalar_type() && lse.sizes() == rows_shape(Q) && lse.scalar_type() == at::kFloat &&
           K.sizes() == V.sizes() && lse.is_contiguous();
  }
};
void gradients(Outputs* o, const Saved& x, PyObject* out) {
  if (out == Py_None) {
    o->add(empty_like_shape(x.Q, x.Q.sizes(), at::kFloat));
    o->add(empty_like_shape(x.Q, x.K.sizes(), at::kFloat));
    o->add(empty_like_shape(x.Q, x.K.sizes(), at::kFloat));
  } else {
    o->take(out, 3, "out=(dQ_part, dK_part, dV_part)");
  }
}

// Q, K, V, O, dO, lse, q_off, kv_off, causal, scale, out, workspace, segments, accumulate, ds_handover, split_groups
PyObject* partial_bwd(Args a) {
  const Saved x(a);
  if (!x.match()) fail(A2D_ERR_INVALID_ARG, "O, dO, lse do not match Q (lse: plain fp32 [heads][nq])");
  // (the library keeps dS at H = 128 only: below, no memory is taken for it)
  const bool keep_ds = truth(a[14]) && (a[11] != Py_None || x.Q.size(2) == 128), acc = truth(a[13]);
  a2d_tile_desc d = descriptor(x.Q, x.K, x.V, a + 6, keep_ds ? A2D_DESC_KEEP_DS : 0);
  d.lo = layout(x.O);
  d.ldo = layout(x.dO);
  const int kvh = (int)x.K.size(0);
  const bool split = truth(a[15]) && kvh != d.heads;
  at::Tensor ws;
  if (a[11] == Py_None) {
    const size_t need = split ? a2d_workspace_bytes(&d, A2D_OP_PARTIAL_BWD_SPLIT, kvh)
                              : a2d_workspace_bytes(&d, keep_ds ? A2D_OP_PARTIAL_BWD_DS : A2D_OP_PARTIAL_BWD, 0);
    ws = empty_like_shape(x.Q, {(int64_t)need}, at::kByte);
  } else {
    ws = tensor(a[11], "workspace");
  }
  if (acc && a[10] == Py_None) fail(A2D_ERR_INVALID_ARG, "accumulate needs out=(dQ_part, dK_part, dV_part)");
  Outputs o;
  gradients(&o, x, a[10]);
  const Segments segs(a[12]);
  void *s = stream(), *w = ws.data_ptr();
  const size_t wb = (size_t)ws.numel() * ws.element_size();
  const void *q = x.Q.data_ptr(), *k = x.K.data_ptr(), *v = x.V.data_ptr(), *O = x.O.data_ptr(), *g = x.dO.data_ptr();
  const float* lse = data<float>(x.lse);
  float *dq = data<float>(o.t[0]), *dk = data<float>(o.t[1]), *dv = data<float>(o.t[2]);
  const Scratch scratch(x.Q, s);
  check(unlocked([&] {
    if (kvh != d.heads)                                // dK_part, dV_part have K's heads
      return a2d_partial_bwd_gqa(&d, kvh, segs.n(), segs.ptr(),
                                 (acc ? A2D_TILE_ACCUMULATE : 0) | (split ? A2D_TILE_SPLIT_GROUPS : 0), q, k, v, O, g, lse,
                                 dq, dk, dv, w, wb, s);
    if (acc) return a2d_partial_bwd_acc(&d, segs.n(), segs.ptr(), q, k, v, O, g, lse, dq, dk, dv, w, wb, s);
    if (segs.given) return a2d_partial_bwd_seg(&d, segs.n(), segs.ptr(), q, k, v, O, g, lse, dq, dk, dv, w, wb, s);
    return a2d_partial_bwd(&d, q, k, v, O, g, lse, dq, dk, dv, w, wb, s);
  }));
  scratch.tell();
  return o.give();
}

// Q, K, V, O, dO, lse, q_off, kv_off, causal, scale, out
PyObject* partial_bwd_static(Args a) {
  const Saved x(a);
  if (!x.match() || x.K.size(0) != x.Q.size(0))
    fail(A2D_ERR_INVALID_ARG, "O, dO, lse do not match Q (lse: plain fp32 [heads][nq]); K, V need Q's head count");
  a2d_tile_desc d = descriptor(x.Q, x.K, x.V, a + 6, 0);
  d.lo = layout(x.O);
  d.ldo = layout(x.dO);
  Outputs o;
  gradients(&o, x, a[10]);
  void* s = stream();
  const Scratch scratch(s);
  check(unlocked([&] {
    return a2d_partial_bwd_static(&d, x.Q.data_ptr(), x.K.data_ptr(), x.V.data_ptr(), x.O.data_ptr(), x.dO.data_ptr(),
                                  data<float>(x.lse), data<float>(o.t[0]), data<float>(o.t[1]), data<float>(o.t[2]), s);
  }));
  scratch.tell();
  return o.give();
}

// the merged output and its layout: a contiguous tensor, or a [heads][nq][H] view written in place
struct Merged {
  bool strided;
  a2d_layout lo;
  explicit Merged(const at::Tensor& O, const char* name) : strided(!O.is_contiguous()), lo{0, 0} {
    if (strided) {
      dev3(O, name);
      lo = layout(O);
    }
  }
};

// O_parts, ms, ls, out_dtype, out
PyObject* fix(Args a) {
  const Parts N(a[0], "O_parts"), m(a[1], "ms"), l(a[2], "ls");
  const int k = N.k();
  if (k < 1 || m.k() != k || l.k() != k) fail(A2D_ERR_INVALID_ARG, "need k >= 1 partial triples");
  const at::Tensor& first = *N.t[0];
  Outputs o;
  if (a[4] == Py_None) {
    o.add(empty_like_shape(first, first.sizes(), dtype_arg(a[3])));
    o.add(empty_like_shape(first, rows_shape(first), at::kFloat));
  } else {
    o.take(a[4], 2, "out=(O, lse)", false);
  }
  for (const Parts* p : {&N, &m, &l}) p->all_plain("the partials and lse");
  plain(o.t[1], "the partials and lse");
  const Merged w(o.t[0], "O");
  const auto np = N.ptrs(), mp = m.ptrs(), lp = l.ptrs();
  const int H = (int)first.size(-1), dt = dtype_code(o.t[0].scalar_type());
  void *s = stream(), *O = o.t[0].data_ptr();
  float* lse = data<float>(o.t[1]);
  const int64_t rows = c10::multiply_integers(rows_shape(first));
  check(unlocked([&] {
    if (w.strided)
      return a2d_fix_strided(k, (int)o.t[0].size(0), (int)o.t[0].size(1), H, dt, np.data(), mp.data(), lp.data(), O, &w.lo,
                             lse, s);
    return a2d_fix(k, rows, H, dt, np.data(), mp.data(), lp.data(), O, lse, s);
  }));
  return o.give();
}

// O_norms, lses, out_dtype, out
PyObject* fix_norm(Args a) {
  const Parts N(a[0], "O_norms"), l(a[1], "lses");
  const int k = N.k();
  if (k < 1 || l.k() != k) fail(A2D_ERR_INVALID_ARG, "need k >= 1 normalised partials");
  const at::Tensor& first = *N.t[0];
  Outputs o;
  if (a[3] == Py_None) {
    o.add(empty_like_shape(first, first.sizes(), dtype_arg(a[2])));
    o.add(empty_like_shape(first, rows_shape(first), at::kFloat));
  } else {
    o.take(a[3], 2, "out=(O, lse)", false);
  }
  N.all_plain("the partials and lse");
  l.all_plain("the partials and lse");
  plain(o.t[1], "the partials and lse");
  const Merged w(o.t[0], "O");
  std::vector<const void*> np;
  for (auto* x : N.t) np.push_back(x->data_ptr());
  const auto lp = l.ptrs();
  const int H = (int)first.size(-1), di = dtype_code(first.scalar_type()), dt = dtype_code(o.t[0].scalar_type());
  void *s = stream(), *O = o.t[0].data_ptr();
  float* lse = data<float>(o.t[1]);
  const int64_t rows = c10::multiply_integers(rows_shape(first));
  check(unlocked([&] {
    if (w.strided)
      return a2d_fix_norm_strided(k, (int)o.t[0].size(0), (int)o.t[0].size(1), H, di, dt, np.data(), lp.data(), O, &w.lo,
                                  lse, s);
    return a2d_fix_norm(k, rows, H, di, dt, np.data(), lp.data(), O, lse, s);
  }));
  return o.give();
}

// O_parts, ms, ls, out
PyObject* attnfix(Args a) {
  const Parts N(a[0], "O_parts"), m(a[1], "ms"), l(a[2], "ls");
  const int k = N.k();
  if (k < 1 || m.k() != k || l.k() != k) fail(A2D_ERR_INVALID_ARG, "need k >= 1 partial triples");
  const at::Tensor& first = *N.t[0];
  Outputs o;
  if (a[3] == Py_None) {
    o.add(empty_like_shape(first, first.sizes(), at::kFloat));
    o.add(empty_like_shape(first, rows_shape(first), at::kFloat));
    o.add(empty_like_shape(first, rows_shape(first), at::kFloat));
  } else {
    o.take(a[3], 3, "the partials");
  }
  for (const Parts* p : {&N, &m, &l}) p->all_plain("the partials");
  const auto np = N.ptrs(), mp = m.ptrs(), lp = l.ptrs();
  const int H = (int)first.size(-1);
  const int64_t rows = c10::multiply_integers(rows_shape(first));
  void* s = stream();
  check(unlocked([&] {
    return a2d_attnfix(k, rows, H, np.data(), mp.data(), lp.data(), data<float>(o.t[0]), data<float>(o.t[1]),
                       data<float>(o.t[2]), s);
  }));
  return o.give();
}

// parts, out_dtype, out
PyObject* fix_bwd(Args a) {
  const Parts p(a[0], "parts");
  const int k = p.k();
  if (k < 1) fail(A2D_ERR_INVALID_ARG, "need k >= 1 partials");
  const at::Tensor& first = *p.t[0];
  Outputs o;
  if (a[2] == Py_None) {
    o.add(empty_like_shape(first, first.sizes(), dtype_arg(a[1])));
  } else {
    o.n = 1;
    o.given[0] = a[2];
    Py_INCREF(a[2]);
    o.t[0] = tensor(a[2], "out");
  }
  p.all_plain("the partials");
  const at::Tensor& out = o.t[0];
  const Merged w(out, "out");
  const auto pp = p.ptrs();
  const int dt = dtype_code(out.scalar_type());
  void* s = stream();
  check(unlocked([&] {
    if (w.strided)
      return a2d_fix_bwd_strided(k, (int)out.size(0), (int)out.size(1), (int)out.size(2), dt, pp.data(), out.data_ptr(),
                                 &w.lo, s);
    return a2d_fix_bwd(k, first.numel(), dt, pp.data(), out.data_ptr(), s);
  }));
  return o.one(0);
}

// the layout with its strides written out
a2d_layout full(const at::Tensor& t) {
  const a2d_layout l = layout(t);
  return l.row ? l : a2d_layout{t.size(1) * t.size(2), t.size(2)};
}

// ---- the whole grid.  Both return None when the batched path does not cover the problem.  Outputs have
// the strides of the inputs they belong to.
bool grid_problem(const at::Tensor& Q, const at::Tensor& K, const at::Tensor& V, const at::Tensor& O,
                  const at::Tensor& dO, Args a, a2d::GridProblem* p) {
  // a: side, causal, cyclic, scale
  for (const at::Tensor* t : {&Q, &K, &V, &O, &dO})
    if (!t->is_cuda() || t->dim() != 3 || t->stride(2) != 1 || t->scalar_type() != at::kBFloat16 ||
        (reinterpret_cast<uintptr_t>(t->data_ptr()) & 15))
      return false;
  if (K.sizes() != V.sizes() || K.size(1) != Q.size(1) || K.size(2) != Q.size(2) || O.sizes() != Q.sizes() ||
      dO.sizes() != Q.sizes() || Q.numel() == 0)
    return false;
  const int64_t side = integer(a[0]);
  if (side < 1 || side > A2D_MAX_PARTS || Q.size(0) > 65535 || Q.size(1) > (1 << 22) || Q.size(2) > 128) return false;
  *p = a2d::GridProblem{(int)Q.size(0), (int)K.size(0), (int)Q.size(1), (int)side, (int)Q.size(2), truth(a[1]), truth(a[2]),
                        scale_of(a[3], Q.size(2)), full(Q), full(K), full(V), full(O), full(dO), full(Q), full(K), full(V)};
  return !a2d::force_generic() && a2d::grid_supported(*p);
}
void hip_check(hipError_t e, const char* who) {
  if (e != hipSuccess) fail(A2D_ERR_HIP, std::string(who) + ": HIP error " + hipGetErrorString(e));
}

// Q, K, V, side, causal, cyclic, scale
PyObject* grid_forward(Args a) {
  const at::Tensor &Q = tensor(a[0], "Q"), &K = tensor(a[1], "K"), &V = tensor(a[2], "V");
  a2d::GridProblem p;
  if (!grid_problem(Q, K, V, Q, Q, a + 3, &p)) Py_RETURN_NONE;
  Outputs o;
  o.add(at::empty_like(Q));
  o.add(empty_like_shape(Q, rows_shape(Q), at::kFloat));
  if (o.t[0].stride(2) != 1) Py_RETURN_NONE;
  p.o = full(o.t[0]);
  const at::Tensor ws = empty_like_shape(Q, {(int64_t)a2d::grid_forward_bytes(p)}, at::kByte);
  hipStream_t s = static_cast<hipStream_t>(stream());
  hipError_t e;
  Py_BEGIN_ALLOW_THREADS
  e = a2d::grid_forward(p, Q.data_ptr(), K.data_ptr(), V.data_ptr(), o.t[0].data_ptr(), data<float>(o.t[1]), ws.data_ptr(), s);
  Py_END_ALLOW_THREADS
  hip_check(e, "grid_forward");
  return o.give();
}

// Q, K, V, O, dO, lse, side, causal, cyclic, scale
PyObject* grid_backward(Args a) {
  const at::Tensor &Q = tensor(a[0], "Q"), &K = tensor(a[1], "K"), &V = tensor(a[2], "V"), &O = tensor(a[3], "O"),
                   &dO = tensor(a[4], "dO"), &lse = tensor(a[5], "lse");
  a2d::GridProblem p;
  if (!grid_problem(Q, K, V, O, dO, a + 6, &p) || lse.scalar_type() != at::kFloat || !lse.is_cuda() ||
      lse.sizes() != rows_shape(Q) || !lse.is_contiguous())
    Py_RETURN_NONE;
  Outputs o;
  for (const at::Tensor* t : {&Q, &K, &V}) o.add(at::empty_like(*t));
  for (int i = 0; i < 3; ++i)
    if (o.t[i].stride(2) != 1) Py_RETURN_NONE;
  p.dq = full(o.t[0]);
  p.dk = full(o.t[1]);
  p.dv = full(o.t[2]);
  const at::Tensor ws = empty_like_shape(Q, {(int64_t)a2d::grid_backward_bytes(p)}, at::kByte);
  hipStream_t s = static_cast<hipStream_t>(stream());
  hipError_t e;
  Py_BEGIN_ALLOW_THREADS
  e = a2d::grid_backward(p, Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), dO.data_ptr(), data<float>(lse),
                         o.t[0].data_ptr(), o.t[1].data_ptr(), o.t[2].data_ptr(), ws.data_ptr(), s);
  Py_END_ALLOW_THREADS
  hip_check(e, "grid_backward");
  return o.give();
}

// ---- diagnostics: a call's route, from numbers alone
PyObject* route_dict(const a2d::Route& r) {
  PyObject* k = PyTuple_New(r.kernels);
  if (!k) throw PythonError();
  for (int i = 0; i < r.kernels; ++i) {
    PyObject* name = PyUnicode_FromString(r.kernel[i]);
    if (!name) {
      Py_DECREF(k);
      throw PythonError();
    }
    PyTuple_SET_ITEM(k, i, name);
  }
  PyObject* d = Py_BuildValue("{s:N,s:i,s:i,s:i,s:i,s:i,s:N,s:N}", "kernels", k, "rows", r.rows, "lanes", r.lanes, "keys", r.keys,
                              "parts_q", r.parts_q, "parts_kv", r.parts_kv, "phased", PyBool_FromLong(r.phased), "apart",
                              PyBool_FromLong(r.apart));
  if (!d) throw PythonError();
  return d;
}

// heads, kv_heads, nq, nkv, hdim, dtype, q_off, kv_off, causal, segments, flags, compute_units
PyObject* tile_route(Args a) {
  a2d_tile_desc d{};
  d.heads = (int32_t)integer(a[0]);
  d.nq = (int32_t)integer(a[2]);
  d.nkv = (int32_t)integer(a[3]);
  d.hdim = (int32_t)integer(a[4]);
  d.dtype = dtype_code(dtype_arg(a[5]));
  d.q_off = integer(a[6]);
  d.kv_off = integer(a[7]);
  d.causal = truth(a[8]);
  d.scale = scale_of(Py_None, d.hdim);
  const Segments segs(a[9]);
  a2d::Route r;
  check(a2d::tile_route(d, (int)integer(a[1]), segs.n(), segs.ptr(), (int)integer(a[10]), (int)integer(a[11]), &r));
  return route_dict(r);
}

// heads, kv_heads, seq, side, hdim, causal, cyclic, backward, compute_units
PyObject* grid_route(Args a) {
  const int64_t heads = integer(a[0]), kv_heads = integer(a[1]), seq = integer(a[2]), hdim = integer(a[4]);
  const a2d_layout plain{seq * hdim, hdim};
  const a2d::GridProblem p{(int)heads, (int)kv_heads, (int)seq, (int)integer(a[3]), (int)hdim, truth(a[5]), truth(a[6]),
                           scale_of(Py_None, hdim), plain, plain, plain, plain, plain, plain, plain, plain};
  a2d::Route r;
  if (!a2d::grid_route(p, truth(a[7]), (int)integer(a[8]), &r)) Py_RETURN_NONE;
  return route_dict(r);
}

template <PyObject* (*F)(Args), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != N) return PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", N, nargs);
  try {
    return F(args);
  } catch (const Error& e) {
    PyObject* v = g_error_class ? PyObject_CallFunction(g_error_class, "is", e.status, e.detail.c_str()) : nullptr;
    if (v) {
      PyErr_SetObject(g_error_class, v);
      Py_DECREF(v);
    } else if (!PyErr_Occurred()) {
      PyErr_SetString(PyExc_RuntimeError, e.detail.c_str());
    }
    return nullptr;
  } catch (const PythonError&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

PyObject* set_error_class(PyObject*, PyObject* cls) {
  Py_INCREF(cls);
  Py_XDECREF(g_error_class);
  g_error_class = cls;
  Py_RETURN_NONE;
}

#define A2D_ENTRY(NAME, N) \
  {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&entry<NAME, N>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    A2D_ENTRY(partial_fwd, 10),    A2D_ENTRY(partial_fwd_norm, 9), A2D_ENTRY(partial_bwd, 16),
    A2D_ENTRY(partial_bwd_static, 11), A2D_ENTRY(fix, 5),          A2D_ENTRY(fix_norm, 4),
    A2D_ENTRY(attnfix, 4),         A2D_ENTRY(fix_bwd, 3),          A2D_ENTRY(grid_forward, 7),
    A2D_ENTRY(grid_backward, 10),  A2D_ENTRY(tile_route, 12),      A2D_ENTRY(grid_route, 9),
    {"set_error_class", set_error_class, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&g_module); }
