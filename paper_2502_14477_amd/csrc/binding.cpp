// Native half of the Python binding: argument marshalling from torch tensors to the C ABI (include/esa.h), output
// and workspace allocation.  Nothing here computes.
//
// A decode step is 40 us of kernels behind three calls, and marshalling each call through ctypes (25 converted
// arguments, a dozen tensor attribute look-ups and views) took 15-20 us of host time per call: the step ran at the
// host's pace, 72-78 us.  Here a call reads the tensors' sizes and strides directly and costs little more than the
// kernel launches behind it.  The functions take their arguments by position; the signatures with names and
// defaults are in binding.py.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/Allocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <map>
#include <string>
#include <utility>

#include "esa.h"

namespace {

PyObject* g_esa_error = nullptr;

// A Python exception is set; unwinds to the entry point.
struct Raised {};

[[noreturn]] void fail(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Raised();
}
[[noreturn]] void fail_esa(long code, const char* text) {
  PyObject* err = PyObject_CallFunction(g_esa_error, "ls", code, text);
  if (err) {
    PyErr_SetObject(g_esa_error, err);
    Py_DECREF(err);
  }
  throw Raised();
}
#define ESA_ASSERT(cond) \
  do {                   \
    if (!(cond)) fail(PyExc_AssertionError, #cond); \
  } while (0)

void check(int rc) {
  if (rc != ESA_OK) fail_esa(rc, esa_last_error());
}

// ---- arguments
const at::Tensor& tensor_of(PyObject* o) {
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch tensor");
  return THPVariable_Unpack(o);
}
const at::Tensor* tensor_or_none(PyObject* o) { return o == Py_None ? nullptr : &tensor_of(o); }
int64_t int_of(PyObject* o) {
  const int64_t v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Raised();
  return v;
}
int int32_of(PyObject* o) {
  const int64_t v = int_of(o);
  if (v != (int)v) fail(PyExc_OverflowError, "integer argument out of range");
  return (int)v;
}
double float_of(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Raised();
  return v;
}
bool true_of(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Raised();
  return v != 0;
}
int dtype_of(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return ESA_F32;
  if (t.scalar_type() == at::kBFloat16) return ESA_BF16;
  fail_esa(ESA_EUNSUPPORTED, (std::string("unsupported torch dtype ") + c10::toString(t.scalar_type())).c_str());
}
void* ptr(const at::Tensor& t) { return t.data_ptr(); }
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }

// A tensor with or without its leading batch dimension: sizes and strides of the `rank` dimensions behind it.
struct View {
  int64_t B, bs;          // batch entries, batch stride
  int64_t n[3], s[3];     // the other dimensions
  bool batched;
};
View view_of(const at::Tensor& t, int rank) {
  View v;
  const auto size = t.sizes(), stride = t.strides();
  if ((int)size.size() != rank && (int)size.size() != rank + 1)
    fail_esa(ESA_EINVAL, ("expected " + std::to_string(rank) + " or " + std::to_string(rank + 1) + " dimensions, got " +
                          std::to_string(size.size())).c_str());
  v.batched = (int)size.size() == rank + 1;
  const int o = v.batched ? 1 : 0;
  for (int i = 0; i < rank; ++i) {
    v.n[i] = size[i + o];
    v.s[i] = stride[i + o];
  }
  v.B = v.batched ? size[0] : 1;
  v.bs = v.batched ? stride[0] : v.n[0] * v.s[0];
  return v;
}

// ---- outputs and scratch
at::Tensor new_tensor(at::IntArrayRef shape, at::ScalarType dtype, const at::Device& dev) {
  return at::empty(shape, at::TensorOptions().dtype(dtype).device(dev));
}
PyObject* wrap(at::Tensor t) { return THPVariable_Wrap(std::move(t)); }
PyObject* wrap_or_none(const at::Tensor& t) {
  if (t.defined()) return THPVariable_Wrap(t);
  Py_RETURN_NONE;
}
PyObject* tuple_of(std::initializer_list<PyObject*> items) {
  PyObject* t = PyTuple_New((Py_ssize_t)items.size());
  Py_ssize_t i = 0;
  for (PyObject* o : items) {
    if (!o || !t) throw Raised();
    PyTuple_SET_ITEM(t, i++, o);
  }
  return t;
}
// [B, n...] or, without a batch dimension, [n...]
struct Shape {
  int64_t dim[4];
  int len = 0;
  Shape(bool batched, int64_t B, std::initializer_list<int64_t> rest) {
    if (batched) dim[len++] = B;
    for (int64_t v : rest) dim[len++] = v;
  }
  operator at::IntArrayRef() const { return at::IntArrayRef(dim, (size_t)len); }
};

// A call's scratch (256-byte aligned): a block of torch's allocator that the call gives back when its kernels are
// enqueued.  The allocator hands it out again in the order of the stream it was taken on, so calls on other streams, of
// other threads or in a graph under capture never share it with this one.
struct Scratch {
  c10::DataPtr block;
  void* p;
  size_t n;
};
Scratch scratch(size_t nbytes) {
  static c10::Allocator* const allocator = c10::GetAllocator(c10::DeviceType::CUDA);      // torch's name for the device type
  Scratch s;
  s.n = nbytes < 256 ? 256 : nbytes;
  s.block = allocator->allocate(s.n);
  s.p = s.block.get();
  ESA_ASSERT((uintptr_t)s.p % 256 == 0);
  return s;
}
// The scratch that attend_local hands over to attend_finish, one per device, grown on demand and kept (never destroyed: the
// allocator may be gone by the time statics are).  The two calls may run on different streams; a block given up for a
// larger one is reused only behind both.
Scratch handed_over(size_t nbytes, const at::Device& dev) {
  static auto& kept = *new std::map<int, at::Tensor>();
  at::Tensor& t = kept[dev.index()];
  if (!t.defined() || (size_t)t.numel() < nbytes) t = new_tensor({(int64_t)nbytes}, at::kByte, dev);
  t.record_stream(c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().unwrap());
  ESA_ASSERT((uintptr_t)t.data_ptr() % 256 == 0);
  Scratch s;
  s.p = t.data_ptr();
  s.n = (size_t)t.numel();
  return s;
}

void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// The library call itself runs without the interpreter lock.
template <typename F>
void launch(F&& f) {
  int rc;
  {
    PyThreadState* ts = PyEval_SaveThread();
    rc = f();
    PyEval_RestoreThread(ts);
  }
  check(rc);
}

#define ESA_ENTRY(name, n_args)                                                                    \
  PyObject* name##_impl(PyObject* const* a);                                                       \
  PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n) {                                    \
    HANDLE_TH_ERRORS                                                                               \
    if (n != (n_args)) {                                                                           \
      PyErr_SetString(PyExc_TypeError, #name ": wrong number of arguments");                       \
      return nullptr;                                                                              \
    }                                                                                              \
    try {                                                                                          \
      return name##_impl(a);                                                                       \
    } catch (const Raised&) {                                                                      \
      return nullptr;                                                                              \
    }                                                                                              \
    END_HANDLE_TH_ERRORS                                                                           \
  }                                                                                                \
  PyObject* name##_impl(PyObject* const* a)

// ---- one tensor of a compression: rows of x, and where they go
struct CompressIo {
  at::Tensor flat;      // set when the head dimensions had to be joined by torch
  View x;
  at::Tensor out_new;   // set when the output is allocated here
  View out;
  void *xp, *op;
};
CompressIo compress_io(const at::Tensor& x, int64_t d_in, int64_t d_c, const at::Tensor* out) {
  CompressIo io;
  const auto size = x.sizes(), stride = x.strides();
  const int nd = (int)size.size();
  io.xp = ptr(x);
  if (nd >= 1 && size[nd - 1] != d_in) {
    // [.., heads, d] joined to [.., heads * d]: without a copy where the heads of a token are contiguous
    if ((nd == 3 || nd == 4) && stride[nd - 2] == size[nd - 1] * stride[nd - 1]) {
      io.x.batched = nd == 4;
      const int o = io.x.batched ? 1 : 0;
      io.x.n[0] = size[o];
      io.x.s[0] = stride[o];
      io.x.n[1] = size[nd - 2] * size[nd - 1];
      io.x.s[1] = stride[nd - 1];
      io.x.B = io.x.batched ? size[0] : 1;
      io.x.bs = io.x.batched ? stride[0] : io.x.n[0] * io.x.s[0];
    } else {
      io.flat = x.flatten(-2);
      io.xp = ptr(io.flat);
      io.x = view_of(io.flat, 2);
    }
  } else {
    io.x = view_of(x, 2);
  }
  ESA_ASSERT(io.x.n[1] == d_in && io.x.s[1] == 1);
  if (out) {
    io.out = view_of(*out, 2);
    io.op = ptr(*out);
    ESA_ASSERT(io.out.B == io.x.B && io.out.n[0] == io.x.n[0] && io.out.n[1] == d_c && io.out.s[1] == 1 && out->scalar_type() == x.scalar_type());
  } else {
    io.out_new = new_tensor(Shape(io.x.batched, io.x.B, {io.x.n[0], d_c}), x.scalar_type(), x.device());
    io.out = view_of(io.out_new, 2);
    io.op = ptr(io.out_new);
  }
  return io;
}
// What the call returns for it: the caller's rows (a batch dimension added or taken as the input has one).
PyObject* compress_result(const CompressIo& io, const at::Tensor* out, PyObject* out_obj) {
  if (!out) return wrap(io.out_new);
  if (io.x.batched == io.out.batched) {
    Py_INCREF(out_obj);
    return out_obj;
  }
  return wrap(io.x.batched ? out->unsqueeze(0) : out->select(0, 0));
}

// x, W, w_layout, d_in, d_c, bias, out
ESA_ENTRY(compress, 7) {
  const at::Tensor &x = tensor_of(a[0]), &W = tensor_of(a[1]);
  const int layout = int32_of(a[2]);
  const int64_t d_in = int_of(a[3]), d_c = int_of(a[4]);
  const at::Tensor *bias = tensor_or_none(a[5]), *out = tensor_or_none(a[6]);
  ESA_ASSERT(W.is_contiguous() && W.scalar_type() == x.scalar_type());
  const int dt = dtype_of(x);
  const CompressIo io = compress_io(x, d_in, d_c, out);
  void *st = stream(), *wp = ptr(W), *bp = ptr(bias);
  launch([&] {
    return esa_compress(io.xp, io.x.n[0], d_in, io.x.s[0], wp, layout, bp, (int)d_c, io.op, io.out.s[0], dt, (int)io.x.B, io.x.bs,
                        io.out.bs, st);
  });
  return compress_result(io, out, a[6]);
}

// xq, Wq, d_in_q, xk, Wk, d_in_k, w_layout, d_c, bias_q, bias_k, out_q, out_k
ESA_ENTRY(compress_qk, 12) {
  const at::Tensor &xq = tensor_of(a[0]), &Wq = tensor_of(a[1]), &xk = tensor_of(a[3]), &Wk = tensor_of(a[4]);
  const int64_t dq = int_of(a[2]), dk = int_of(a[5]), d_c = int_of(a[7]);
  const int layout = int32_of(a[6]);
  const at::Tensor *bq = tensor_or_none(a[8]), *bk = tensor_or_none(a[9]), *oq = tensor_or_none(a[10]), *ok = tensor_or_none(a[11]);
  ESA_ASSERT(Wq.is_contiguous() && Wk.is_contiguous() && Wq.scalar_type() == xq.scalar_type() && Wk.scalar_type() == xk.scalar_type());
  const CompressIo q = compress_io(xq, dq, d_c, oq), k = compress_io(xk, dk, d_c, ok);
  ESA_ASSERT(q.x.B == k.x.B && q.x.n[0] == k.x.n[0] && xq.scalar_type() == xk.scalar_type());
  const int dt = dtype_of(xq);
  void *st = stream(), *wq = ptr(Wq), *wk = ptr(Wk), *bqp = ptr(bq), *bkp = ptr(bk);
  launch([&] {
    return esa_compress_qk(q.xp, dq, q.x.s[0], wq, bqp, q.op, q.out.s[0], q.x.bs, q.out.bs, k.xp, dk, k.x.s[0], wk, bkp, k.op,
                           k.out.s[0], k.x.bs, k.out.bs, q.x.n[0], (int)d_c, layout, dt, (int)q.x.B, st);
  });
  return tuple_of({compress_result(q, oq, a[10]), compress_result(k, ok, a[11])});
}

void score_args_ok(const at::Tensor& qc, const View& q, const at::Tensor& kc, const View& k) {
  ESA_ASSERT(k.B == q.B && k.n[1] == q.n[1] && q.s[1] == 1 && k.s[1] == 1);
  ESA_ASSERT(q.s[0] == q.n[1] && k.s[0] == q.n[1] && kc.scalar_type() == qc.scalar_type());
}

// qc, kc_cache, m_lo, m_hi, eps, out
ESA_ENTRY(score, 6) {
  const at::Tensor &qc = tensor_of(a[0]), &kc = tensor_of(a[1]);
  const int64_t m_lo = int_of(a[2]), m_hi = int_of(a[3]), n = m_hi - m_lo;
  const int eps = int32_of(a[4]);
  const at::Tensor* out = tensor_or_none(a[5]);
  const View q = view_of(qc, 2), k = view_of(kc, 2);
  score_args_ok(qc, q, kc, k);
  at::Tensor fresh;
  View sv;
  if (out) {
    sv = view_of(*out, 1);
  } else {
    fresh = new_tensor(Shape(q.batched, q.B, {n > 0 ? n : 0}), at::kFloat, qc.device());
    sv = view_of(fresh, 1);
  }
  const int dt = dtype_of(qc), l_c = (int)q.n[0], B = (int)q.B;
  const Scratch ws = scratch(esa_score_workspace_bytes(l_c, n, eps, B));
  void *st = stream(), *qp = ptr(qc), *kp = ptr(kc), *sp = out ? ptr(*out) : ptr(fresh), *wp = ws.p;
  const size_t wn = ws.n;
  launch([&] {
    return esa_score(qp, l_c, kp, m_lo, m_hi, (int)q.n[1], eps, (float*)sp, dt, B, q.bs, k.bs, B > 1 ? sv.bs : (n > 1 ? n : 1), wp, wn, st);
  });
  if (!out) return wrap(std::move(fresh));
  if (q.batched == sv.batched) {
    Py_INCREF(a[5]);
    return a[5];
  }
  return wrap(q.batched ? out->unsqueeze(0) : out->select(0, 0));
}

// score, k, base
ESA_ENTRY(select_topk, 3) {
  const at::Tensor& score = tensor_of(a[0]);
  const int k = int32_of(a[1]);
  const int64_t base = int_of(a[2]);
  const View s = view_of(score, 1);
  const int64_t n = s.n[0], k_eff = k < n ? k : n;
  ESA_ASSERT(score.scalar_type() == at::kFloat && (n == 0 || s.s[0] == 1));
  at::Tensor idx = new_tensor(Shape(s.batched, s.B, {k_eff}), at::kInt, score.device());
  const Scratch ws = scratch(esa_select_topk_workspace_bytes(n, k, (int)s.B));
  void *st = stream(), *sp = ptr(score), *ip = ptr(idx), *wp = ws.p;
  const size_t wn = ws.n;
  launch([&] {
    return esa_select_topk((const float*)sp, n, k, base, (int32_t*)ip, (int)s.B, s.B > 1 ? s.bs : (n > 1 ? n : 1),
                           k_eff > 1 ? k_eff : 1, wp, wn, st);
  });
  return wrap(std::move(idx));
}

// score, k, base, out
ESA_ENTRY(select_topk_static, 4) {
  const at::Tensor& score = tensor_of(a[0]);
  const int k = int32_of(a[1]);
  const int64_t base = int_of(a[2]);
  const at::Tensor* out = tensor_or_none(a[3]);
  const View s = view_of(score, 1);
  const int64_t n = s.n[0], k_eff = k < n ? k : n;
  ESA_ASSERT(score.scalar_type() == at::kFloat && (n == 0 || s.s[0] == 1));
  at::Tensor fresh;
  View iv;
  if (out) {
    iv = view_of(*out, 1);
    ESA_ASSERT(out->scalar_type() == at::kInt && iv.B == s.B && iv.n[0] == k_eff && out->is_contiguous());
  } else {
    fresh = new_tensor(Shape(s.batched, s.B, {k_eff}), at::kInt, score.device());
  }
  void *st = stream(), *sp = ptr(score), *ip = out ? ptr(*out) : ptr(fresh);
  launch([&] {
    return esa_select_topk_static((const float*)sp, n, k, base, (int32_t*)ip, (int)s.B, s.B > 1 ? s.bs : (n > 1 ? n : 1),
                                  k_eff > 1 ? k_eff : 1, st);
  });
  if (!out) return wrap(std::move(fresh));
  if (s.batched == iv.batched) {
    Py_INCREF(a[3]);
    return a[3];
  }
  return wrap(s.batched ? out->unsqueeze(0) : out->select(0, 0));
}

// The key and value caches: [B?, S, h_kv, d], heads contiguous, same strides and type.
View caches_of(const at::Tensor& k, const at::Tensor& v, bool same_shape) {
  const View kv = view_of(k, 3), vv = view_of(v, 3);
  ESA_ASSERT(kv.s[2] == 1 && kv.s[1] == kv.n[2] && v.scalar_type() == k.scalar_type());
  ESA_ASSERT(vv.s[0] == kv.s[0] && vv.s[1] == kv.s[1] && vv.s[2] == kv.s[2] && vv.bs == kv.bs);
  ESA_ASSERT(!same_shape || (vv.B == kv.B && vv.n[0] == kv.n[0] && vv.n[1] == kv.n[1] && vv.n[2] == kv.n[2]));
  return kv;
}

// qc, kc_cache, m_lo, m_hi, k, k_cache, v_cache, eps
ESA_ENTRY(score_select_gather, 8) {
  const at::Tensor &qc = tensor_of(a[0]), &kc = tensor_of(a[1]);
  const int64_t m_lo = int_of(a[2]), m_hi = int_of(a[3]), n = m_hi - m_lo;
  const int k = int32_of(a[4]), eps = int32_of(a[7]);
  const at::Tensor *kcache = tensor_or_none(a[5]), *vcache = tensor_or_none(a[6]);
  const View q = view_of(qc, 2), kv = view_of(kc, 2);
  score_args_ok(qc, q, kc, kv);
  const int64_t n0 = n > 0 ? n : 0, k_eff = k < n0 ? k : n0;
  const int B = (int)q.B, l_c = (int)q.n[0], dt = dtype_of(qc);
  const at::Device dev = qc.device();
  at::Tensor score, idx, ks, vs;
  if (n > k) score = new_tensor(Shape(q.batched, q.B, {n0}), at::kFloat, dev);
  idx = new_tensor(Shape(q.batched, q.B, {k_eff}), at::kInt, dev);
  View c = {};
  if (kcache) {
    ESA_ASSERT(vcache != nullptr);
    c = caches_of(*kcache, *vcache, true);
    ESA_ASSERT(c.B == q.B && kcache->scalar_type() == qc.scalar_type() && kcache->is_cuda());
    ks = new_tensor(Shape(q.batched, q.B, {k_eff, c.n[1], c.n[2]}), kcache->scalar_type(), dev);
    vs = new_tensor(Shape(q.batched, q.B, {k_eff, c.n[1], c.n[2]}), kcache->scalar_type(), dev);
  }
  const Scratch ws = scratch(esa_score_select_gather_workspace_bytes(l_c, n, eps, k, B));
  void *st = stream(), *qp = ptr(qc), *kp = ptr(kc), *sp = score.defined() ? ptr(score) : nullptr, *ip = ptr(idx), *wp = ws.p;
  void *kcp = ptr(kcache), *vcp = kcache ? ptr(*vcache) : nullptr, *ksp = kcache ? ptr(ks) : nullptr, *vsp = kcache ? ptr(vs) : nullptr;
  const size_t wn = ws.n;
  launch([&] {
    return esa_score_select_gather(qp, l_c, kp, m_lo, m_hi, (int)q.n[1], eps, k, (float*)sp, (int32_t*)ip, kcp, vcp, c.s[0],
                                   (int)c.n[1], (int)c.n[2], ksp, vsp, dt, B, q.bs, kv.bs, n > 1 ? n : 1, k_eff > 1 ? k_eff : 1,
                                   kcache ? c.bs : 0, kcache ? k_eff * c.n[1] * c.n[2] : 0, wp, wn, st);
  });
  return tuple_of({wrap_or_none(score), wrap(std::move(idx)), wrap_or_none(ks), wrap_or_none(vs)});
}

// Device address of a KV cache: a GPU tensor, or pinned host memory (the KV cache offloaded to the host as in
// Appendix B; the gather kernel then fetches the selected rows over the host link).
void* cache_ptr(const at::Tensor& t) {
  if (t.is_cuda()) return ptr(t);
  if (!t.is_pinned())
    fail(PyExc_ValueError, "a KV cache in host memory must be pinned (torch's pin_memory), pageable memory is not addressable by the GPU");
  void* dptr = nullptr;
  const hipError_t e = hipHostGetDevicePointer(&dptr, ptr(t), 0);
  if (e != hipSuccess || !dptr)
    fail_esa(ESA_EHIP, ("hipHostGetDevicePointer failed (" + std::to_string((int)e) + "): the pinned cache is not mapped into the GPU").c_str());
  return dptr;
}

// k_cache, v_cache, idx
ESA_ENTRY(gather_kv, 3) {
  const at::Tensor &k = tensor_of(a[0]), &v = tensor_of(a[1]), &idx = tensor_of(a[2]);
  const View c = caches_of(k, v, true), i = view_of(idx, 1);
  const int64_t n_sel = i.n[0];
  ESA_ASSERT(idx.scalar_type() == at::kInt && i.B == c.B && (n_sel == 0 || i.s[0] == 1));
  at::Tensor ks = new_tensor(Shape(c.batched, c.B, {n_sel, c.n[1], c.n[2]}), k.scalar_type(), idx.device());
  at::Tensor vs = new_tensor(Shape(c.batched, c.B, {n_sel, c.n[1], c.n[2]}), k.scalar_type(), idx.device());
  const int dt = dtype_of(k);
  void *st = stream(), *kp = cache_ptr(k), *vp = cache_ptr(v), *ip = ptr(idx), *ksp = ptr(ks), *vsp = ptr(vs);
  launch([&] {
    return esa_gather_kv(kp, vp, c.s[0], (const int32_t*)ip, (int)n_sel, (int)c.n[1], (int)c.n[2], ksp, vsp, dt, (int)c.B, c.bs,
                         c.B > 1 ? i.bs : (n_sel > 1 ? n_sel : 1), n_sel * c.n[1] * c.n[2], st);
  });
  return tuple_of({wrap(std::move(ks)), wrap(std::move(vs))});
}

// Queries, caches and outputs common to the attention calls.
struct AttendIo {
  View q, c;
  int l_c, h, h_kv, d, B, dt;
  float scale;
  at::Tensor out, lse;
  void *qp, *kp, *vp;
};
AttendIo attend_io(PyObject* q_obj, PyObject* k_obj, PyObject* v_obj, int64_t t0, PyObject* scale, PyObject* want_lse) {
  const at::Tensor &q = tensor_of(q_obj), &k = tensor_of(k_obj), &v = tensor_of(v_obj);
  AttendIo io;
  io.q = view_of(q, 3);
  io.c = caches_of(k, v, false);
  ESA_ASSERT(q.is_contiguous());
  io.B = (int)io.q.B;
  io.l_c = (int)io.q.n[0];
  io.h = (int)io.q.n[1];
  io.d = (int)io.q.n[2];
  io.h_kv = (int)io.c.n[1];
  // what the kernels address with the queries' sizes: both caches have their batch, head size and type
  ESA_ASSERT(io.c.n[2] == io.q.n[2] && io.c.B == io.q.B && k.scalar_type() == q.scalar_type());
  const View vv = view_of(v, 3);
  ESA_ASSERT(vv.B == io.c.B && vv.n[1] == io.c.n[1] && vv.n[2] == io.c.n[2]);
  if (io.c.n[0] < t0 + io.l_c || vv.n[0] < t0 + io.l_c) fail(PyExc_AssertionError, "the cache must already hold the current tokens");
  io.dt = dtype_of(q);
  io.scale = scale == Py_None ? (float)(1.0 / std::sqrt((double)io.d)) : (float)float_of(scale);
  if (want_lse) {       // null: the call has no outputs
    io.out = new_tensor(q.sizes(), q.scalar_type(), q.device());
    if (true_of(want_lse)) io.lse = new_tensor(Shape(io.q.batched, io.q.B, {io.l_c, io.h}), at::kFloat, q.device());
  }
  io.qp = ptr(q);
  io.kp = ptr(k);
  io.vp = ptr(v);
  return io;
}
PyObject* attend_result(AttendIo& io) {
  if (!io.lse.defined()) return wrap(std::move(io.out));
  return tuple_of({wrap(std::move(io.out)), wrap(std::move(io.lse))});
}
int64_t row_elems(const AttendIo& io) { return (int64_t)io.l_c * io.h * io.d; }
float* lse_ptr(const AttendIo& io) { return io.lse.defined() ? (float*)ptr(io.lse) : nullptr; }

// Gathered rows [B?, n_sel, h_kv, d]
struct Gathered {
  void *k = nullptr, *v = nullptr;
  int n_sel = 0;
  int64_t bs = 0;
};
Gathered gathered_of(PyObject* k_obj, PyObject* v_obj, const AttendIo& io) {
  Gathered g;
  const at::Tensor* k = tensor_or_none(k_obj);
  if (!k || k->numel() == 0) return g;
  const at::Tensor& v = tensor_of(v_obj);
  const View kv = view_of(*k, 3), vv = view_of(v, 3);
  ESA_ASSERT(k->is_contiguous() && v.is_contiguous());
  ESA_ASSERT(kv.B == vv.B && kv.n[0] == vv.n[0] && kv.n[1] == vv.n[1] && kv.n[2] == vv.n[2]);
  ESA_ASSERT(kv.B == io.B && kv.n[1] == io.h_kv && kv.n[2] == io.d && dtype_of(*k) == io.dt && dtype_of(v) == io.dt);
  g.k = ptr(*k);
  g.v = ptr(v);
  g.n_sel = (int)kv.n[0];
  g.bs = kv.bs;
  return g;
}

// q, k_cache, v_cache, t0, l_i, l_l, idx, scale, return_lse
ESA_ENTRY(attend_indexed, 9) {
  const int64_t t0 = int_of(a[3]), l_i = int_of(a[4]), l_l = int_of(a[5]);
  AttendIo io = attend_io(a[0], a[1], a[2], t0, a[7], a[8]);
  const at::Tensor* idx = tensor_or_none(a[6]);
  int n_sel = 0;
  int64_t idx_bs = 0;
  void* ip = nullptr;
  if (idx && idx->numel() > 0) {
    const View i = view_of(*idx, 1);
    ESA_ASSERT(idx->scalar_type() == at::kInt && i.s[0] == 1 && i.B == io.B);
    n_sel = (int)i.n[0];
    idx_bs = i.bs;
    ip = ptr(*idx);
  }
  const Scratch ws = scratch(esa_attend_indexed_workspace_bytes(io.l_c, io.h, io.h_kv, io.d, io.dt, io.B, n_sel));
  void *st = stream(), *wp = ws.p, *op = ptr(io.out);
  const size_t wn = ws.n;
  launch([&] {
    return esa_attend_indexed(io.qp, io.l_c, io.h, io.h_kv, io.d, io.kp, io.vp, io.c.s[0], t0, l_i, l_l, (const int32_t*)ip, n_sel,
                              idx_bs, io.scale, op, lse_ptr(io), io.dt, io.B, io.q.bs, io.c.bs, row_elems(io), wp, wn, st);
  });
  return attend_result(io);
}

// q, k_cache, v_cache, t0, l_i, l_l, k_sel, v_sel, w, rope_base, scale, return_lse
ESA_ENTRY(attend_reencoded, 12) {
  const int64_t t0 = int_of(a[3]), l_i = int_of(a[4]), l_l = int_of(a[5]);
  AttendIo io = attend_io(a[0], a[1], a[2], t0, a[10], a[11]);
  const Gathered g = gathered_of(a[6], a[7], io);
  const double w = float_of(a[8]), base = float_of(a[9]);
  const Scratch ws = scratch(esa_attend_reencoded_workspace_bytes(io.l_c, io.h, io.h_kv, io.d, io.dt, io.B, l_l));
  void *st = stream(), *wp = ws.p, *op = ptr(io.out);
  const size_t wn = ws.n;
  launch([&] {
    return esa_attend_reencoded(io.qp, io.l_c, io.h, io.h_kv, io.d, io.kp, io.vp, io.c.s[0], t0, l_i, l_l, g.k, g.v, g.n_sel, io.scale,
                                w, base, op, lse_ptr(io), io.dt, io.B, io.q.bs, io.c.bs, g.bs, row_elems(io), wp, wn, st);
  });
  return attend_result(io);
}

// q, k_cache, v_cache, t0, l_i, l_l, k_sel, v_sel, scale, return_lse, split (None: the one-call form)
ESA_ENTRY(attend, 11) {
  const int64_t t0 = int_of(a[3]), l_i = int_of(a[4]), l_l = int_of(a[5]);
  AttendIo io = attend_io(a[0], a[1], a[2], t0, a[8], a[9]);
  const Gathered g = gathered_of(a[6], a[7], io);
  const bool one_call = a[10] == Py_None;
  const int split = one_call ? 0 : int32_of(a[10]);
  const size_t need = esa_attend_workspace_bytes(io.l_c, io.h, io.h_kv, io.d, io.dt, io.B);
  const Scratch ws = one_call ? scratch(need) : handed_over(need, io.out.device());
  void *st = stream(), *wp = ws.p, *op = ptr(io.out);
  const size_t wn = ws.n;
  launch([&] {
    if (one_call)
      return esa_attend(io.qp, io.l_c, io.h, io.h_kv, io.d, io.kp, io.vp, io.c.s[0], t0, l_i, l_l, g.k, g.v, g.n_sel, io.scale, op,
                        lse_ptr(io), io.dt, io.B, io.q.bs, io.c.bs, g.bs, row_elems(io), wp, wn, st);
    return esa_attend_finish(io.qp, io.l_c, io.h, io.h_kv, io.d, io.kp, io.vp, io.c.s[0], t0, l_i, l_l, g.k, g.v, g.n_sel, io.scale,
                             split, op, lse_ptr(io), io.dt, io.B, io.q.bs, io.c.bs, g.bs, row_elems(io), wp, wn, st);
  });
  return attend_result(io);
}

// q, k_cache, v_cache, t0, l_i, l_l, scale, split
ESA_ENTRY(attend_local, 8) {
  const int64_t t0 = int_of(a[3]), l_i = int_of(a[4]), l_l = int_of(a[5]);
  const AttendIo io = attend_io(a[0], a[1], a[2], t0, a[6], nullptr);
  const int split = int32_of(a[7]);
  const Scratch ws = handed_over(esa_attend_workspace_bytes(io.l_c, io.h, io.h_kv, io.d, io.dt, io.B), tensor_of(a[0]).device());
  void *st = stream(), *wp = ws.p;
  const size_t wn = ws.n;
  launch([&] {
    return esa_attend_local(io.qp, io.l_c, io.h, io.h_kv, io.d, io.kp, io.vp, io.c.s[0], t0, l_i, l_l, io.scale, split, io.dt, io.B,
                            io.q.bs, io.c.bs, wp, wn, st);
  });
  Py_RETURN_NONE;
}

// x, pos0, pos_step, base, out
ESA_ENTRY(rope, 5) {
  const at::Tensor& x = tensor_of(a[0]);
  const double pos0 = float_of(a[1]), step = float_of(a[2]), base = float_of(a[3]);
  const at::Tensor* out = tensor_or_none(a[4]);
  const View xv = view_of(x, 3);
  at::Tensor fresh;
  View ov;
  if (out) {
    ov = view_of(*out, 3);
    ESA_ASSERT(ov.B == xv.B && ov.n[0] == xv.n[0] && ov.n[1] == xv.n[1] && ov.n[2] == xv.n[2] && out->scalar_type() == x.scalar_type());
  } else {
    fresh = new_tensor(Shape(xv.batched, xv.B, {xv.n[0], xv.n[1], xv.n[2]}), x.scalar_type(), x.device());
    ov = view_of(fresh, 3);
  }
  ESA_ASSERT(xv.s[2] == 1 && xv.s[1] == xv.n[2] && ov.s[2] == 1 && ov.s[1] == xv.n[2]);
  const int dt = dtype_of(x);
  void *st = stream(), *xp = ptr(x), *op = out ? ptr(*out) : ptr(fresh);
  launch([&] {
    return esa_rope(xp, xv.n[0], (int)xv.n[1], (int)xv.n[2], xv.s[0], pos0, step, base, op, ov.s[0], dt, (int)xv.B, xv.bs, ov.bs, st);
  });
  if (!out) return wrap(std::move(fresh));
  Py_INCREF(a[4]);
  return a[4];
}

// t0, l_i, l_l
ESA_ENTRY(segments, 3) {
  int64_t i_end = 0, l_start = 0;
  check(esa_segments(int_of(a[0]), int_of(a[1]), int_of(a[2]), &i_end, &l_start));
  return tuple_of({PyLong_FromLongLong(i_end), PyLong_FromLongLong(l_start)});
}

// the exception class for libesa's errors
ESA_ENTRY(set_error_class, 1) {
  Py_XDECREF(g_esa_error);
  Py_INCREF(a[0]);
  g_esa_error = a[0];
  Py_RETURN_NONE;
}

#define ESA_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ESA_METHOD(compress), ESA_METHOD(compress_qk), ESA_METHOD(score), ESA_METHOD(select_topk),
                         ESA_METHOD(select_topk_static), ESA_METHOD(score_select_gather), ESA_METHOD(gather_kv),
                         ESA_METHOD(attend_indexed), ESA_METHOD(attend_reencoded), ESA_METHOD(attend), ESA_METHOD(attend_local),
                         ESA_METHOD(rope), ESA_METHOD(segments), ESA_METHOD(set_error_class), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "argument marshalling for libesa", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
