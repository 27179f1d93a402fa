// The calls of the Python binding, from torch tensors to the C ABI (include/usp.h), as a CPython extension
// module.  Host code only: reads addresses, sizes, strides and types from the tensors, fills the
// descriptors, takes the current stream and calls libusp.so with the interpreter lock released.  The
// checks, their order and the errors are those that binding.py documents; a status other than USP_OK is
// returned as a number for binding.py to raise.
//
// What it is for: a call's kernels last 4 to 12 us on small shapes, and the same marshalling in Python and ctypes
// took the host 7.7 to 9 us per call of the FP8 and merge entry points and 13 to 26 us of the
// attention; 3.4 to 4.3 and 3.5 to 13.6 us here, most of it the launches.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <vector>

#include "usp.h"

namespace {

// ---- errors: a Python exception has been set -------------------------------------------------------
struct PyFailure {};

[[noreturn]] void fail(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw PyFailure();
}
void require(bool cond, const char* text) {   // the binding's assertions
  if (!cond) fail(PyExc_AssertionError, text);
}

constexpr int kUnsupportedDtype = -1000;      // status: binding.py names the dtype

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch tensor");
  return THPVariable_Unpack(o);
}
void* address(PyObject* o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }

int dtype_of(const at::Tensor& t) {
  switch (t.scalar_type()) {
    case at::kFloat: return USP_F32;
    case at::kBFloat16: return USP_BF16;
    case at::kByte: return USP_FP8_E4M3FN;
    default: return kUnsupportedDtype;
  }
}

// int(x) of a Python object
int64_t whole(PyObject* o) {
  if (PyLong_CheckExact(o)) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyFailure();
    return v;
  }
  PyObject* n = PyNumber_Long(o);
  if (!n) throw PyFailure();
  const long long v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw PyFailure();
  return v;
}

// a list or tuple (or any sequence) of objects that outlive the call
struct Sequence {
  PyObject* fast;
  explicit Sequence(PyObject* o) : fast(PySequence_Fast(o, "expected a sequence")) {
    if (!fast) throw PyFailure();
  }
  ~Sequence() { Py_DECREF(fast); }
  Sequence(const Sequence&) = delete;
  Sequence& operator=(const Sequence&) = delete;
  Py_ssize_t size() const { return PySequence_Fast_GET_SIZE(fast); }
  PyObject* operator[](Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(fast, i); }
};

// ---- streams: None = torch's current stream of the current device, else a handle or a stream object ----
PyObject *g_get_device = nullptr, *g_get_raw_stream = nullptr;

void* stream_handle(PyObject* o) {
  PyObject* h;
  if (o == Py_None) {
    PyObject* dev = PyObject_CallNoArgs(g_get_device);
    if (!dev) throw PyFailure();
    h = PyObject_CallOneArg(g_get_raw_stream, dev);
    Py_DECREF(dev);
  } else if (PyLong_Check(o)) {
    Py_INCREF(o);
    h = o;
  } else {
    h = PyObject_GetAttrString(o, "cuda_stream");
  }
  if (!h) throw PyFailure();
  void* p = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  if (!p && PyErr_Occurred()) throw PyFailure();
  return p;
}

template <class F>
int unlocked(F call) {
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = call();
  Py_END_ALLOW_THREADS
  return status;
}

// ---- entry points: positional arguments only, checked by binding.py's signatures -----------------------
// every C++ exception ends here
template <class F>
PyObject* guarded(Py_ssize_t given, Py_ssize_t want, F body) {
  if (given != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    return body();
  } catch (const PyFailure&) {
    return nullptr;
  } catch (...) {   // torch's exceptions as torch's own functions raise them: OutOfMemoryError, IndexError, ..
    torch::translate_exception_to_python(std::current_exception());
    return nullptr;
  }
}

// fp8_quant(x, q, scales, stream)
PyObject* fp8_quant(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 4, [&]() -> PyObject* {
    const at::Tensor& x = tensor(a[0]);
    const int dt = dtype_of(x);
    if (dt == kUnsupportedDtype) return PyLong_FromLong(dt);
    const int64_t rows = x.size(0), cols = x.size(1);
    const void* xp = x.data_ptr();
    uint8_t* q = (uint8_t*)address(a[1]);
    float* s = (float*)address(a[2]);
    void* st = stream_handle(a[3]);
    return PyLong_FromLong(unlocked([&] { return usp_fp8_quant(rows, cols, dt, xp, q, s, st); }));
  });
}

// fp8_dequant(q, scales, y, stream)
PyObject* fp8_dequant(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 4, [&]() -> PyObject* {
    const at::Tensor &q = tensor(a[0]), &y = tensor(a[2]);
    const int dt = dtype_of(y);
    if (dt == kUnsupportedDtype) return PyLong_FromLong(dt);
    const int64_t rows = q.size(0), cols = q.size(1);
    const uint8_t* qp = (const uint8_t*)q.data_ptr();
    const float* s = (const float*)address(a[1]);
    void* yp = y.data_ptr();
    void* st = stream_handle(a[3]);
    return PyLong_FromLong(unlocked([&] { return usp_fp8_dequant(rows, cols, dt, qp, s, yp, st); }));
  });
}

void row_map(PyObject* n, PyObject* src, PyObject* dst, usp_row_map* m) {
  const Sequence ns(n), ss(src), ds(dst);
  if (ns.size() < 4 || ss.size() < 4 || ds.size() < 4) fail(PyExc_IndexError, "a row map has four dimensions");
  for (int k = 0; k < 4; ++k) {
    m->n[k] = whole(ns[k]);
    m->src_stride[k] = whole(ss[k]);
    m->dst_stride[k] = whole(ds[k]);
  }
}

// fp8_quant_mapped(x, n, src_stride, dst_stride, cols, q, scales, stream)
PyObject* fp8_quant_mapped(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 8, [&]() -> PyObject* {
    const at::Tensor& x = tensor(a[0]);
    const int dt = dtype_of(x);
    if (dt == kUnsupportedDtype) return PyLong_FromLong(dt);
    usp_row_map m;
    row_map(a[1], a[2], a[3], &m);
    const int64_t cols = whole(a[4]);
    const void* xp = x.data_ptr();
    uint8_t* q = (uint8_t*)address(a[5]);
    float* s = (float*)address(a[6]);
    void* st = stream_handle(a[7]);
    return PyLong_FromLong(unlocked([&] { return usp_fp8_quant_mapped(&m, cols, dt, xp, q, s, st); }));
  });
}

// fp8_dequant_mapped(q, scales, n, src_stride, dst_stride, y, stream)
PyObject* fp8_dequant_mapped(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    const at::Tensor &q = tensor(a[0]), &y = tensor(a[5]);
    const int dt = dtype_of(y);
    if (dt == kUnsupportedDtype) return PyLong_FromLong(dt);
    usp_row_map m;
    row_map(a[2], a[3], a[4], &m);
    const int64_t cols = q.size(1);
    const uint8_t* qp = (const uint8_t*)q.data_ptr();
    const float* s = (const float*)address(a[1]);
    void* yp = y.data_ptr();
    void* st = stream_handle(a[6]);
    return PyLong_FromLong(unlocked([&] { return usp_fp8_dequant_mapped(&m, cols, dt, qp, s, yp, st); }));
  });
}

// lse_merge(o1, lse1, o2, lse2, o_out, lse_out, stream)
PyObject* lse_merge(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    const at::Tensor& o1 = tensor(a[0]);
    const int dt = dtype_of(o1);
    if (dt == kUnsupportedDtype) return PyLong_FromLong(dt);
    const int64_t d = o1.size(-1), rows = d ? o1.numel() / d : 0;
    const void *p1 = o1.data_ptr(), *p2 = address(a[2]);
    const float *l1 = (const float*)address(a[1]), *l2 = (const float*)address(a[3]);
    void* po = address(a[4]);
    float* lo = (float*)address(a[5]);
    void* st = stream_handle(a[6]);
    return PyLong_FromLong(unlocked([&] { return usp_lse_merge(rows, (int32_t)d, dt, p1, l1, p2, l2, po, lo, st); }));
  });
}

// ---- ring attention -------------------------------------------------------------------------------------
struct RingCall {
  usp_attn_desc desc;
  std::vector<int32_t> lens;
  std::vector<const void*> k, v, ks, vs, mask;
  bool has_v = false, has_ks = false, has_vs = false, has_mask = false;
  const void* q;
  void* out;
  float* lse;
};

bool addresses(PyObject* o, std::vector<const void*>* to) {
  if (o == Py_None) return false;
  const Sequence s(o);
  to->resize(s.size());
  for (Py_ssize_t i = 0; i < s.size(); ++i) (*to)[i] = address(s[i]);
  return true;
}

// q, k_chunks, v_chunks, k_scales, v_scales, key_mask, softmax_scale, flags, out, lse at a[0..9]; what
// make_attn_desc in binding.py does.  Status USP_OK or kUnsupportedDtype.
int describe(PyObject* const* a, RingCall* c) {
  const at::Tensor &q = tensor(a[0]), &out = tensor(a[8]);
  const Sequence ks(a[1]);
  usp_attn_desc& d = c->desc;
  if (q.dim() != 4) fail(PyExc_ValueError, "q must be [B, H, Sq, d]");
  d.B = (int32_t)q.size(0); d.H = (int32_t)q.size(1); d.Sq = (int32_t)q.size(2); d.d = (int32_t)q.size(3);
  d.n_chunks = (int32_t)ks.size();
  if (ks.size() == 0) fail(PyExc_IndexError, "k_chunks is empty");
  d.qo_dtype = dtype_of(q);
  d.kv_dtype = dtype_of(tensor(ks[0]));
  if (d.qo_dtype == kUnsupportedDtype || d.kv_dtype == kUnsupportedDtype) return kUnsupportedDtype;
  require(q.stride(3) == 1 && out.dim() == 4 && out.stride(3) == 1, "the head dimension of q and out must be contiguous");
  c->lens.resize(ks.size());
  const at::Tensor* first = nullptr;   // first chunk with keys
  bool dense = true;
  for (Py_ssize_t i = 0; i < ks.size(); ++i) {
    const at::Tensor& k = tensor(ks[i]);
    if (k.dim() != 4) fail(PyExc_ValueError, "KV chunks must be [B, H, Sc, d]");
    c->lens[i] = (int32_t)k.size(2);
    if (k.size(2) <= 0) continue;
    if (!first) first = &k;
    dense = dense && k.is_contiguous();
  }
  if (!dense)
    for (Py_ssize_t i = 0; i < ks.size(); ++i) {
      const at::Tensor& k = tensor(ks[i]);
      if (k.size(2) > 0) require(k.strides() == first->strides() && k.stride(3) == 1, "strided KV chunks must share one stride triple");
    }
  for (int i = 0; i < 3; ++i) {
    d.q_stride[i] = q.stride(i);
    d.o_stride[i] = out.stride(i);
    d.kv_stride[i] = dense || !first ? 0 : first->stride(i);   // all zero: every chunk dense for its own length
  }
  d.chunk_len = c->lens.data();
  d.softmax_scale = (float)PyFloat_AsDouble(a[6]);
  if (PyErr_Occurred()) throw PyFailure();
  d.flags = (uint32_t)whole(a[7]);
  c->q = q.data_ptr();
  addresses(a[1], &c->k);
  c->has_v = addresses(a[2], &c->v);
  c->has_ks = addresses(a[3], &c->ks);
  c->has_vs = addresses(a[4], &c->vs);
  c->has_mask = addresses(a[5], &c->mask);
  // (the library reads n_chunks entries of each)
  require((!c->has_v || c->v.size() >= c->k.size()) && (!c->has_ks || c->ks.size() >= c->k.size()) && (!c->has_vs || c->vs.size() >= c->k.size()) &&
              (!c->has_mask || c->mask.size() >= c->k.size()),
          "one entry per chunk is needed in v_chunks, k_scales, v_scales and key_mask");
  c->out = out.data_ptr();
  c->lse = (float*)address(a[9]);
  return USP_OK;
}

// ring_attn_fwd(q, k_chunks, v_chunks, k_scales, v_scales, key_mask, softmax_scale, flags, out, lse, workspace,
//               compute_stream, copy_stream): the status, or the workspace that was allocated for the call
PyObject* ring_attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 13, [&]() -> PyObject* {
    RingCall c;
    const int st = describe(a, &c);
    if (st != USP_OK) return PyLong_FromLong(st);
    void* ws = nullptr;
    size_t ws_bytes = 0;
    at::Tensor own;
    const size_t need = usp_ring_attn_workspace_bytes(&c.desc);
    if (need == (size_t)-1) return PyLong_FromLong(USP_ERR_INVALID_ARG);
    if (a[10] != Py_None) {
      const at::Tensor& w = tensor(a[10]);
      ws = w.data_ptr();
      ws_bytes = (size_t)w.numel() * w.element_size();
    } else if (need > 0) {
      own = at::empty({(int64_t)need}, tensor(a[0]).options().dtype(at::kByte).requires_grad(false));
      ws = own.data_ptr();
      ws_bytes = need;
    }
    void* cs = stream_handle(a[11]);
    void* xs = a[12] == Py_None ? nullptr : stream_handle(a[12]);
    const int status = unlocked([&] {
      return usp_ring_attn_fwd(&c.desc, c.q, c.k.data(), c.has_v ? c.v.data() : nullptr, c.has_ks ? (const float* const*)c.ks.data() : nullptr,
                               c.has_vs ? (const float* const*)c.vs.data() : nullptr,
                               c.has_mask ? (const uint8_t* const*)c.mask.data() : nullptr, c.out, c.lse, ws, ws_bytes, cs, xs);
    });
    if (status == USP_OK && own.defined()) return THPVariable_Wrap(own);
    return PyLong_FromLong(status);
  });
}

// ring_attn_fwd_noalloc(q, k_chunks, v_chunks, k_scales, v_scales, key_mask, softmax_scale, flags, out, lse, compute_stream)
PyObject* ring_attn_fwd_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&]() -> PyObject* {
    RingCall c;
    const int st = describe(a, &c);
    if (st != USP_OK) return PyLong_FromLong(st);
    void* cs = stream_handle(a[10]);
    return PyLong_FromLong(unlocked([&] {
      return usp_ring_attn_fwd_noalloc(&c.desc, c.q, c.k.data(), c.has_v ? c.v.data() : nullptr, c.has_ks ? (const float* const*)c.ks.data() : nullptr,
                                       c.has_vs ? (const float* const*)c.vs.data() : nullptr,
                                       c.has_mask ? (const uint8_t* const*)c.mask.data() : nullptr, c.out, c.lse, cs);
    }));
  });
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {METHOD(fp8_quant), METHOD(fp8_dequant), METHOD(fp8_quant_mapped), METHOD(fp8_dequant_mapped),
                          METHOD(lse_merge), METHOD(ring_attn_fwd), METHOD(ring_attn_fwd_noalloc), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_usp_calls", "usp entry points on torch tensors", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__usp_calls() {
  PyObject* c = PyImport_ImportModule("torch._C");
  if (!c) return nullptr;
  g_get_device = PyObject_GetAttrString(c, "_cuda_getDevice");
  g_get_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
  Py_DECREF(c);
  if (!g_get_device || !g_get_raw_stream) return nullptr;
  return PyModule_Create(&kModule);
}
