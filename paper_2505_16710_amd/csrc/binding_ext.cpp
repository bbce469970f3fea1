// Native half of the Python binding (module _seco_ext): takes torch tensors, builds the seco_desc, allocates the
// outputs and workspaces the caller did not supply and calls the C ABI on the current HIP stream.
//
// A call through ctypes (descriptor fields, stride arrays, torch.empty and pointer objects, all in Python) costs
// 13 - 20 us of host time, more than most of the kernels of a short chunk; this one costs 3 - 5 us, of which the
// kernel launch is the largest part.  The entry points are looked up in the library that the Python side has
// loaded (seco_init gets its path), so there is one copy of libseco_hip.so in the process.
#include "binding_common.h"

namespace {

using namespace seco_ext;

seco_desc chunk_desc(const Tensor& q, const Tensor& k, PyObject* q_start, PyObject* scale, const Tensor& o, const Tensor* g) {
  seco_desc d;
  strides3(q, d.q_stride);
  strides3(o, d.o_stride);
  strides3(k, d.kv_stride);
  strides3(g ? *g : k, d.g_stride);
  d.batch = (int32_t)q.size(0);
  d.n_q_heads = (int32_t)q.size(1);
  d.n_kv_heads = (int32_t)k.size(1);
  d.head_dim = (int32_t)q.size(3);
  d.chunk_len = (int32_t)q.size(2);
  d.q_start = int32(q_start);
  d.dtype = dtype_code(q);
  d.softmax_scale = (float)real(scale);
  return d;
}
seco_desc rows_desc(const Tensor& t, int64_t rows, int64_t q_start, int dtype) {   // strides: left to the caller
  seco_desc d;
  strides3(t, d.q_stride);
  d.batch = (int32_t)t.size(0);
  d.n_q_heads = d.n_kv_heads = (int32_t)t.size(1);
  d.head_dim = (int32_t)t.size(3);
  d.chunk_len = (int32_t)rows;
  d.q_start = (int32_t)q_start;
  d.dtype = dtype;
  d.softmax_scale = 1.f;
  return d;
}
bool same_layout(const Tensor& a, const Tensor& b) { return a.sizes() == b.sizes() && a.strides() == b.strides(); }

// The descriptor carries ONE stride triple for K and V and one for gK and gV, and the kernels index LSE as a
// contiguous fp32 [B, Hq, C] array: refuse tensors that do not fit that instead of computing on wrong addresses.
void check_shared(const Tensor& k, const Tensor& v, const Tensor* gk, const Tensor* gv, const Tensor& lse) {
  if (!same_layout(k, v)) raise(PyExc_ValueError, "k_cache and v_cache must share shape and strides");
  if (gk && !same_layout(*gk, *gv)) raise(PyExc_ValueError, "gk and gv must share shape and strides");
  if (gk && (gk->scalar_type() != at::kFloat || gv->scalar_type() != at::kFloat))
    raise(PyExc_TypeError, "gk / gv must be float32");
  if (lse.scalar_type() != at::kFloat || !lse.is_contiguous())
    raise(PyExc_ValueError, "lse must be a contiguous float32 [B, Hq, C] tensor");
}

// (q, k_cache, v_cache, q_start, scale, o, lse, stream, ws) -> (o, lse)
PyObject* fwd(PyObject* const* a) {
  const Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
  const Tensor o = a[5] == Py_None ? at::empty_like(q, q.options().requires_grad(false)) : tensor(a[5]);
  const Tensor lse = a[6] == Py_None
      ? at::empty(q.sizes().slice(0, 3), q.options().dtype(at::kFloat).requires_grad(false)) : tensor(a[6]);
  if (q.dim() != 4 || lse.sizes() != q.sizes().slice(0, 3)) raise(PyExc_ValueError, "lse must have shape [B, Hq, C]");
  check_shared(k, v, nullptr, nullptr, lse);
  const seco_desc d = chunk_desc(q, k, a[3], a[4], o, nullptr);
  void* s = stream(a[7]);
  Tensor ws;
  if (a[8] == Py_None) {
    const size_t n = workspace(d, SECO_OP_FWD);
    if (n > 0) ws = scratch((int64_t)n, q, s);
  } else if (a[8] != Py_False) {
    ws = tensor(a[8]);
  }
  check(lib.seco_chunk_attn_fwd(&d, ptr(q), ptr(k), ptr(v), ptr(o), fptr(lse), ws.defined() ? ptr(ws) : nullptr,
                                ws.defined() ? nbytes(ws) : 0, s), "seco_chunk_attn_fwd");
  PyObject* po = a[5] == Py_None ? THPVariable_Wrap(o) : (Py_INCREF(a[5]), a[5]);
  PyObject* pl = a[6] == Py_None ? THPVariable_Wrap(lse) : (Py_INCREF(a[6]), a[6]);
  return Py_BuildValue("NN", po, pl);
}

// (q, k_cache, v_cache, o, lse, d_o, gk, gv, q_start, scale, d_q, ws, stream, chunk_weight, weight_chunk_len, dq_weight)
PyObject* bwd(PyObject* const* a) {
  const Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &o = tensor(a[3]), &lse = tensor(a[4]),
               &d_o = tensor(a[5]), &gk = tensor(a[6]), &gv = tensor(a[7]);
  const Tensor dq = a[10] == Py_None ? like(q) : tensor(a[10]);
  if (o.strides() != d_o.strides() || q.strides() != dq.strides())
    raise(PyExc_ValueError, "o/d_o and q/d_q must share strides");
  check_shared(k, v, &gk, &gv, lse);
  const seco_desc d = chunk_desc(q, k, a[8], a[9], o, &gk);
  void* s = stream(a[12]);
  const Tensor ws = a[11] == Py_None ? scratch((int64_t)std::max<size_t>(workspace(d, SECO_OP_BWD), 256), q, s) : tensor(a[11]);
  if (a[13] == Py_None) {
    check(lib.seco_chunk_attn_bwd(&d, ptr(q), ptr(k), ptr(v), ptr(o), fptr(lse), ptr(d_o), ptr(dq), fptr(gk), fptr(gv),
                                  ptr(ws), nbytes(ws), s), "seco_chunk_attn_bwd");
  } else {
    const std::vector<float> w = floats(a[13]);
    const int32_t n = (int32_t)w.size(), wlen = int32(a[14]);
    if (a[15] != Py_None) {
      const std::vector<float> wq = floats(a[15]);
      if (wq.size() != w.size()) raise(PyExc_ValueError, "dq_weight and chunk_weight must have one entry per chunk");
      check(lib.spaco_chunk_attn_bwd_sparse_dq(&d, ptr(q), ptr(k), ptr(v), ptr(o), fptr(lse), ptr(d_o), ptr(dq), fptr(gk),
                                               fptr(gv), w.data(), wq.data(), n, wlen, ptr(ws), nbytes(ws), s),
            "spaco_chunk_attn_bwd_sparse_dq");
    } else {
      check(lib.spaco_chunk_attn_bwd(&d, ptr(q), ptr(k), ptr(v), ptr(o), fptr(lse), ptr(d_o), ptr(dq), fptr(gk), fptr(gv),
                                     w.data(), n, wlen, ptr(ws), nbytes(ws), s), "spaco_chunk_attn_bwd");
    }
  }
  return a[10] == Py_None ? THPVariable_Wrap(dq) : (Py_INCREF(a[10]), a[10]);
}

// (q, k_cache, v_cache, o, lse, d_o, d_q, gk, gv, q_start, scale, stream)
PyObject* bwd_noalloc(PyObject* const* a) {
  const Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &o = tensor(a[3]), &lse = tensor(a[4]),
               &d_o = tensor(a[5]), &dq = tensor(a[6]), &gk = tensor(a[7]), &gv = tensor(a[8]);
  if (o.strides() != d_o.strides() || q.strides() != dq.strides())
    raise(PyExc_ValueError, "o/d_o and q/d_q must share strides");
  check_shared(k, v, &gk, &gv, lse);
  const seco_desc d = chunk_desc(q, k, a[9], a[10], o, &gk);
  check(lib.seco_chunk_attn_bwd_noalloc(&d, ptr(q), ptr(k), ptr(v), ptr(o), fptr(lse), ptr(d_o), ptr(dq), fptr(gk), fptr(gv),
                                        stream(a[11])), "seco_chunk_attn_bwd_noalloc");
  return Py_INCREF(a[6]), a[6];
}

// (q_rows, k_cache, v_cache, o, lse, d_o_rows, gk, gv, q_start, scale, chunk_len, row_stats, d_q, ws, stream, row_weight,
//  weight_chunk_len)
PyObject* bwd_gather(PyObject* const* a) {
  const Tensor &q_rows = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &o = tensor(a[3]), &lse = tensor(a[4]),
               &do_rows = tensor(a[5]), &gk = tensor(a[6]), &gv = tensor(a[7]), &stats = tensor(a[11]);
  const int64_t C = integer(a[10]);
  if (q_rows.dim() != 4 || do_rows.dim() != 4) raise(PyExc_ValueError, "expected [batch, head, row, head_dim] tensors");
  const Tensor qc = q_rows.slice(2, 0, C);
  const Tensor dq = a[12] == Py_None ? like(qc) : tensor(a[12]);
  if (o.strides() != do_rows.strides() || qc.strides() != dq.strides())
    raise(PyExc_ValueError, "o/d_o and q/d_q must share strides");
  check_shared(k, v, &gk, &gv, lse);
  if (stats.scalar_type() != at::kFloat || !stats.is_contiguous() || stats.dim() != 4)
    raise(PyExc_ValueError, "row_stats must be a contiguous fp32 [2, B, Hq, stat_rows] tensor");
  const seco_desc d = chunk_desc(qc, k, a[8], a[9], o, &gk);
  void* s = stream(a[14]);
  const Tensor ws = a[13] == Py_None ? scratch((int64_t)std::max<size_t>(workspace(d, SECO_OP_BWD), 256), qc, s) : tensor(a[13]);
  const int32_t later = (int32_t)(q_rows.size(2) - C);
  if (a[15] != Py_None) {
    const std::vector<float> w = floats(a[15]);
    int64_t wlen = a[16] == Py_None ? 0 : integer(a[16]);
    if (wlen == 0) wlen = C;
    check(lib.spaco_chunk_attn_bwd_gather(&d, ptr(q_rows), ptr(k), ptr(v), ptr(o), fptr(lse), ptr(do_rows), ptr(dq), fptr(gk),
                                          fptr(gv), fptr(stats), stats.size(3), later, w.data(), (int32_t)w.size(),
                                          (int32_t)wlen, ptr(ws), nbytes(ws), s), "spaco_chunk_attn_bwd_gather");
  } else {
    check(lib.seco_chunk_attn_bwd_gather(&d, ptr(q_rows), ptr(k), ptr(v), ptr(o), fptr(lse), ptr(do_rows), ptr(dq), fptr(gk),
                                         fptr(gv), fptr(stats), stats.size(3), later, ptr(ws), nbytes(ws), s),
          "seco_chunk_attn_bwd_gather");
  }
  return a[12] == Py_None ? THPVariable_Wrap(dq) : (Py_INCREF(a[12]), a[12]);
}

seco_desc g_desc(const Tensor& g) {
  seco_desc d = rows_desc(g, 1, 0, SECO_F32);
  for (int64_t* st : {d.q_stride, d.o_stride, d.kv_stride, d.g_stride}) strides3(g, st);
  return d;
}
int64_t row_end(PyObject* o, const Tensor& g) { return o == Py_None ? g.size(2) : integer(o); }

// (gk, gv, row_begin, row_end, stream)
PyObject* zero(PyObject* const* a) {
  const Tensor *gk = opt_tensor(a[0]), *gv = opt_tensor(a[1]);
  const Tensor& ref = gk ? *gk : tensor(a[1]);
  const seco_desc d = g_desc(ref);
  check(lib.kvgrad_zero(&d, fptr(gk), fptr(gv), integer(a[2]), row_end(a[3], ref), stream(a[4])), "kvgrad_zero");
  Py_RETURN_NONE;
}

// (dst_k, dst_v, src_k, src_v, scale, row_begin, row_end, stream)
PyObject* accumulate(PyObject* const* a) {
  const Tensor *dk = opt_tensor(a[0]), *dv = opt_tensor(a[1]), *sk = opt_tensor(a[2]), *sv = opt_tensor(a[3]);
  const Tensor& ref = dk ? *dk : tensor(a[1]);
  const seco_desc d = g_desc(ref);
  if ((dk && sk && dk->strides() != sk->strides()) || (dv && sv && dv->strides() != sv->strides()))
    raise(PyExc_ValueError, "dst and src must share strides");
  check(lib.kvgrad_accumulate(&d, fptr(dk), fptr(dv), fptr(sk), fptr(sv), (float)real(a[4]), integer(a[5]),
                              row_end(a[6], ref), stream(a[7])), "kvgrad_accumulate");
  Py_RETURN_NONE;
}

// (k_new, v_new, k_cache, v_cache, row_begin, stream, rope_base)
PyObject* append(PyObject* const* a) {
  const Tensor &kn = tensor(a[0]), &vn = tensor(a[1]), &kc = tensor(a[2]), &vc = tensor(a[3]);
  seco_desc d = rows_desc(kn, kn.size(2), integer(a[4]), dtype_code(kn));
  strides3(kn, d.o_stride);
  strides3(kc, d.kv_stride);
  strides3(kn, d.g_stride);
  if (vn.strides() != kn.strides() || vc.strides() != kc.strides()) raise(PyExc_ValueError, "k/v must share strides");
  if (a[6] != Py_None)
    check(lib.kv_append_rope(&d, ptr(kn), ptr(vn), ptr(kc), ptr(vc), (float)real(a[6]), stream(a[5])), "kv_append_rope");
  else
    check(lib.kv_append(&d, ptr(kn), ptr(vn), ptr(kc), ptr(vc), stream(a[5])), "kv_append");
  Py_RETURN_NONE;
}

// (gk, gv, row_begin, n_rows, dtype, scaler, d_k, d_v, stream, rope_base) -> (d_k, d_v)
PyObject* readout(PyObject* const* a) {
  const Tensor &gk = tensor(a[0]), &gv = tensor(a[1]);
  if (gk.dim() != 4) raise(PyExc_ValueError, "expected a [batch, head, row, head_dim] tensor with contiguous head_dim");
  Tensor dk, dv;
  if (a[6] == Py_None) {
    if (!THPDtype_Check(a[4])) raise(PyExc_TypeError, "dtype must be a torch dtype");
    dk = at::empty({gk.size(0), gk.size(1), integer(a[3]), gk.size(3)},
                   gk.options().dtype(reinterpret_cast<THPDtype*>(a[4])->scalar_type).requires_grad(false));
  } else {
    dk = tensor(a[6]);
  }
  dv = a[7] == Py_None ? like(dk) : tensor(a[7]);
  if (gv.strides() != gk.strides() || dv.strides() != dk.strides())
    raise(PyExc_ValueError, "gk/gv and d_k/d_v must share strides");
  seco_desc d = rows_desc(dk, dk.size(2), integer(a[2]), dtype_code(dk));
  strides3(dk, d.o_stride);
  strides3(dk, d.kv_stride);
  strides3(gk, d.g_stride);
  if (a[9] != Py_None)
    check(lib.kvgrad_readout_rope(&d, fptr(gk), fptr(gv), ptr(dk), ptr(dv), (float)real(a[5]), (float)real(a[9]), stream(a[8])),
          "kvgrad_readout_rope");
  else
    check(lib.kvgrad_readout(&d, fptr(gk), fptr(gv), ptr(dk), ptr(dv), (float)real(a[5]), stream(a[8])), "kvgrad_readout");
  PyObject* pk = a[6] == Py_None ? THPVariable_Wrap(dk) : (Py_INCREF(a[6]), a[6]);
  PyObject* pv = a[7] == Py_None ? THPVariable_Wrap(dv) : (Py_INCREF(a[7]), a[7]);
  return Py_BuildValue("NN", pk, pv);
}

// (x, pos_start, rope_base, inverse, out, stream) -> out
PyObject* rotate(PyObject* const* a) {
  const Tensor& x = tensor(a[0]);
  const Tensor out = a[4] == Py_None ? like(x) : tensor(a[4]);
  seco_desc d = rows_desc(x, x.size(2), 0, x.scalar_type() == at::kBFloat16 ? SECO_BF16 : SECO_F32);
  for (int64_t* st : {d.kv_stride, d.g_stride}) strides3(x, st);
  strides3(out, d.o_stride);
  const int inv = PyObject_IsTrue(a[3]);
  if (inv < 0) throw Raised{};
  check(lib.rope_rotate(&d, (int32_t)x.size(1), ptr(x), ptr(out), integer(a[1]), (float)real(a[2]), inv, stream(a[5])),
        "rope_rotate");
  return a[4] == Py_None ? THPVariable_Wrap(out) : (Py_INCREF(a[4]), a[4]);
}

// (library path, SecoError)
PyObject* init(PyObject* const* a) {
  const char* path = PyUnicode_AsUTF8(a[0]);
  if (!path) throw Raised{};
  void* h = dlopen(path, RTLD_NOW);
  if (!h) raise(PyExc_ImportError, dlerror());
#define X(name)                                                        \
  lib.name = reinterpret_cast<decltype(&::name)>(dlsym(h, #name));    \
  if (!lib.name) raise(PyExc_ImportError, "entry point missing: " #name);
  SECO_ENTRIES(X)
#undef X
  Py_INCREF(a[1]);
  g_error = a[1];
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    SECO_METHOD("init", init, 2), SECO_METHOD("fwd", fwd, 9), SECO_METHOD("bwd", bwd, 16), SECO_METHOD("bwd_noalloc", bwd_noalloc, 12),
    SECO_METHOD("bwd_gather", bwd_gather, 17), SECO_METHOD("zero", zero, 5), SECO_METHOD("accumulate", accumulate, 8),
    SECO_METHOD("append", append, 7), SECO_METHOD("readout", readout, 10), SECO_METHOD("rotate", rotate, 6),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_seco_ext", "native half of the binding", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__seco_ext() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddFunctions(m, seco_ext::step_methods) < 0) Py_CLEAR(m);
  return m;
}
