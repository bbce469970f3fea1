// The training step of chunk_loop.py, one chunk at a time, on the host side: what is launched, in which order, on which
// buffers.  Second source of the extension module of the binding.
//
// A chunk of the step is about 60 launches of a few microseconds each.  Driven from Python, with the matrix products
// through the framework (17 - 19 us of host time per call), a two-layer step over 4096 tokens in chunks of 512 took
// 9.1 ms, of which the GPU worked 6.7; here a launch costs 2 - 4 us of host time, activations are carved from two
// blocks allocated once per step, and the products are the library's own (gemm_bf16.hip) where type, alignment and size
// allow: 3.4 ms, in which the GPU is busy throughout.
#include <map>
#include <memory>

#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/variable.h>

#include "binding_common.h"

namespace seco_ext {
namespace {

// A block of device memory handed out front to back; `mark` / `reset` free everything taken since.
struct Arena {
  Tensor buf;
  size_t used = 0;
  void create(size_t bytes_total, const Tensor& like_t) { buf = bytes((int64_t)bytes_total, like_t); }
  void* take(size_t n) {
    if (used + n > nbytes(buf)) raise(PyExc_RuntimeError, "activation block too small");
    void* p = static_cast<char*>(buf.data_ptr()) + used;
    used += (n + 255) & ~(size_t)255;
    return p;
  }
};

struct Param {
  Tensor w;              // contiguous
  bool wanted = false;
  Tensor grad;           // undefined until the first chunk adds to it
  std::vector<int64_t> sizes;                    // gains: the parameter's own shape and type (w: dm elements, in the
  at::ScalarType type = at::kFloat;              // type the norm computes its rows in)
};

struct Layer {
  Param norm1, norm2, wqkv, wo, w1, w2;
  int64_t ff = 0;                                // width of this layer's MLP
  float *part1 = nullptr, *part2 = nullptr;      // partial sums of the gains' gradients
  Tensor k, v, gk, gv;                           // KV cache and KV-gradient buffers, [B, Hkv, N, D]
  std::map<int64_t, std::pair<Tensor, Tensor>> kept;   // q_start -> (O rows [B, C, Hq, D], LSE) of stage 1
  Tensor q_all, do_all, o_all, dq_all, stats;    // transposed backward order only
};

// What the backward of a layer needs of a chunk's forward; C rows per sequence.
struct Saved {
  void *x1, *h1, *qkv, *o, *x2, *h2, *u, *a;
  float *r1, *lse, *r2;
  Tensor keep_o, keep_lse;                       // O and LSE taken back from stage 1; wide tail: x1 and h1 of the final norm
};

enum Keep { kCompute = 0, kStore = 1, kReuse = 2 };

struct Step {
  int64_t L, Hq, Hkv, D, B, N, dm, ff, V, W, HD;   // ff: the widest MLP; W: columns of the joint projection
  double scale, rope_base;                         // rope_base 0: no rotary embedding
  int dtype;
  size_t e;                                        // bytes per element
  int tail;                                        // type of the final norm's result, the head and the logits: dtype, or
                                                   // fp32 behind a bf16 body when both parameters are fp32
  Param emb, head, norm_f;
  float* part_f = nullptr;
  Tensor parts;
  Tensor result;                                   // the loss (the caller's sum), and 1 if a token lies outside the embedding table
  std::vector<Layer> layers;
  Arena stage1, stage2;
  void* s = nullptr;                               // stream of the current call
  bool trained = false;                            // a chunk has been back-propagated

  at::TensorOptions opts() const { return emb.w.options().requires_grad(false); }
  Tensor view(void* p, at::IntArrayRef sizes) { return at::from_blob(p, sizes, opts()); }
  Tensor view(void* p, at::IntArrayRef sizes, const Param& w) { return at::from_blob(p, sizes, w.w.options().requires_grad(false)); }

  // ---- matrix products: the library's own kernel where it takes the operands, the framework's otherwise
  // Small products are bound by their launch, which costs 17 - 19 us of host time through the framework and 3 here; of large
  // ones the framework's kernels are faster, by up to 1.8 times at 8192 rows.  The line between them, in multiply-adds and
  // by the rows of the chunk (R; gradients: of the matrix), lies where the two meet.  Measured with epilogue against
  // product and row pass, in us, own / framework, R x K -> N:
  //   forward     2048 x 4096 -> 1024  29 / 36     1024 x 4096 -> 4096  41 / 45     2048 x 2048 -> 8192  78 / 71
  //               4096 x 1024 -> 1024  18 / 22     8192 x 1024 -> 1024  29 / 30     4096 x 4096 -> 1024  51 / 44
  //   backward    2048 x 2048 <- 2048  26 / 27     1024 x 4096 <- 4096  41 / 41     2048 x 4096 <- 4096  74 / 67
  //               4096 x 1024 <- 1024  18 / 23     8192 x 1024 <- 1024  29 / 30     4096 x 1024 <- 4096  50 / 42
  //   gradient    512: 4096 x 1024  12 / 18     8192: 4096 x 4096  236 / 255     512: 8192 x 2048  39 / 28
  //               2048: 4096 x 14336  267 / 273     8192: 4096 x 14336  1054 / 1010     2048: 14336 x 4096  297 / 273
  static bool worth(int form, int64_t M, int64_t N_, int64_t K) {
    const double work = (double)M * N_ * K;
    if (form == DEC_GEMM_NN) return work <= (M <= 2048 ? 0x1p34 : 0x1p33);
    if (form == DEC_GEMM_NT) return work <= (M <= 2048 ? 0x1p33 : 0x1p32);
    return M <= 4096 && work < 0x1p38;
  }
  // (operands have the type of the matrix)
  static bool own(const Param& w, int form, int64_t M, int64_t N_, int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
    return w.w.scalar_type() == at::kBFloat16 && worth(form, M, N_, K) && lib.dec_gemm_supported(form, M, N_, K, lda, ldb, ldc);
  }
  // c[M, n] = a[M, K] w[K, n]
  void mm(void* c, void* a, const Param& w, int64_t M) {
    const int64_t K = w.w.size(0), n = w.w.size(1);
    if (own(w, DEC_GEMM_NN, M, n, K, K, n, n)) {
      check(lib.dec_gemm(DEC_GEMM_NN, DEC_GEMM_STORE, a, ptr(w.w), c, nullptr, M, n, K, K, n, n, s), "dec_gemm");
    } else {
      Tensor out = view(c, {M, n}, w);
      at::mm_out(out, view(a, {M, K}, w), w.w);
    }
  }
  // u = h w, a = silu(u)
  void mm_silu(void* u, void* a, void* h, const Param& w, int64_t M) {
    const int64_t K = w.w.size(0), n = w.w.size(1);
    if (own(w, DEC_GEMM_NN, M, n, K, K, n, n)) {
      check(lib.dec_gemm(DEC_GEMM_NN, DEC_GEMM_SILU, h, ptr(w.w), u, a, M, n, K, K, n, n, s), "dec_gemm");
    } else {
      mm(u, h, w, M);
      check(lib.dec_silu(dtype, u, a, M * n, s), "dec_silu");
    }
  }
  // d_x[M, K] = d_y[M, n] w[K, n]^T; u non-NULL: times silu'(u)
  void mm_bwd(void* dx, void* dy, const Param& w, int64_t M, void* u = nullptr) {
    const int64_t K = w.w.size(0), n = w.w.size(1);
    if (own(w, DEC_GEMM_NT, M, K, n, n, n, K)) {
      check(lib.dec_gemm(DEC_GEMM_NT, u ? DEC_GEMM_SILU_BWD : DEC_GEMM_STORE, dy, ptr(w.w), dx, u, M, K, n, n, n, K, s), "dec_gemm");
    } else {
      Tensor out = view(dx, {M, K}, w);
      at::mm_out(out, view(dy, {M, n}, w), w.w.t());
      if (u) check(lib.dec_silu_bwd(dtype, u, dx, M * K, s), "dec_silu_bwd");
    }
  }
  // grad[K, n] += x[M, K]^T d_y[M, n] (fp32 inside the product, rounded once per chunk)
  void add(Param& w, void* x, void* dy, int64_t M) {
    if (!w.wanted) return;
    const int64_t K = w.w.size(0), n = w.w.size(1);
    const bool first = !w.grad.defined();
    if (first) w.grad = at::empty({K, n}, w.w.options().requires_grad(false));
    if (own(w, DEC_GEMM_TN, K, n, M, K, n, n)) {
      check(lib.dec_gemm(DEC_GEMM_TN, first ? DEC_GEMM_STORE : DEC_GEMM_ADD, x, dy, ptr(w.grad), nullptr, K, n, M, K, n, n, s), "dec_gemm");
    } else if (first) {
      at::mm_out(w.grad, view(x, {M, K}, w).t(), view(dy, {M, n}, w));
    } else {
      w.grad.addmm_(view(x, {M, K}, w).t(), view(dy, {M, n}, w));
    }
  }

  // both gradients of y = x w: grad[K, n] += x[M, K]^T d_y[M, n], d_x[M, K] = d_y w^T (u non-NULL: times silu'(u))
  void grads(Param& w, void* x, void* dx, void* dy, int64_t M, void* u = nullptr) {
    const int64_t K = w.w.size(0), n = w.w.size(1);
    if (w.wanted && own(w, DEC_GEMM_TN, K, n, M, K, n, n) && own(w, DEC_GEMM_NT, M, K, n, n, n, K)) {
      const bool first = !w.grad.defined();
      if (first) w.grad = at::empty({K, n}, w.w.options().requires_grad(false));
      check((first ? lib.dec_gemm_first_grads : lib.dec_gemm_grads)(dy, ptr(w.w), dx, u, x, ptr(w.grad), M, K, n, s), "dec_gemm_grads");
    } else {
      add(w, x, dy, M);
      mm_bwd(dx, dy, w, M, u);
    }
  }

  // ---- attention
  seco_desc desc(int64_t C, int64_t q_start, const Layer& l) const {
    seco_desc d;
    const int64_t q[3] = {C * W, D, W}, o[3] = {C * HD, D, HD};
    for (int i = 0; i < 3; ++i) {
      d.q_stride[i] = q[i];
      d.o_stride[i] = o[i];
      d.kv_stride[i] = l.k.stride(i);
      d.g_stride[i] = l.gk.stride(i);
    }
    d.batch = (int32_t)B;
    d.n_q_heads = (int32_t)Hq;
    d.n_kv_heads = (int32_t)Hkv;
    d.head_dim = (int32_t)D;
    d.chunk_len = (int32_t)C;
    d.q_start = (int32_t)q_start;
    d.dtype = dtype;
    d.softmax_scale = (float)scale;
    return d;
  }
  char* at_col(void* qkv, int64_t col) const { return static_cast<char*>(qkv) + col * (int64_t)e; }
  void rotate(void* qkv, int64_t C, int64_t q_start, bool inverse) {
    if (rope_base == 0.0) return;
    seco_desc d = desc(C, 0, layers[0]);
    d.n_kv_heads = d.n_q_heads;
    const int64_t st[3] = {C * W, D, W};
    for (int64_t* x : {d.q_stride, d.o_stride, d.kv_stride, d.g_stride}) std::copy(st, st + 3, x);
    check(lib.rope_rotate(&d, (int32_t)Hq, qkv, qkv, q_start, (float)rope_base, inverse, s), "rope_rotate");
  }
  // queries turned in place, keys (turned) and values to the cache; or, on the way back, the queries' gradient turned back and
  // the key and value gradients from gK / gV: one launch where the library's call takes the sizes
  bool rope_qkv(Layer& l, void* qkv, int64_t C, int64_t q_start, bool inverse) {
    if (rope_base == 0.0) return false;
    const Tensor &k = inverse ? l.gk : l.k, &v = inverse ? l.gv : l.v;
    const int64_t st[3] = {k.stride(0), k.stride(1), k.stride(2)};
    const int rc = lib.dec_rope_qkv(dtype, inverse, qkv, ptr(k), ptr(v), st, B, Hq, Hkv, C, D, q_start, (float)rope_base, s);
    if (rc == SECO_ERR_TOO_LARGE) return false;
    check(rc, "dec_rope_qkv");
    return true;
  }
  // the joint projection of h, its queries turned and its keys and values in the cache
  void project(Layer& l, void* qkv, void* h, int64_t C, int64_t q_start) {
    const int64_t M = B * C;
    if (rope_base != 0.0 && D == 128 && own(l.wqkv, DEC_GEMM_NN, M, W, dm, dm, W, W)) {
      const int64_t st[3] = {l.k.stride(0), l.k.stride(1), l.k.stride(2)};
      const int rc = lib.dec_gemm_qkv(h, ptr(l.wqkv.w), qkv, ptr(l.k), ptr(l.v), st, B, Hq, Hkv, C, dm, q_start, (float)rope_base, s);
      if (rc != SECO_ERR_TOO_LARGE) return check(rc, "dec_gemm_qkv");
    }
    mm(qkv, h, l.wqkv, M);
    append(l, qkv, C, q_start);
  }
  void append(Layer& l, void* qkv, int64_t C, int64_t q_start) {
    if (rope_qkv(l, qkv, C, q_start, false)) return;
    rotate(qkv, C, q_start, false);
    seco_desc d = desc(C, q_start, l);
    std::copy(d.q_stride, d.q_stride + 3, d.o_stride);
    std::copy(d.q_stride, d.q_stride + 3, d.g_stride);
    d.n_q_heads = d.n_kv_heads;
    d.softmax_scale = 1.f;
    void *k = at_col(qkv, HD), *v = at_col(qkv, HD + Hkv * D);
    if (rope_base != 0.0)
      check(lib.kv_append_rope(&d, k, v, ptr(l.k), ptr(l.v), (float)rope_base, s), "kv_append_rope");
    else
      check(lib.kv_append(&d, k, v, ptr(l.k), ptr(l.v), s), "kv_append");
  }
  void readout(Layer& l, void* d_qkv, int64_t C, int64_t q_start) {
    if (rope_qkv(l, d_qkv, C, q_start, true)) return;
    rotate(d_qkv, C, q_start, true);
    seco_desc d = desc(C, q_start, l);
    std::copy(d.q_stride, d.q_stride + 3, d.o_stride);
    std::copy(d.q_stride, d.q_stride + 3, d.kv_stride);
    d.n_q_heads = d.n_kv_heads;
    d.softmax_scale = 1.f;
    void *dk = at_col(d_qkv, HD), *dv = at_col(d_qkv, HD + Hkv * D);
    if (rope_base != 0.0)
      check(lib.kvgrad_readout_rope(&d, fptr(l.gk), fptr(l.gv), dk, dv, 1.f, (float)rope_base, s), "kvgrad_readout_rope");
    else
      check(lib.kvgrad_readout(&d, fptr(l.gk), fptr(l.gv), dk, dv, 1.f, s), "kvgrad_readout");
  }
  // O and LSE of the chunk, whose k / v are in the cache.  (kReuse: the rebuilt chunk has the same inputs and the kernels are
  // deterministic, so the values are identical and the cache rows already hold this chunk's K/V.)
  void attention(Layer& l, Saved& sv, int64_t C, int64_t q_start, Keep keep, Arena& mem) {
    if (keep == kReuse) {
      rotate(sv.qkv, C, q_start, false);
      // the span of stage 1 that holds this chunk's rows (the chunk itself, or a longer span to cut from)
      auto it = l.kept.upper_bound(q_start);
      if (it == l.kept.begin()) raise(PyExc_RuntimeError, "no kept attention output");
      --it;
      const int64_t a = q_start - it->first;
      if (a + C > it->second.first.size(1)) raise(PyExc_ValueError, "the chunk's kept attention outputs are in two spans of stage 1");
      sv.keep_o = it->second.first;
      sv.keep_lse = it->second.second;
      if (a != 0 || C != sv.keep_o.size(1)) {
        sv.keep_o = sv.keep_o.slice(1, a, a + C).contiguous();
        sv.keep_lse = sv.keep_lse.slice(2, a, a + C).contiguous();
      }
      sv.o = ptr(sv.keep_o);
      sv.lse = fptr(sv.keep_lse);
      return;
    }
    if (keep == kStore) {
      sv.keep_o = at::empty({B, C, Hq, D}, opts());
      sv.keep_lse = at::empty({B, Hq, C}, opts().dtype(at::kFloat));
      l.kept[q_start] = {sv.keep_o, sv.keep_lse};
      sv.o = ptr(sv.keep_o);
      sv.lse = fptr(sv.keep_lse);
    } else {
      sv.o = mem.take(B * C * HD * e);
      sv.lse = static_cast<float*>(mem.take(B * Hq * C * 4));
    }
    const seco_desc d = desc(C, q_start, l);
    const size_t n = workspace(d, SECO_OP_FWD);
    Tensor ws;
    if (n > 0) ws = bytes((int64_t)n, emb.w);
    check(lib.seco_chunk_attn_fwd(&d, sv.qkv, ptr(l.k), ptr(l.v), sv.o, sv.lse, n ? ptr(ws) : nullptr, n, s), "seco_chunk_attn_fwd");
  }
  void attention_bwd(Layer& l, const Saved& sv, void* d_o, void* d_qkv, int64_t C, int64_t q_start, const std::vector<float>& w,
                     const std::vector<float>& wq, int64_t wlen) {
    seco_desc d = desc(C, q_start, l);
    const Tensor ws = bytes((int64_t)std::max<size_t>(workspace(d, SECO_OP_BWD), 256), emb.w);
    const size_t nw = nbytes(ws);
    if (l.q_all.defined()) {
      // transposed order: this chunk's finished gK/gV rows from its own and every later chunk's query rows, whose Q and
      // dO the layer has kept; nothing is added to earlier rows.  w: weights of the row chunks under Alg. 2
      auto heads = [&](void* p, int64_t row) { return at::from_blob(p, {B, Hq, C, D}, {C * row, D, row, 1}, opts()); };
      l.q_all.slice(2, q_start, q_start + C).copy_(heads(sv.qkv, W));
      l.do_all.slice(2, q_start, q_start + C).copy_(heads(d_o, HD));
      l.o_all.slice(2, q_start, q_start + C).copy_(heads(sv.o, HD));
      Tensor dq = l.dq_all.slice(2, q_start, q_start + C);
      for (int i = 0; i < 3; ++i) d.q_stride[i] = d.o_stride[i] = l.q_all.stride(i);
      auto row = [&](const Tensor& t) { return static_cast<char*>(ptr(t)) + q_start * t.stride(2) * (int64_t)e; };
      const int32_t later = (int32_t)(N - q_start - C);
      if (w.empty())
        check(lib.seco_chunk_attn_bwd_gather(&d, row(l.q_all), ptr(l.k), ptr(l.v), row(l.o_all), sv.lse, row(l.do_all), ptr(dq),
                                             fptr(l.gk), fptr(l.gv), fptr(l.stats), l.stats.size(3), later, ptr(ws), nw, s),
              "seco_chunk_attn_bwd_gather");
      else
        check(lib.spaco_chunk_attn_bwd_gather(&d, row(l.q_all), ptr(l.k), ptr(l.v), row(l.o_all), sv.lse, row(l.do_all), ptr(dq),
                                              fptr(l.gk), fptr(l.gv), fptr(l.stats), l.stats.size(3), later, w.data(),
                                              (int32_t)w.size(), (int32_t)wlen, ptr(ws), nw, s), "spaco_chunk_attn_bwd_gather");
      heads(d_qkv, W).copy_(dq);
    } else if (w.empty() && wq.empty()) {
      check(lib.seco_chunk_attn_bwd(&d, sv.qkv, ptr(l.k), ptr(l.v), sv.o, sv.lse, d_o, d_qkv, fptr(l.gk), fptr(l.gv), ptr(ws), nw, s),
            "seco_chunk_attn_bwd");
    } else {
      const std::vector<float> ones(wq.size(), 1.f);
      const std::vector<float>& cw = w.empty() ? ones : w;
      const int32_t n = (int32_t)cw.size();
      if (wq.empty())
        check(lib.spaco_chunk_attn_bwd(&d, sv.qkv, ptr(l.k), ptr(l.v), sv.o, sv.lse, d_o, d_qkv, fptr(l.gk), fptr(l.gv), cw.data(), n,
                                       (int32_t)wlen, ptr(ws), nw, s), "spaco_chunk_attn_bwd");
      else if (wq.size() != cw.size())
        raise(PyExc_ValueError, "dq_weight and chunk_weight must have one entry per chunk");
      else
        check(lib.spaco_chunk_attn_bwd_sparse_dq(&d, sv.qkv, ptr(l.k), ptr(l.v), sv.o, sv.lse, d_o, d_qkv, fptr(l.gk), fptr(l.gv),
                                                 cw.data(), wq.data(), n, (int32_t)wlen, ptr(ws), nw, s),
              "spaco_chunk_attn_bwd_sparse_dq");
    }
  }

  // ---- one chunk.  Returns its logits; saved: receives what the backward needs of every layer and, last, of the final norm
  // (NULL in stage 1, where the residual stream is updated in place and the layers share their buffers).
  // to_cache: only as far as the last layer's cache rows (and, kept, its attention output); returns NULL
  void* forward(const Tensor& tok, int64_t C, int64_t q_start, Keep keep, Arena& mem, std::vector<Saved>* saved, Tensor& x0,
                bool to_cache = false) {
    const int64_t R = B * C;
    auto rows = [&](int64_t n) { return mem.take((size_t)(R * n) * e); };
    auto stats = [&]() { return static_cast<float*>(mem.take((size_t)R * 4)); };
    auto norm = [&](void* x, void* y, const Param& g, void* xo, void* h, float* r) {
      check(lib.dec_add_rmsnorm(dtype, x, y, ptr(g.w), xo, h, r, R, dm, s), "dec_add_rmsnorm");
    };
    // the chunk's rows of the table, written by the first norm
    x0 = layers.empty() ? at::index(emb.w, {tok}) : at::empty({R, dm}, opts());
    void *x = ptr(x0), *y = rows(dm), *logits = mem.take((size_t)(R * V) * head.w.element_size());
    bool have_y = false;
    const size_t base = mem.used;
    for (Layer& l : layers) {
      if (!saved) mem.used = base;
      Saved sv{};
      sv.x1 = have_y && saved ? rows(dm) : x;
      sv.h1 = rows(dm);
      sv.r1 = stats();
      if (&l == &layers.front())
        check(lib.dec_embed_rmsnorm_checked(dtype, ptr(emb.w), static_cast<const int64_t*>(ptr(tok)), ptr(l.norm1.w), x, sv.h1, sv.r1, R, dm,
                                            emb.w.size(0), fptr(result) + 1, s), "dec_embed_rmsnorm");
      else
        norm(x, y, l.norm1, sv.x1, sv.h1, sv.r1);
      sv.qkv = rows(W);
      if (keep == kReuse)
        mm(sv.qkv, sv.h1, l.wqkv, R);
      else
        project(l, sv.qkv, sv.h1, C, q_start);
      if (to_cache && &l == &layers.back() && keep == kCompute) return nullptr;
      attention(l, sv, C, q_start, keep, mem);
      if (to_cache && &l == &layers.back()) return nullptr;
      mm(y, sv.o, l.wo, R);
      sv.x2 = saved ? rows(dm) : x;
      sv.h2 = rows(dm);
      sv.r2 = stats();
      norm(sv.x1, y, l.norm2, sv.x2, sv.h2, sv.r2);
      sv.u = rows(l.ff);
      sv.a = rows(l.ff);
      mm_silu(sv.u, sv.a, sv.h2, l.w1, R);
      mm(y, sv.a, l.w2, R);
      have_y = true;
      x = sv.x2;
      if (saved) saved->push_back(std::move(sv));
    }
    if (!saved) mem.used = base;
    Saved sv{};
    sv.r1 = stats();
    if (tail == dtype) {
      sv.x1 = have_y && saved ? rows(dm) : x;
      sv.h1 = rows(dm);
      norm(x, have_y ? y : nullptr, norm_f, sv.x1, sv.h1, sv.r1);
    } else {
      const Tensor xr = view(x, {R, dm});
      sv.keep_o = (have_y ? xr + view(y, {R, dm}) : xr).to(at::kFloat);   // (the residual sum rounds to the body's type)
      sv.keep_lse = at::empty_like(sv.keep_o);
      sv.x1 = ptr(sv.keep_o);
      sv.h1 = ptr(sv.keep_lse);
      check(lib.dec_add_rmsnorm(tail, sv.x1, nullptr, ptr(norm_f.w), nullptr, sv.h1, sv.r1, R, dm, s), "dec_add_rmsnorm");
    }
    mm(logits, sv.h1, head, R);
    if (saved) saved->push_back(std::move(sv));
    return logits;
  }

  // Adds the chunk's parameter gradients; d_logits: gradient of its loss at the logits.
  void backward(void* d_logits, const Tensor& tok, int64_t C, int64_t q_start, std::vector<Saved>& saved, Arena& mem,
                const std::vector<float>& w, const std::vector<std::vector<float>>& wq, int64_t wlen) {
    const int64_t R = B * C;
    auto rows = [&](int64_t n) { return mem.take((size_t)(R * n) * e); };
    void *dh = rows(dm), *dx = rows(dm), *du = rows(ff), *d_o = rows(HD), *d_qkv = rows(W);
    // dx <- dx + gradient of the norm at x (first: without dx)
    auto norm_bwd = [&](void* x, const Param& g, float* r, float* part, bool first) {
      check(lib.dec_rmsnorm_bwd(dtype, x, ptr(g.w), r, dh, first ? nullptr : dx, dx, part, R, dm, s), "dec_rmsnorm_bwd");
    };
    const Saved fin = std::move(saved.back());
    saved.pop_back();
    if (tail == dtype) {
      grads(head, fin.h1, dh, d_logits, R);
      norm_bwd(fin.x1, norm_f, fin.r1, part_f, true);
    } else {
      const Tensor dh_f = at::empty_like(fin.keep_o), dx_f = at::empty_like(fin.keep_o);
      grads(head, fin.h1, ptr(dh_f), d_logits, R);
      check(lib.dec_rmsnorm_bwd(tail, fin.x1, ptr(norm_f.w), fin.r1, ptr(dh_f), nullptr, ptr(dx_f), part_f, R, dm, s), "dec_rmsnorm_bwd");
      view(dx, {R, dm}).copy_(dx_f);
    }
    static const std::vector<float> none;
    for (int64_t i = L - 1; i >= 0; --i) {
      Layer& l = layers[i];
      const Saved& sv = saved[i];
      grads(l.w2, sv.a, du, dx, R, sv.u);
      grads(l.w1, sv.h2, dh, du, R);
      norm_bwd(sv.x2, l.norm2, sv.r2, l.part2, false);
      grads(l.wo, sv.o, d_o, dx, R);
      attention_bwd(l, sv, d_o, d_qkv, C, q_start, w, wq.empty() ? none : wq[i], wlen);
      readout(l, d_qkv, C, q_start);
      grads(l.wqkv, sv.h1, dh, d_qkv, R);
      norm_bwd(sv.x1, l.norm1, sv.r1, l.part1, false);
    }
    if (emb.wanted) {
      if (!emb.grad.defined()) emb.grad = at::zeros({emb.w.size(0), dm}, opts());
      check(lib.dec_embedding_bwd(dtype, dx, static_cast<const int64_t*>(ptr(tok)), ptr(emb.grad), R, dm, emb.w.size(0), s),
            "dec_embedding_bwd");
    }
  }
};

constexpr char kName[] = "seco_step";
Step& step_of(PyObject* o) {
  void* p = PyCapsule_GetPointer(o, kName);
  if (!p) throw Raised{};
  return *static_cast<Step*>(p);
}
void begin(Step& st) {
  st.s = stream(Py_None);
}

// contiguous from a 16-byte boundary on, which a piece of a larger buffer need not be
Tensor laid_out(const Tensor& t) {
  const Tensor c = t.contiguous();
  return reinterpret_cast<uintptr_t>(c.data_ptr()) & 15u ? c.clone() : c;
}
Param param(PyObject* o) {
  const Tensor& t = tensor(o);
  Param p;
  p.wanted = t.requires_grad();
  p.w = laid_out(t.detach());
  return p;
}

// The kernels take sizes from the first parameters and addresses on trust, so every matrix is compared with what will be
// assumed of it before anything is allocated or launched.  rows, cols: -1 leaves that size free (at least `least`).
void check_matrix(const Tensor& t, const char* name, int64_t rows, int64_t cols, int64_t least = 1) {
  auto fits = [&](int i, int64_t n) { return n < 0 ? t.size(i) >= least : t.size(i) == n; };
  if (t.dim() == 2 && fits(0, rows) && fits(1, cols)) return;
  PyErr_Format(PyExc_ValueError, "the shape of %s does not fit the decoder's: expected [%lld, %lld] (-1: any size)", name,
               (long long)rows, (long long)cols);
  throw Raised{};
}

// The gain of a norm over rows of dm elements.  As it multiplies the rows by broadcasting, it may hold dm elements or
// one, behind any number of leading ones, and be of a narrower type than the rows.
void check_gain(const Tensor& t, const char* name, int64_t dm, at::ScalarType rows) {
  if ((t.numel() != dm && t.numel() != 1) || (t.dim() > 0 && t.size(-1) != t.numel())) {
    PyErr_Format(PyExc_ValueError, "the shape of %s does not fit the decoder's: expected [%lld] or one element", name, (long long)dm);
    throw Raised{};
  }
  if (at::promote_types(t.scalar_type(), rows) != rows) {
    PyErr_Format(PyExc_TypeError, "parameters must share one dtype: %s is wider than the rows it multiplies", name);
    throw Raised{};
  }
}
Param gain(PyObject* o, int64_t dm, at::ScalarType rows) {
  const Tensor& t = tensor(o);
  Param p;
  p.wanted = t.requires_grad();
  p.sizes = t.sizes().vec();
  p.type = t.scalar_type();
  p.w = laid_out(t.detach().to(rows).reshape({-1}).expand({dm}));
  return p;
}

// (config, params): config = (n_layers, Hq, Hkv, D, scale, rope_base or None, B, N, chunk rows of stage 1, of stage 2, transposed);
// params = [emb, head, norm_f, then norm1, norm2, wq, wk, wv, wo, w1, w2 of every layer] -> step
PyObject* step_new(PyObject* const* a) {
  if (!PyTuple_Check(a[0]) || PyTuple_GET_SIZE(a[0]) != 11 || !PyList_Check(a[1])) raise(PyExc_TypeError, "expected (tuple of 11, list)");
  auto cfg = [&](int i) { return PyTuple_GET_ITEM(a[0], i); };
  auto st = std::make_unique<Step>();
  st->L = integer(cfg(0));
  st->Hq = integer(cfg(1));
  st->Hkv = integer(cfg(2));
  st->D = integer(cfg(3));
  st->scale = real(cfg(4));
  st->rope_base = cfg(5) == Py_None ? 0.0 : real(cfg(5));
  st->B = integer(cfg(6));
  st->N = integer(cfg(7));
  const int64_t c1 = integer(cfg(8)), c2 = integer(cfg(9));
  const bool transposed = PyObject_IsTrue(cfg(10)) == 1;
  if (PyList_GET_SIZE(a[1]) != 3 + 8 * st->L) raise(PyExc_ValueError, "wrong number of parameters");
  if (st->L < 0 || st->Hq < 1 || st->Hkv < 1 || st->D < 1 || st->B < 1 || st->N < 1 || c1 < 1 || c2 < 1)
    raise(PyExc_ValueError, "sizes must be positive");
  st->HD = st->Hq * st->D;
  st->W = st->HD + 2 * st->Hkv * st->D;
  auto par = [&](int64_t i) { return PyList_GET_ITEM(a[1], i); };
  const Tensor& first = tensor(par(0));
  const at::ScalarType body = first.scalar_type();
  st->dtype = dtype_code(first);
  check_matrix(first, "emb", -1, -1);
  st->dm = first.size(1);
  check_matrix(tensor(par(1)), "head", st->dm, -1);
  // (a wider gain makes the rows behind it wider)
  const at::ScalarType tail = at::promote_types(body, tensor(par(2)).scalar_type());
  check_gain(tensor(par(2)), "norm_f", st->dm, tail);
  if (tensor(par(1)).scalar_type() != tail)
    raise(PyExc_TypeError, "head must have the dtype of the rows of the final norm: the wider one of emb's and norm_f's");
  st->tail = dtype_code(tensor(par(1)));
  for (int64_t i = 0; i < st->L; ++i) {
    auto at_layer = [&](int64_t k) -> const Tensor& { return tensor(par(3 + 8 * i + k)); };
    check_gain(at_layer(0), "norm1", st->dm, body);
    check_gain(at_layer(1), "norm2", st->dm, body);
    check_matrix(at_layer(2), "wq", st->dm, st->HD);
    check_matrix(at_layer(3), "wk", st->dm, st->Hkv * st->D);
    check_matrix(at_layer(4), "wv", st->dm, st->Hkv * st->D);
    check_matrix(at_layer(5), "wo", st->HD, st->dm);
    check_matrix(at_layer(6), "w1", st->dm, -1, 0);
    check_matrix(at_layer(7), "w2", at_layer(6).size(1), st->dm);
    for (int64_t k = 2; k < 8; ++k)
      if (at_layer(k).scalar_type() != body) raise(PyExc_TypeError, "parameters must share one dtype");
  }
  for (int64_t i = 0; i < 3 + 8 * st->L; ++i)
    if (!tensor(par(i)).is_cuda() || tensor(par(i)).device() != first.device())
      raise(PyExc_ValueError, "parameters must be on one GPU");
  st->emb = param(par(0));
  st->head = param(par(1));
  st->norm_f = gain(par(2), st->dm, tail);
  const Tensor& em = st->emb.w;
  st->e = em.element_size();
  st->V = st->head.w.size(1);
  st->ff = 0;
  const at::TensorOptions f32 = st->opts().dtype(at::kFloat);
  const int64_t n_parts = (2 * st->L + 1) * DEC_GAIN_BLOCKS * st->dm;
  st->parts = at::zeros({n_parts + 2}, f32);
  st->result = st->parts.slice(0, n_parts, n_parts + 2);
  auto part = [&](int64_t i) { return fptr(st->parts) + i * DEC_GAIN_BLOCKS * st->dm; };
  st->part_f = part(2 * st->L);
  st->layers.resize(st->L);
  for (int64_t i = 0; i < st->L; ++i) {
    Layer& l = st->layers[i];
    const int64_t p0 = 3 + 8 * i;
    l.norm1 = gain(par(p0), st->dm, body);
    l.norm2 = gain(par(p0 + 1), st->dm, body);
    // one projection product (and one gradient product each way) for queries, keys and values instead of three
    const Tensor &q = tensor(par(p0 + 2)), &k = tensor(par(p0 + 3)), &v = tensor(par(p0 + 4));
    l.wqkv.w = at::cat({q.detach(), k.detach(), v.detach()}, 1);
    l.wqkv.wanted = q.requires_grad() || k.requires_grad() || v.requires_grad();
    l.wo = param(par(p0 + 5));
    l.w1 = param(par(p0 + 6));
    l.w2 = param(par(p0 + 7));
    l.ff = l.w1.w.size(1);
    st->ff = std::max(st->ff, l.ff);
    l.part1 = part(2 * i);
    l.part2 = part(2 * i + 1);
    // (cache rows are written before they are read; the gradient rows are cleared before stage 2)
    l.k = at::empty({st->B, st->Hkv, st->N, st->D}, st->opts());
    l.v = at::empty_like(l.k);
    l.gk = at::empty({st->B, st->Hkv, st->N, st->D}, f32);
    l.gv = at::empty_like(l.gk);
    if (transposed) {
      for (Tensor* t : {&l.q_all, &l.do_all, &l.o_all, &l.dq_all}) *t = at::empty({st->B, st->Hq, st->N, st->D}, st->opts());
      l.stats = at::empty({2, st->B, st->Hq, (st->N + 3) / 4 * 4}, f32);
    }
  }
  // activations: see forward / backward for what is taken (each piece rounded up to 256 bytes)
  const size_t e = st->e;
  auto layer_bytes = [&](int64_t R) { return (size_t)R * ((4 * st->dm + st->W + st->HD + 2 * st->ff) * e + 8 + 4 * st->Hq) + 12 * 256; };
  auto other_bytes = [&](int64_t R) { return (size_t)R * (3 * st->dm * e + st->V * st->head.w.element_size() + 4) + 8 * 256; };
  auto bwd_bytes = [&](int64_t R) { return (size_t)R * (2 * st->dm + st->ff + st->HD + st->W) * e + 8 * 256; };
  const int64_t R1 = st->B * c1, R2 = st->B * c2;
  st->stage1.create(layer_bytes(R1) + other_bytes(R1), em);
  st->stage2.create(st->L * layer_bytes(R2) + other_bytes(R2) + bwd_bytes(R2), em);
  PyObject* cap = PyCapsule_New(st.get(), kName, [](PyObject* o) { delete static_cast<Step*>(PyCapsule_GetPointer(o, kName)); });
  if (!cap) throw Raised{};
  st.release();
  return cap;
}

// rows [s0, s1) of every sequence; the kernels read as many entries as the chunk has tokens, one behind the other (of one sequence
// reshape alone would give a view with the stride of t's columns)
Tensor chunk_of(const Step& st, const Tensor& t, int64_t s0, int64_t s1) {
  if (t.device() != st.emb.w.device() || t.scalar_type() != at::kLong || t.dim() != 2 || t.size(0) != st.B || t.size(1) < s1)
    raise(PyExc_ValueError, "tokens, targets: int64 [B, N] on the parameters' GPU");
  if (s0 < 0 || s1 <= s0 || s1 > st.N) raise(PyExc_ValueError, "chunk outside the sequence");
  return t.slice(1, s0, s1).reshape({-1}).contiguous();
}

// where the losses of rows [s0, s1) of every sequence go
float* losses_at(const Step& st, const Tensor& losses, int64_t s0, int64_t s1) {
  if (losses.device() != st.emb.w.device() || losses.scalar_type() != at::kFloat || !losses.is_contiguous() || losses.numel() < st.B * s1)
    raise(PyExc_ValueError, "losses: one float32 per token");
  return fptr(losses) + s0 * st.B;
}

// (step, tokens, targets, s0, s1, losses, store): inference over rows [s0, s1) of every sequence; their losses (None: the
// chunk is rebuilt later with the same launches, which then give the losses; here it ends at the last layer's cache rows)
PyObject* step_infer(PyObject* const* a) {
  Step& st = step_of(a[0]);
  begin(st);
  const int64_t s0 = integer(a[3]), s1 = integer(a[4]);
  const Tensor tok = chunk_of(st, tensor(a[1]), s0, s1), tgt = chunk_of(st, tensor(a[2]), s0, s1);
  const bool to_cache = a[5] == Py_None;
  float* losses = to_cache ? nullptr : losses_at(st, tensor(a[5]), s0, s1);
  st.stage1.used = 0;
  Tensor x0;
  void* logits = st.forward(tok, s1 - s0, s0, PyObject_IsTrue(a[6]) == 1 ? kStore : kCompute, st.stage1, nullptr, x0, to_cache);
  if (!to_cache)
    check(lib.dec_cross_entropy(st.tail, logits, static_cast<const int64_t*>(ptr(tgt)), losses, tok.numel(), st.V, st.s), "dec_cross_entropy");
  Py_RETURN_NONE;
}

// (step): clears the KV-gradient buffers
PyObject* step_zero(PyObject* const* a) {
  Step& st = step_of(a[0]);
  begin(st);
  for (Layer& l : st.layers) {
    seco_desc d = st.desc(1, 0, l);
    check(lib.kvgrad_zero(&d, fptr(l.gk), fptr(l.gv), 0, st.N, st.s), "kvgrad_zero");
  }
  Py_RETURN_NONE;
}

// (step, tokens, targets, s0, s1, reuse, weights or None, weight chunk length, per-layer dQ weights or None, losses or None):
// rebuilds the chunk and back-propagates its loss
PyObject* step_train(PyObject* const* a) {
  Step& st = step_of(a[0]);
  begin(st);
  const int64_t s0 = integer(a[3]), s1 = integer(a[4]);
  const Tensor tok = chunk_of(st, tensor(a[1]), s0, s1), tgt = chunk_of(st, tensor(a[2]), s0, s1);
  std::vector<float> w;
  if (a[6] != Py_None) w = floats(a[6]);
  std::vector<std::vector<float>> wq;
  if (a[8] != Py_None) {
    if (!PyList_Check(a[8]) || PyList_GET_SIZE(a[8]) != st.L) raise(PyExc_ValueError, "dq weights: one entry per layer");
    for (int64_t i = 0; i < st.L; ++i) {
      PyObject* x = PyList_GET_ITEM(a[8], i);
      wq.push_back(x == Py_None ? std::vector<float>() : floats(x));
    }
  }
  float* losses = a[9] == Py_None ? nullptr : losses_at(st, tensor(a[9]), s0, s1);
  st.stage2.used = 0;
  std::vector<Saved> saved;
  saved.reserve(st.L + 1);
  Tensor x0;
  void* logits = st.forward(tok, s1 - s0, s0, PyObject_IsTrue(a[5]) == 1 ? kReuse : kCompute, st.stage2, &saved, x0);
  const int64_t* target = static_cast<const int64_t*>(ptr(tgt));
  if (losses)
    check(lib.dec_cross_entropy_both(st.tail, logits, target, losses, tok.numel(), st.V, st.s), "dec_cross_entropy_both");
  else
    check(lib.dec_cross_entropy(st.tail, logits, target, nullptr, tok.numel(), st.V, st.s), "dec_cross_entropy");
  st.trained = true;
  st.backward(logits, tok, s1 - s0, s0, saved, st.stage2, w, wq, integer(a[7]));
  Py_RETURN_NONE;
}

// (step) -> fp32 [2]: room for the loss, and 1 if a token of a chunk so far lies outside the embedding table, else 0
PyObject* step_result(PyObject* const* a) { return THPVariable_Wrap(step_of(a[0]).result); }

// (step) -> gradients in the order of step_new's params; None where no chunk reached the parameter
PyObject* step_grads(PyObject* const* a) {
  Step& st = step_of(a[0]);
  begin(st);
  std::vector<Tensor> out = {st.emb.grad, st.head.grad};
  const Tensor sums = at::empty({2 * st.L + 1, st.dm}, st.parts.options()), gains = st.dtype == SECO_F32 ? sums : at::empty({2 * st.L + 1, st.dm}, st.opts());
  check(lib.dec_gain_sums(st.dtype, fptr(st.parts), fptr(sums), st.dtype == SECO_F32 ? nullptr : ptr(gains), 2 * st.L + 1, st.dm, st.s),
        "dec_gain_sums");
  auto gain = [&](int64_t i, const Param& p) {
    if (!st.trained) return Tensor();
    if (p.type == gains.scalar_type() && p.sizes.size() == 1 && p.sizes[0] == st.dm) return gains.select(0, i);
    Tensor g = sums.select(0, i);
    int64_t n = 1;
    for (int64_t x : p.sizes) n *= x;
    if (n != st.dm) g = g.sum();
    return g.to(p.type).reshape(p.sizes);
  };
  out.push_back(gain(2 * st.L, st.norm_f));
  for (int64_t i = 0; i < st.L; ++i) {
    Layer& l = st.layers[i];
    out.push_back(gain(2 * i, l.norm1));
    out.push_back(gain(2 * i + 1, l.norm2));
    const int64_t kv = st.Hkv * st.D;
    Tensor q, k, v;
    if (l.wqkv.grad.defined()) {
      q = at::empty({st.dm, st.HD}, st.opts());
      k = at::empty({st.dm, kv}, st.opts());
      v = at::empty({st.dm, kv}, st.opts());
      const int64_t e = (int64_t)st.e;
      check(lib.dec_split_columns(ptr(l.wqkv.grad), ptr(q), ptr(k), ptr(v), st.dm, st.HD * e, kv * e, kv * e, st.s), "dec_split_columns");
    }
    for (const Tensor& t : {q, k, v}) out.push_back(t);
    out.push_back(l.wo.grad);
    out.push_back(l.w1.grad);
    out.push_back(l.w2.grad);
  }
  PyObject* list = PyList_New((Py_ssize_t)out.size());
  if (!list) throw Raised{};
  for (size_t i = 0; i < out.size(); ++i) {
    PyObject* o = out[i].defined() ? THPVariable_Wrap(out[i]) : (Py_INCREF(Py_None), Py_None);
    PyList_SET_ITEM(list, (Py_ssize_t)i, o);
  }
  return list;
}

// (tensor) -> whether anything waits for a gradient to arrive at this leaf: hooks of the tensor, or of the node that
// accumulates into its .grad
PyObject* has_grad_hooks(PyObject* const* a) {
  const Tensor& t = tensor(a[0]);
  bool any = !torch::autograd::impl::hooks(t).empty() || torch::autograd::impl::post_acc_grad_hooks(t) != nullptr;
  if (const auto node = torch::autograd::impl::try_get_grad_accumulator(t))
    any = any || !node->pre_hooks().empty() || !node->post_hooks().empty() || !node->tensor_pre_hooks().empty();
  return PyBool_FromLong(any);
}

}  // namespace

PyMethodDef step_methods[] = {SECO_METHOD("step_new", step_new, 2),   SECO_METHOD("step_infer", step_infer, 7),
                              SECO_METHOD("step_zero", step_zero, 1), SECO_METHOD("step_train", step_train, 10),
                              SECO_METHOD("step_result", step_result, 1), SECO_METHOD("step_grads", step_grads, 1), SECO_METHOD("has_grad_hooks", has_grad_hooks, 1), {nullptr, nullptr, 0, nullptr}};

}  // namespace seco_ext
