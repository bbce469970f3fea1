// fp32 kernels for chunked causal attention: forward, dQ and dK/dV on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 products and sums, 157 TFLOP/s on this GPU), for any head_dim that is a multiple of 4
// up to 256.
//
// The fp32 configuration is small (cfg1: 4 heads, 256-row chunks, 1024 tokens), so what bounds it is how much of the
// GPU a call can occupy and the length of the dependent chains, not bandwidth: a workgroup owns only 16 query rows
// (forward, dQ) or 16 cache rows (dK/dV), its wavefronts divide the other dimension among themselves, and their partial
// results are combined through LDS in wavefront order (one writer per element, fixed order: reproducible).  Operands
// come straight from global memory (they are a few hundred KB, L2-resident) as 16-byte loads in the two forms below,
// with no LDS staging and no barrier in the loop.
//
// Operand forms (lane l, i = l % 16, g = l / 16; a contraction may visit its index in any order, so each lane takes
// four consecutive elements with one load and instruction j uses the j-th):
//   row form  X[r0 + i][16 t + 4 g + j]   contraction over head_dim, instruction (t, j)
//   col form  X[r0 + 4 g + r][64 n + 4 i + j]   contraction over rows, instruction r; output (n, j)
// A score tile computed as (rows of X) x (rows of Y) leaves lane l with Y row i and X rows 4 g + r, r = 0..3: exactly
// the second operand of the col form.  An output tile holds head_dim 64 n + 16 g + 4 r + j for the lane's row i.
// Positions past head_dim are read from the row's last four elements and multiplied by zero (row form) or dropped
// (col form); rows past the end are clamped and masked.
// Per call of cfg1, on average: forward 13 us, backward 18 us (the fp32 matrix rate of the CUs that have a row tile: a
// wavefront's MFMAs of one 16 x 16 block take 1000 - 2000 cycles).
#include "mfma_tiles.h"
#include "seco_internal.h"

namespace seco {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kRows = 16;   // rows a workgroup owns
// blocks of 16 that every head_dim that NT blocks are used for (SECO_F32_DISPATCH) fills; past head_dim lie later ones
template <int NT> constexpr int kWhole = NT <= 2 ? 0 : NT <= 4 ? 2 : NT <= 5 ? 4 : NT <= 8 ? 5 : NT <= 12 ? 8 : 12;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// row form of the row at `row` (this lane's), NT blocks of 16 elements, the last of them repeating the row's end past
// head_dim.  (No branch around a load: a block whose condition differs over the lanes made the compiler wait for
// every load before the next one was issued.)
template <int NT>
__device__ __forceinline__ void load_rows(const float* row, int D, int g, f32x4 (&x)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) x[t] = load4(row + min(16 * t + 4 * g, D - 4));
}
// ... to be kept as the second operand of a score tile: zero past head_dim
template <int NT>
__device__ __forceinline__ void mask_kept(int D, int g, f32x4 (&x)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) x[t][j] = 16 * t + 4 * g < D ? x[t][j] : 0.f;
}
// (two chains: a tile's products are dependent, 32 cycles each)
template <int NT>
__device__ __forceinline__ f32x4 score(const f32x4 (&x)[NT], const f32x4 (&kept)[NT]) {
  f32x4 s[2] = {zero4(), zero4()};
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j & 1] = mfma4(x[t][j], kept[t][j], s[j & 1]);
  return s[0] + s[1];
}
// col form: rows first + 4 g + r, clamped to `last`
template <int ND>
__device__ __forceinline__ void load_cols(const float* base, int64_t stride, int first, int last, int D, int i, int g,
                                          f32x4 (&x)[4][ND]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float* row = base + (int64_t)min(first + 4 * g + r, last) * stride;
#pragma unroll
    for (int n = 0; n < ND; ++n) x[r][n] = load4(row + min(64 * n + 4 * i, D - 4));
  }
}
template <int ND>
__device__ __forceinline__ void accumulate(const f32x4 (&x)[4][ND], const f32x4& w, f32x4 (&acc)[ND][4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int n = 0; n < ND; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[n][j] = mfma4(x[r][n][j], w[r], acc[n][j]);
}
template <int ND>
__device__ __forceinline__ void clear(f32x4 (&acc)[ND][4]) {
#pragma unroll
  for (int n = 0; n < ND; ++n)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[n][j] = zero4();
}
// LDS image of a workgroup's partial outputs: [wavefront][row i][64 ND] floats, rows padded by 4 floats
template <int ND> constexpr int kPartRow = 64 * ND + 4;
template <int ND>
__device__ __forceinline__ void store_part(float* part, int w, int i, int g, const f32x4 (&acc)[ND][4], float scale) {
  float* row = part + (w * kRows + i) * kPartRow<ND>;
#pragma unroll
  for (int n = 0; n < ND; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4 v = {acc[n][0][r] * scale, acc[n][1][r] * scale, acc[n][2][r] * scale, acc[n][3][r] * scale};
      *reinterpret_cast<f32x4*>(row + 64 * n + 16 * g + 4 * r) = v;
    }
}
// row form -> col form of 16 rows, through a wavefront's own part of that image (a wavefront's LDS accesses are in order)
template <int ND, int NT>
__device__ __forceinline__ void turn(float* own, const f32x4 (&x)[NT], int i, int g, f32x4 (&c)[4][ND]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(own + i * kPartRow<ND> + 16 * t + 4 * g) = x[t];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int n = 0; n < ND; ++n) c[r][n] = load4(own + (4 * g + r) * kPartRow<ND> + 64 * n + 4 * i);
}
// sum over the wavefronts, in order, of row i's elements d .. d + 3
template <int ND, int NW>
__device__ __forceinline__ f32x4 sum_part(const float* part, int i, int d) {
  f32x4 s = zero4();
#pragma unroll
  for (int w = 0; w < NW; ++w) s += load4(part + (w * kRows + i) * kPartRow<ND> + d);
  return s;
}

// O = softmax(s Q K^T) V and LSE.  NB column blocks of 16 per step and wavefront.
template <int NT, int NB, int NW>
__global__ __launch_bounds__(NW * 64) void fwd_f32_kernel(AttnParams p) {
  constexpr int ND = (NT + 3) / 4;
  extern __shared__ float part[];                       // partial O; then (reference, sum) per wavefront and row
  float* ml = part + NW * kRows * kPartRow<ND>;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int r0 = (gridDim.x - 1 - blockIdx.x) * kRows, h = blockIdx.y, b = blockIdx.z, D = p.D;
  const float* K = static_cast<const float*>(p.k) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const float* V = static_cast<const float*>(p.v) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const int qpos = p.q_start + r0 + i, kv_end = p.q_start + min(r0 + kRows, p.C);
  f32x4 qf[NT];
  load_rows<NT>(static_cast<const float*>(p.q) + b * p.qs[0] + h * p.qs[1] + (int64_t)min(r0 + i, p.C - 1) * p.qs[2], D, g, qf);
  mask_kept<NT>(D, g, qf);
  const float c = p.scale * kLog2e;
  float m = -INFINITY, l = 0.f;                         // m in log2 units; l: this lane's share of the row's sum
  f32x4 o[ND][4];
  clear<ND>(o);
  for (int c0 = w * 16 * NB; c0 < kv_end; c0 += NW * 16 * NB) {
    f32x4 s[NB], vx[NB][4][ND];
    {
      f32x4 kx[NB][NT];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) load_rows<NT>(K + (int64_t)min(c0 + 16 * nb + i, kv_end - 1) * p.kvs[2], D, g, kx[nb]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) load_cols<ND>(V, p.kvs[2], c0 + 16 * nb, kv_end - 1, D, i, g, vx[nb]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) s[nb] = score<NT>(kx[nb], qf);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[nb][r] = c0 + 16 * nb + 4 * g + r <= qpos ? s[nb][r] * c : -INFINITY;
        mx = fmaxf(mx, s[nb][r]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32)));
    const float ref = mx == -INFINITY ? 0.f : mx;       // a row that has seen nothing yet
    const float alpha = fast_exp2(m - ref);
    m = mx;
    l *= alpha;
#pragma unroll
    for (int n = 0; n < ND; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) o[n][j] *= alpha;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[nb][r] = fast_exp2(s[nb][r] - ref);
        l += s[nb][r];
      }
      accumulate<ND>(vx[nb], s[nb], o);
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  store_part<ND>(part, w, i, g, o, 1.f);
  if (g == 0) {
    ml[(w * kRows + i) * 2] = m;
    ml[(w * kRows + i) * 2 + 1] = l;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kRows * ND * 16; e += NW * 64) {
    const int row = e / (ND * 16), d = 4 * (e % (ND * 16));
    if (r0 + row >= p.C || d >= D) continue;
    float M = -INFINITY;
#pragma unroll
    for (int v = 0; v < NW; ++v) M = fmaxf(M, ml[(v * kRows + row) * 2]);   // finite: column 0 is always visible
    float L = 0.f;
    f32x4 acc = zero4();
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      const float a = fast_exp2(ml[(v * kRows + row) * 2] - M);
      L += a * ml[(v * kRows + row) * 2 + 1];
      acc += a * load4(part + (v * kRows + row) * kPartRow<ND> + d);
    }
    float* out = static_cast<float*>(p.o_out) + b * p.os[0] + h * p.os[1] + (int64_t)(r0 + row) * p.os[2] + d;
    *reinterpret_cast<f32x4*>(out) = acc * (1.f / L);
    if (d == 0) p.lse[((int64_t)b * p.Hq + h) * p.C + r0 + row] = (M + __log2f(L)) * kLn2;
  }
}

// The backward of a chunk in one launch: the first n_dq workgroups own 16 query rows each (dQ), the others 16 cache rows
// (dK/dV); neither needs the other's results, since both take rowsum(dO * O) from the O and dO rows they hold anyway.
// (As three launches - rowsum, dQ, dK/dV - a call of cfg1 took 35 us, each launch 3 - 4 us before its first load returns
// and on a quarter of the CUs.)  A row operand that is also needed in col form is turned through LDS instead of being
// loaded twice: the loads are what bounds a workgroup's loop (64 bytes per clock and CU).

// dQ = s * sum over the runs of cache rows in `seg` of w * dS K (one run with weight 1 over all visible rows: the exact dQ)
template <int NT, int NW>
__device__ __forceinline__ void dq_f32(const AttnParams& p, const SegTable& seg, int item, float* part) {
  constexpr int ND = (NT + 3) / 4;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int n_rt = (p.C + kRows - 1) / kRows, rt = item / (p.Hq * p.B), bh = item - rt * p.Hq * p.B, b = bh / p.Hq, h = bh - b * p.Hq;
  const int r0 = (n_rt - 1 - rt) * kRows, D = p.D;      // the rows that see most first
  const float* K = static_cast<const float*>(p.k) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const float* V = static_cast<const float*>(p.v) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const int row = min(r0 + i, p.C - 1), qpos = p.q_start + r0 + i, kv_end = p.q_start + min(r0 + kRows, p.C);
  f32x4 qf[NT], dof[NT], of[NT];
  const int64_t orow = b * p.os[0] + h * p.os[1] + (int64_t)row * p.os[2];
  load_rows<NT>(static_cast<const float*>(p.q) + b * p.qs[0] + h * p.qs[1] + (int64_t)row * p.qs[2], D, g, qf);
  load_rows<NT>(static_cast<const float*>(p.d_o) + orow, D, g, dof);
  load_rows<NT>(static_cast<const float*>(p.o) + orow, D, g, of);
  const float lse = p.lse[((int64_t)b * p.Hq + h) * p.C + row] * kLog2e, c = p.scale * kLog2e;
  mask_kept<NT>(D, g, qf);
  mask_kept<NT>(D, g, dof);
  float delta = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) delta += of[t][j] * dof[t][j];
  delta += __shfl_xor(delta, 16);
  delta += __shfl_xor(delta, 32);
  float* own = part + w * kRows * kPartRow<ND>;
  f32x4 dq[ND][4];
  clear<ND>(dq);
  int next = w;                                         // blocks of all runs are dealt to the wavefronts in turn
  for (int si = 0; si < seg.n; ++si) {
    const int end = min(kv_end, seg.col_end[si]), begin = seg.col_begin[si];
    if (begin >= end) break;
    const float wt = seg.weight[si];
    int c0 = begin + 16 * next;
    for (; c0 < end; c0 += 16 * NW) {
      f32x4 kx[NT], vx[NT], kc[4][ND], ds;
      const int64_t at = (int64_t)min(c0 + i, end - 1) * p.kvs[2];
      load_rows<NT>(K + at, D, g, kx);
      load_rows<NT>(V + at, D, g, vx);
      const f32x4 s = score<NT>(kx, qf), dp = score<NT>(vx, dof);
      turn<ND, NT>(own, kx, i, g, kc);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = c0 + 4 * g + r;
        const float pr = col <= qpos && col < end ? fast_exp2(__builtin_fmaf(s[r], c, -lse)) : 0.f;
        ds[r] = wt * (pr * (dp[r] - delta));
      }
      accumulate<ND>(kc, ds, dq);
    }
    next = (c0 - begin) / 16 - (end - begin + 15) / 16;   // this wavefront's next block, counted from the run's end
  }
  store_part<ND>(part, w, i, g, dq, 1.f);
  __syncthreads();
  for (int e = threadIdx.x; e < kRows * ND * 16; e += NW * 64) {
    const int rr = e / (ND * 16), d = 4 * (e % (ND * 16));
    if (r0 + rr >= p.C || d >= D) continue;
    float* out = static_cast<float*>(p.d_q) + b * p.qs[0] + h * p.qs[1] + (int64_t)(r0 + rr) * p.qs[2] + d;
    *reinterpret_cast<f32x4*>(out) = p.scale * sum_part<ND, NW>(part, rr, d);
  }
}

// gK[c] += w * s * sum_h dS^T Q, gV[c] += w * sum_h P^T dO for 16 cache rows (exclusive owner); the wavefronts divide
// the (query head, block of 16 query rows) pairs that see them.
template <int NT, int NW>
__device__ __forceinline__ void dkdv_f32(const AttnParams& p, const SegTable& seg, int item, float* part) {
  constexpr int ND = (NT + 3) / 4;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int tile = item / (p.Hkv * p.B), bh = item - tile * p.Hkv * p.B, b = bh / p.Hkv, kvh = bh - b * p.Hkv, D = p.D;
  int si = 0;
  while (si + 1 < seg.n && tile >= seg.tile_begin[si + 1]) ++si;
  const int c0 = seg.col_begin[si] + (tile - seg.tile_begin[si]) * kRows, c_end = seg.col_end[si];
  const float weight = seg.weight[si];
  f32x4 kf[NT], vf[NT];
  const int64_t at = b * p.kvs[0] + kvh * p.kvs[1] + (int64_t)min(c0 + i, c_end - 1) * p.kvs[2];
  load_rows<NT>(static_cast<const float*>(p.k) + at, D, g, kf);
  load_rows<NT>(static_cast<const float*>(p.v) + at, D, g, vf);
  mask_kept<NT>(D, g, kf);
  mask_kept<NT>(D, g, vf);
  const float c = p.scale * kLog2e;
  float* own = part + w * kRows * kPartRow<ND>;
  f32x4 dk[ND][4], dv[ND][4];
  clear<ND>(dk);
  clear<ND>(dv);
  // the group's first head (per-head products of 64-bit strides in the loop would cost scalar registers that are not there)
  const int h0 = kvh * p.G;
  const float* q_group = static_cast<const float*>(p.q) + b * p.qs[0] + h0 * p.qs[1];
  const float* do_group = static_cast<const float*>(p.d_o) + b * p.os[0] + h0 * p.os[1];
  const float* o_group = static_cast<const float*>(p.o) + b * p.os[0] + h0 * p.os[1];
  const float* lse_group = p.lse + ((int64_t)b * p.Hq + h0) * p.C;
  const int rb0 = max(0, c0 - p.q_start) / kRows, n_rb = (p.C + kRows - 1) / kRows - rb0;   // row blocks that see the tile
  for (int it = w; it < n_rb * p.G; it += NW) {
    const int hg = it / n_rb, q0 = (rb0 + it - hg * n_rb) * kRows, row = min(q0 + i, p.C - 1);
    const int64_t orow = hg * p.os[1] + (int64_t)row * p.os[2];
    f32x4 pr, ds, x[4][ND], qx[NT], dox[NT];
    // (the longest rows: Q is requested when O is no longer needed; with all three in registers beside K, V and both
    // sums 31 of them went to memory, in every iteration)
    constexpr bool kLate = NT > 12;
    const float* qrow = q_group + hg * p.qs[1] + (int64_t)row * p.qs[2];
    if (!kLate) load_rows<NT>(qrow, D, g, qx);
    load_rows<NT>(do_group + orow, D, g, dox);
    const float lse = lse_group[(int64_t)hg * p.C + row] * kLog2e;
    float delta = 0.f;                                  // of row i
    {
      f32x4 ox[NT];
      load_rows<NT>(o_group + orow, D, g, ox);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) delta += t < kWhole<NT> || 16 * t + 4 * g < D ? ox[t][j] * dox[t][j] : 0.f;
    }
    if (kLate) {
      asm volatile("" : "+v"(delta) : : "memory");
      load_rows<NT>(qrow, D, g, qx);
    }
    delta += __shfl_xor(delta, 16);
    delta += __shfl_xor(delta, 32);
    const f32x4 s = score<NT>(qx, kf), dp = score<NT>(dox, vf);
    turn<ND, NT>(own, dox, i, g, x);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int qr = q0 + 4 * g + r;
      const bool seen = qr < p.C && c0 + i <= p.q_start + qr;
      const float row_lse = __shfl(lse, 4 * g + r), row_delta = __shfl(delta, 4 * g + r);   // (by all lanes)
      pr[r] = seen ? fast_exp2(__builtin_fmaf(s[r], c, -row_lse)) : 0.f;
      ds[r] = pr[r] * (dp[r] - row_delta);
    }
    accumulate<ND>(x, pr, dv);
    turn<ND, NT>(own, qx, i, g, x);
    accumulate<ND>(x, ds, dk);
  }
  // gV's elements, then gK's; their old values are requested before the partial sums are exchanged
  constexpr int kQuads = kRows * ND * 16, kPer = (2 * kQuads + NW * 64 - 1) / (NW * 64);
  auto target = [&](int e, float*& q, float& wt) {      // false: nothing there
    const int pass = e / kQuads, rr = (e % kQuads) / (ND * 16), d = 4 * (e % (ND * 16));
    q = (pass ? p.gk : p.gv) + b * p.gs[0] + kvh * p.gs[1] + (int64_t)min(c0 + rr, c_end - 1) * p.gs[2] + min(d, D - 4);
    wt = pass ? weight * p.scale : weight;
    return e < 2 * kQuads && c0 + rr < c_end && d < D;
  };
  f32x4 old[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    float *q, wt;
    target(min((int)threadIdx.x + k * NW * 64, 2 * kQuads - 1), q, wt);
    old[k] = load4(q);
  }
  store_part<ND>(part, w, i, g, dv, 1.f);
  store_part<ND>(part + NW * kRows * kPartRow<ND>, w, i, g, dk, 1.f);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = threadIdx.x + k * NW * 64;
    float *q, wt;
    if (!target(e, q, wt)) continue;
    *reinterpret_cast<f32x4*>(q) = old[k] + wt * sum_part<ND, NW>(part + e / kQuads * (NW * kRows * kPartRow<ND>),
                                                                  (e % kQuads) / (ND * 16), 4 * (e % (ND * 16)));
  }
}

template <int NT, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_f32_kernel(AttnParams p, SegTable dq_runs, SegTable seg, int n_dq) {
  extern __shared__ float part[];                       // two images of partial outputs
  if ((int)blockIdx.x < n_dq)
    dq_f32<NT, NW>(p, dq_runs, blockIdx.x, part);
  else
    dkdv_f32<NT, NW>(p, seg, blockIdx.x - n_dq, part);
}

// Wavefronts per workgroup: as many as the register file holds of the kernel at that head_dim.
template <int NT> constexpr int kFwdWaves = NT <= 4 ? 16 : NT <= 8 ? 8 : 4;
template <int NT> constexpr int kBwdWaves = NT <= 4 ? 8 : 4;

template <int NT>
int fwd_nt(const AttnParams& p, hipStream_t s) {
  constexpr int NW = kFwdWaves<NT>, smem = NW * kRows * (kPartRow<(NT + 3) / 4> + 2) * 4;
  auto kern = fwd_f32_kernel<NT, (NT > 4 && NT <= 8 ? 2 : 1), NW>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  ProfScope prof(kKernelFwd, s);
  hipLaunchKernelGGL(kern, dim3((p.C + kRows - 1) / kRows, p.Hq, p.B), dim3(NW * 64), smem, s, p);
  return launch_status();
}
template <int NT>
int bwd_nt(const AttnParams& p, const SegTable& dq_runs, const SegTable& seg, bool dq, hipStream_t s) {
  constexpr int NW = kBwdWaves<NT>, smem = 2 * NW * kRows * kPartRow<(NT + 3) / 4> * 4;
  auto kern = bwd_f32_kernel<NT, NW>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  const int64_t n_dq = dq ? (int64_t)((p.C + kRows - 1) / kRows) * p.Hq * p.B : 0;
  const int64_t total = n_dq + (int64_t)seg.tile_begin[seg.n] * p.Hkv * p.B;
  if (total > 0x7fffffff) return SECO_ERR_TOO_LARGE;
  ProfScope prof(n_dq == 0 ? kKernelDkdv : seg.tile_begin[seg.n] ? kKernelBwd : kKernelDq, s);
  hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(NW * 64), smem, s, p, dq_runs, seg, (int)n_dq);
  return launch_status();
}

}  // namespace

// head_dim in blocks of 16: the sizes in use exactly, others by the next larger one
#define SECO_F32_DISPATCH(F, ...)                       \
  switch ((p.D + 15) / 16) {                            \
    case 1: case 2: return F<2>(__VA_ARGS__);           \
    case 3: case 4: return F<4>(__VA_ARGS__);           \
    case 5: return F<5>(__VA_ARGS__);                   \
    case 6: case 7: case 8: return F<8>(__VA_ARGS__);   \
    case 9: case 10: case 11: case 12: return F<12>(__VA_ARGS__); \
    default: return F<16>(__VA_ARGS__);                 \
  }

int launch_fwd_f32(const AttnParams& p, hipStream_t s) { SECO_F32_DISPATCH(fwd_nt, p, s) }

// Both passes of the fp32 backward are one launch: dQ is noted in p.pending and goes out with dK/dV (launch_dkdv_f32;
// with an empty table when there are no cache rows to cover).  rowsum(dO * O) is taken from O and dO where it is used.
int launch_dq_f32(const AttnParams& p, const SegTable* dq_runs, hipStream_t) {
  SegTable& runs = p.pending->runs;
  runs = SegTable{};
  runs.n = 1;
  runs.col_end[0] = p.q_start + p.C;
  runs.weight[0] = 1.f;
  if (dq_runs) runs = *dq_runs;
  p.pending->dq = true;
  return SECO_OK;
}

int launch_dkdv_f32(const AttnParams& p, const SegTable& seg, hipStream_t s) {
  static_assert(kColTileF32 == kRows, "one workgroup per column tile");
  const bool dq = p.pending->dq;
  p.pending->dq = false;
  if (!dq && seg.tile_begin[seg.n] == 0) return SECO_OK;
  SECO_F32_DISPATCH(bwd_nt, p, p.pending->runs, seg, dq, s)
}

}  // namespace seco
