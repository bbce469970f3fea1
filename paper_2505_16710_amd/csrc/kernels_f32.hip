// fp32 kernels for chunked causal attention: forward, dQ and dK/dV on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 products and sums, 157 TFLOP/s on this GPU), for any head_dim that is a multiple of 4
// up to 256.
//
// The fp32 configuration is small (cfg1: 4 heads, 256-row chunks, 1024 tokens), so what bounds it is how much of the
// GPU a call can occupy and the length of the dependent chains, not bandwidth: a workgroup owns only 16 query rows
// (forward, dQ) or 16 cache rows (dK/dV), its wavefronts divide the other dimension among themselves, and their partial
// results are combined through LDS in wavefront order (one writer per element, fixed order: reproducible).  Operands
// come straight from global memory (they are a few hundred KB, L2-resident) as 16-byte loads in the two forms below,
// with no LDS staging and no barrier in the loop.  The kernels before these used the vector ALU with one wavefront
// per row and a shuffle per (row, column): per call of cfg1, on average, forward 131 us (now 13), dQ 148 (20), dK/dV 87 (13).
//
// Operand forms (lane l, i = l % 16, g = l / 16; a contraction may visit its index in any order, so each lane takes
// four consecutive elements with one load and instruction j uses the j-th):
//   row form  X[r0 + i][16 t + 4 g + j]   contraction over head_dim, instruction (t, j)
//   col form  X[r0 + 4 g + r][64 n + 4 i + j]   contraction over rows, instruction r; output (n, j)
// A score tile computed as (rows of X) x (rows of Y) leaves lane l with Y row i and X rows 4 g + r, r = 0..3: exactly
// the second operand of the col form.  An output tile holds head_dim 64 n + 16 g + 4 r + j for the lane's row i.
// Positions past head_dim are read from the row's last four elements and multiplied by zero (row form) or dropped
// (col form); rows past the end are clamped and masked.
#include "mfma_tiles.h"
#include "seco_internal.h"

namespace seco {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kRows = 16;   // rows a workgroup owns

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// row form of the row at `row` (this lane's): kept as the second operand of a score tile, zero past head_dim
template <int ND>
__device__ __forceinline__ void load_kept(const float* row, int D, int g, f32x4 (&x)[4 * ND]) {
#pragma unroll
  for (int t = 0; t < 4 * ND; ++t) x[t] = 16 * t + 4 * g < D ? load4(row + 16 * t + 4 * g) : zero4();
}
template <int ND>
__device__ __forceinline__ void load_rows(const float* row, int D, int g, f32x4 (&x)[4 * ND]) {
#pragma unroll
  for (int t = 0; t < 4 * ND; ++t)
    if (16 * t < D) x[t] = load4(row + min(16 * t + 4 * g, D - 4));
}
template <int ND>
__device__ __forceinline__ f32x4 score(const f32x4 (&x)[4 * ND], const f32x4 (&kept)[4 * ND], int D) {
  f32x4 s = zero4();
#pragma unroll
  for (int t = 0; t < 4 * ND; ++t)
    if (16 * t < D) {
#pragma unroll
      for (int j = 0; j < 4; ++j) s = mfma4(x[t][j], kept[t][j], s);
    }
  return s;
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
// sum over the wavefronts, in order, of row i's elements d .. d + 3
template <int ND, int NW>
__device__ __forceinline__ f32x4 sum_part(const float* part, int i, int d) {
  f32x4 s = zero4();
#pragma unroll
  for (int w = 0; w < NW; ++w) s += load4(part + (w * kRows + i) * kPartRow<ND> + d);
  return s;
}

// O = softmax(s Q K^T) V and LSE.  NB column blocks of 16 per step and wavefront.
template <int ND, int NB, int NW>
__global__ __launch_bounds__(NW * 64) void fwd_f32_kernel(AttnParams p) {
  extern __shared__ float part[];                       // partial O; then (reference, sum) per wavefront and row
  float* ml = part + NW * kRows * kPartRow<ND>;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int r0 = (gridDim.x - 1 - blockIdx.x) * kRows, h = blockIdx.y, b = blockIdx.z, D = p.D;
  const float* K = static_cast<const float*>(p.k) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const float* V = static_cast<const float*>(p.v) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const int qpos = p.q_start + r0 + i, kv_end = p.q_start + min(r0 + kRows, p.C);
  f32x4 qf[4 * ND];
  load_kept<ND>(static_cast<const float*>(p.q) + b * p.qs[0] + h * p.qs[1] + (int64_t)min(r0 + i, p.C - 1) * p.qs[2], D, g, qf);
  const float c = p.scale * kLog2e;
  float m = -INFINITY, l = 0.f;                         // m in log2 units; l: this lane's share of the row's sum
  f32x4 o[ND][4];
  clear<ND>(o);
  for (int c0 = w * 16 * NB; c0 < kv_end; c0 += NW * 16 * NB) {
    f32x4 s[NB], vx[NB][4][ND];
    {
      f32x4 kx[NB][4 * ND];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) load_rows<ND>(K + (int64_t)min(c0 + 16 * nb + i, kv_end - 1) * p.kvs[2], D, g, kx[nb]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) load_cols<ND>(V, p.kvs[2], c0 + 16 * nb, kv_end - 1, D, i, g, vx[nb]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) s[nb] = score<ND>(kx[nb], qf, D);
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

// dQ = s * sum over the runs of cache rows in `seg` of w * dS K (one run with weight 1 over all visible rows: the
// exact dQ).
template <int ND, int NW>
__global__ __launch_bounds__(NW * 64) void dq_f32_kernel(AttnParams p, SegTable seg) {
  extern __shared__ float part[];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int r0 = (gridDim.x - 1 - blockIdx.x) * kRows, h = blockIdx.y, b = blockIdx.z, D = p.D;
  const float* K = static_cast<const float*>(p.k) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const float* V = static_cast<const float*>(p.v) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const int row = min(r0 + i, p.C - 1), qpos = p.q_start + r0 + i, kv_end = p.q_start + min(r0 + kRows, p.C);
  f32x4 qf[4 * ND], dof[4 * ND];
  load_kept<ND>(static_cast<const float*>(p.q) + b * p.qs[0] + h * p.qs[1] + (int64_t)row * p.qs[2], D, g, qf);
  load_kept<ND>(static_cast<const float*>(p.d_o) + b * p.os[0] + h * p.os[1] + (int64_t)row * p.os[2], D, g, dof);
  const int64_t stat = ((int64_t)b * p.Hq + h) * p.C + row;
  const float lse = p.lse[stat] * kLog2e, delta = p.delta[stat], c = p.scale * kLog2e;
  f32x4 dq[ND][4];
  clear<ND>(dq);
  int turn = w;                                         // blocks of all runs are dealt to the wavefronts in turn
  for (int si = 0; si < seg.n; ++si) {
    const int end = min(kv_end, seg.col_end[si]), begin = seg.col_begin[si];
    if (begin >= end) break;
    const float wt = seg.weight[si];
    int c0 = begin + 16 * turn;
    for (; c0 < end; c0 += 16 * NW) {
      f32x4 kc[4][ND], ds;
      {
        f32x4 kx[4 * ND], vx[4 * ND];
        const int64_t at = (int64_t)min(c0 + i, end - 1) * p.kvs[2];
        load_rows<ND>(K + at, D, g, kx);
        load_rows<ND>(V + at, D, g, vx);
        load_cols<ND>(K, p.kvs[2], c0, end - 1, D, i, g, kc);
        const f32x4 s = score<ND>(kx, qf, D), dp = score<ND>(vx, dof, D);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int col = c0 + 4 * g + r;
          const float pr = col <= qpos && col < end ? fast_exp2(__builtin_fmaf(s[r], c, -lse)) : 0.f;
          ds[r] = wt * (pr * (dp[r] - delta));
        }
      }
      accumulate<ND>(kc, ds, dq);
    }
    turn = (c0 - begin) / 16 - (end - begin + 15) / 16;   // this wavefront's next block, counted from the run's end
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
template <int ND, int NW>
__global__ __launch_bounds__(NW * 64) void dkdv_f32_kernel(AttnParams p, SegTable seg) {
  extern __shared__ float part[];                       // partial dV, then (behind a barrier) partial dK
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int tile = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z, D = p.D;
  int si = 0;
  while (si + 1 < seg.n && tile >= seg.tile_begin[si + 1]) ++si;
  const int c0 = seg.col_begin[si] + (tile - seg.tile_begin[si]) * kRows, c_end = seg.col_end[si];
  const float weight = seg.weight[si];
  f32x4 kf[4 * ND], vf[4 * ND];
  const int64_t at = b * p.kvs[0] + kvh * p.kvs[1] + (int64_t)min(c0 + i, c_end - 1) * p.kvs[2];
  load_kept<ND>(static_cast<const float*>(p.k) + at, D, g, kf);
  load_kept<ND>(static_cast<const float*>(p.v) + at, D, g, vf);
  const float c = p.scale * kLog2e;
  f32x4 dk[ND][4], dv[ND][4];
  clear<ND>(dk);
  clear<ND>(dv);
  const int rb0 = max(0, c0 - p.q_start) / kRows, n_rb = (p.C + kRows - 1) / kRows - rb0;   // row blocks that see the tile
  for (int it = w; it < n_rb * p.G; it += NW) {
    const int hg = it / n_rb, q0 = (rb0 + it - hg * n_rb) * kRows, h = kvh * p.G + hg;
    const float* Q = static_cast<const float*>(p.q) + b * p.qs[0] + h * p.qs[1];
    const float* dO = static_cast<const float*>(p.d_o) + b * p.os[0] + h * p.os[1];
    f32x4 pr, ds, x[4][ND];
    {
      f32x4 qx[4 * ND], dox[4 * ND];
      const int row = min(q0 + i, p.C - 1);
      load_rows<ND>(Q + (int64_t)row * p.qs[2], D, g, qx);
      load_rows<ND>(dO + (int64_t)row * p.os[2], D, g, dox);
      if (ND < 4) load_cols<ND>(dO, p.os[2], q0, p.C - 1, D, i, g, x);   // early, where registers allow
      const f32x4 s = score<ND>(qx, kf, D), dp = score<ND>(dox, vf, D);
      const int64_t stat = ((int64_t)b * p.Hq + h) * p.C;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qr = q0 + 4 * g + r, qc = min(qr, p.C - 1);
        const bool seen = qr < p.C && c0 + i <= p.q_start + qr;
        pr[r] = seen ? fast_exp2(__builtin_fmaf(s[r], c, -p.lse[stat + qc] * kLog2e)) : 0.f;
        ds[r] = pr[r] * (dp[r] - p.delta[stat + qc]);
      }
    }
    if (ND == 4) load_cols<ND>(dO, p.os[2], q0, p.C - 1, D, i, g, x);
    accumulate<ND>(x, pr, dv);
    load_cols<ND>(Q, p.qs[2], q0, p.C - 1, D, i, g, x);
    accumulate<ND>(x, ds, dk);
  }
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    if (pass) __syncthreads();
    store_part<ND>(part, w, i, g, pass ? dk : dv, pass ? p.scale : 1.f);
    __syncthreads();
    float* out = (pass ? p.gk : p.gv) + b * p.gs[0] + kvh * p.gs[1];
    for (int e = threadIdx.x; e < kRows * ND * 16; e += NW * 64) {
      const int rr = e / (ND * 16), d = 4 * (e % (ND * 16));
      if (c0 + rr >= c_end || d >= D) continue;
      f32x4* at_g = reinterpret_cast<f32x4*>(out + (int64_t)(c0 + rr) * p.gs[2] + d);
      *at_g += weight * sum_part<ND, NW>(part, rr, d);
    }
  }
}

// Wavefronts per workgroup: as many as the register file holds of the kernel at that head_dim.
template <int ND> constexpr int kFwdWaves = ND == 1 ? 16 : ND == 2 ? 8 : 4;
template <int ND> constexpr int kBwdWaves = ND == 1 ? 8 : 4;

template <int ND>
int fwd_nd(const AttnParams& p, hipStream_t s) {
  constexpr int NW = kFwdWaves<ND>, smem = NW * kRows * (kPartRow<ND> + 2) * 4;
  auto kern = fwd_f32_kernel<ND, ND == 2 ? 2 : 1, NW>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  ProfScope prof(kKernelFwd, s);
  hipLaunchKernelGGL(kern, dim3((p.C + kRows - 1) / kRows, p.Hq, p.B), dim3(NW * 64), smem, s, p);
  return launch_status();
}
template <int ND>
int dq_nd(const AttnParams& p, const SegTable& seg, hipStream_t s) {
  constexpr int NW = kFwdWaves<ND>, smem = NW * kRows * kPartRow<ND> * 4;
  auto kern = dq_f32_kernel<ND, NW>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  ProfScope prof(kKernelDq, s);
  hipLaunchKernelGGL(kern, dim3((p.C + kRows - 1) / kRows, p.Hq, p.B), dim3(NW * 64), smem, s, p, seg);
  return launch_status();
}
template <int ND>
int dkdv_nd(const AttnParams& p, const SegTable& seg, hipStream_t s) {
  constexpr int NW = kBwdWaves<ND>, smem = NW * kRows * kPartRow<ND> * 4;
  auto kern = dkdv_f32_kernel<ND, NW>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  ProfScope prof(kKernelDkdv, s);
  hipLaunchKernelGGL(kern, dim3(seg.tile_begin[seg.n], p.Hkv, p.B), dim3(NW * 64), smem, s, p, seg);
  return launch_status();
}

}  // namespace

int launch_fwd_f32(const AttnParams& p, hipStream_t s) {
  switch ((p.D + 63) / 64) {
    case 1: return fwd_nd<1>(p, s);
    case 2: return fwd_nd<2>(p, s);
    case 3: return fwd_nd<3>(p, s);
    default: return fwd_nd<4>(p, s);
  }
}

int launch_dq_f32(const AttnParams& p, const SegTable* dq_runs, hipStream_t s) {
  SegTable all = {};
  all.n = 1;
  all.col_end[0] = p.q_start + p.C;
  all.weight[0] = 1.f;
  const SegTable& seg = dq_runs ? *dq_runs : all;
  switch ((p.D + 63) / 64) {
    case 1: return dq_nd<1>(p, seg, s);
    case 2: return dq_nd<2>(p, seg, s);
    case 3: return dq_nd<3>(p, seg, s);
    default: return dq_nd<4>(p, seg, s);
  }
}

int launch_dkdv_f32(const AttnParams& p, const SegTable& seg, hipStream_t s) {
  static_assert(kColTileF32 == kRows, "one workgroup per column tile");
  if (seg.tile_begin[seg.n] == 0) return SECO_OK;
  switch ((p.D + 63) / 64) {
    case 1: return dkdv_nd<1>(p, seg, s);
    case 2: return dkdv_nd<2>(p, seg, s);
    case 3: return dkdv_nd<3>(p, seg, s);
    default: return dkdv_nd<4>(p, seg, s);
  }
}

}  // namespace seco
