// Bandwidth-bound helpers: KV-gradient buffer zero / axpy (the gradient relay of the
// paper's appendix listing, "grad + base * scaler"), cache append and gradient read-out with and without rotary
// embedding; and the merge steps of the split forward / dQ kernels (short chunks).
#include "merge_body.h"
#include "decoder.h"
#include "rope.h"
#include "seco_internal.h"

namespace seco {
namespace {

// Row-range helpers.  A workgroup covers kRowUnroll * rpb rows of one (batch, head): `u` consecutive threads walk
// along a row (u units of 16 or 32 bytes per row, u <= 128), rpb = 256 / u rows side by side, and each thread has
// kRowUnroll rows in flight.  Rows come from blockIdx.x, (batch, head) from blockIdx.y, both with a stride loop over
// the rest; blockIdx.z selects the tensor (gK or gV, keys or values): both are handled by one launch.  All index
// arithmetic is 32-bit and per workgroup except the row number: a flat 64-bit item index, divided three times per
// item, took longer than the memory access of short row ranges (zeroing 2 x 1 MiB: 4.6 us, now 2.4).
constexpr int kRowUnroll = 4;

// base(bh) before the rows of a (batch, head); rows(row, rpb, c): rows row, row + rpb, .. and unit c are this thread's
template <typename Base, typename Rows>
__device__ __forceinline__ void for_rows(int n_bh, int u, int64_t nrows, Base base, Rows rows) {
  const int rpb = 256 / u;
  const int lr = threadIdx.x / u, c = threadIdx.x - lr * u;
  if (lr >= rpb) return;
  for (int bh = blockIdx.y; bh < n_bh; bh += gridDim.y) {
    base(bh);
    for (int64_t row = (int64_t)blockIdx.x * (rpb * kRowUnroll) + lr; row < nrows;
         row += (int64_t)gridDim.x * (rpb * kRowUnroll))
      rows(row, rpb, c);
  }
}

template <bool kAxpy>
__global__ __launch_bounds__(256) void kvgrad_kernel(float* __restrict__ dst_a, float* __restrict__ dst_b,
                                                     const float* __restrict__ src_a, const float* __restrict__ src_b,
                                                     float scale, int n_bh, int H, int d4, int64_t gs0, int64_t gs1,
                                                     int64_t gs2, int64_t r0, int64_t nrows) {
  float* __restrict__ dst = blockIdx.z ? dst_b : dst_a;
  const float* __restrict__ src = blockIdx.z ? src_b : src_a;
  int64_t at = 0;
  for_rows(n_bh, d4, nrows, [&](int bh) { at = (bh / H) * gs0 + (bh % H) * gs1 + r0 * gs2; },
           [&](int64_t row, int rpb, int c) {
    float4 x[kRowUnroll], y[kRowUnroll];
    const int64_t off = at + row * gs2 + 4 * c, step = rpb * gs2;
    if (kAxpy) {
#pragma unroll
      for (int k = 0; k < kRowUnroll; ++k)
        if (row + k * rpb < nrows) {
          x[k] = *reinterpret_cast<const float4*>(src + off + k * step);
          y[k] = *reinterpret_cast<const float4*>(dst + off + k * step);
        }
    }
#pragma unroll
    for (int k = 0; k < kRowUnroll; ++k)
      if (row + k * rpb < nrows) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (kAxpy) {
          v.x = y[k].x + scale * x[k].x;
          v.y = y[k].y + scale * x[k].y;
          v.z = y[k].z + scale * x[k].z;
          v.w = y[k].w + scale * x[k].w;
        }
        *reinterpret_cast<float4*>(dst + off + k * step) = v;
      }
  });
}

//   M = max m_s,  L = sum l_s 2^(m_s - M),  O = sum o_s 2^(m_s - M) / L,  LSE = (M + log2 L) ln 2.
// Lane i of a group loads (m, l) of splits i and i + 32 once; max, sum and the per-split weights then travel by
// cross-lane shuffles.
template <int GP, int K>
__global__ __launch_bounds__(256) void fwd_merge_kernel(AttnParams p) {
  const int64_t R = (int64_t)p.B * p.Hq * p.C;
  const int group = (threadIdx.x >> 5) % GP, l32 = threadIdx.x & 31;
  const int64_t mine = (int64_t)blockIdx.x * (8 / GP) + (threadIdx.x >> 5) / GP;
  const int64_t rowid = min(mine, R - 1);          // surplus threads of the last block repeat the last row, no store
  // (m, l) of splits l32 and l32 + 32, then the partials, all in flight together
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const f32x2* ml = reinterpret_cast<const f32x2*>(p.part_ml) + rowid;
  const f32x2 a0 = ml[min(l32, p.n_splits - 1) * R], a1 = ml[min(l32 + 32, p.n_splits - 1) * R];
  f32x4 x[K];
  load_partials<GP, K>(p.part, p.n_splits, R, rowid, group, l32, x);
  const float m0 = l32 < p.n_splits ? a0[0] : -INFINITY, s0 = l32 < p.n_splits ? a0[1] : 0.f;
  const float m1 = l32 + 32 < p.n_splits ? a1[0] : -INFINITY, s1 = l32 + 32 < p.n_splits ? a1[1] : 0.f;
  float M = fmaxf(m0, m1);
#pragma unroll
  for (int sh = 16; sh > 0; sh >>= 1) M = fmaxf(M, __shfl_xor(M, sh, 32));
  const float w0 = m0 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m0 - M);
  const float w1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m1 - M);
  float L = w0 * s0 + w1 * s1;
#pragma unroll
  for (int sh = 16; sh > 0; sh >>= 1) L += __shfl_xor(L, sh, 32);
  float4 acc;
  const bool store = merge_partials<GP, K>(x, p.n_splits, group, [&](int k) {
    const int sp = group + k * GP;
    return __shfl(sp < 32 ? w0 : w1, sp & 31, 32);
  }, acc);
  if (!store || mine >= R) return;
  const float inv = 1.f / L;
  const bf16x4 v = {(__bf16)(acc.x * inv), (__bf16)(acc.y * inv), (__bf16)(acc.z * inv), (__bf16)(acc.w * inv)};
  *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.o_out) + row_offset(p, rowid, p.os) + 4 * l32) = v;
  if (l32 == 0) p.lse[rowid] = (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
}

template <int GP, int K>
__global__ __launch_bounds__(256) void dq_merge_kernel(AttnParams p) { dq_merge_body<GP, K>(p, blockIdx.x); }

// (Loads without a condition, on a clamped row: with one the compiler waited for each before it issued the next, 18.7 us
// for 2 x 4 MiB.)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Row-range copy into the cache, 16 bytes per thread and row.  Strides arrive in units of 16 bytes.
__global__ __launch_bounds__(256) void rows_copy_kernel(u32x4* __restrict__ dst_a, u32x4* __restrict__ dst_b,
                                                        const u32x4* __restrict__ src_a, const u32x4* __restrict__ src_b,
                                                        int n_bh, int H, int C, int v16, int64_t ds0, int64_t ds1,
                                                        int64_t ds2, int64_t ss0, int64_t ss1, int64_t ss2, int64_t r0) {
  u32x4* __restrict__ dst = blockIdx.z ? dst_b : dst_a;
  const u32x4* __restrict__ src = blockIdx.z ? src_b : src_a;
  int64_t to = 0, from = 0;
  for_rows(n_bh, v16, C, [&](int bh) {
    const int b = bh / H, h = bh % H;
    to = b * ds0 + h * ds1 + r0 * ds2;
    from = b * ss0 + h * ss1;
  }, [&](int64_t row, int rpb, int c) {
    u32x4 x[kRowUnroll];
#pragma unroll
    for (int k = 0; k < kRowUnroll; ++k)
      x[k] = src[from + min(row + k * rpb, (int64_t)C - 1) * ss2 + c];
#pragma unroll
    for (int k = 0; k < kRowUnroll; ++k)
      if (row + k * rpb < C) dst[to + (row + k * rpb) * ds2 + c] = x[k];
  });
}

// Read-out of KV-gradient rows: 8 consecutive floats per thread and row (32 bytes in, 16 or 32 bytes out).
template <bool kBf16>
__global__ __launch_bounds__(256) void readout_kernel(void* __restrict__ out_a, void* __restrict__ out_b,
                                                      const float* __restrict__ g_a, const float* __restrict__ g_b,
                                                      float scaler, int n_bh, int H, int C, int d8, int64_t os0,
                                                      int64_t os1, int64_t os2, int64_t gs0, int64_t gs1, int64_t gs2,
                                                      int64_t r0) {
  void* __restrict__ out = blockIdx.z ? out_b : out_a;
  const float* __restrict__ g = blockIdx.z ? g_b : g_a;
  int64_t to = 0, from = 0;
  for_rows(n_bh, d8, C, [&](int bh) {
    const int b = bh / H, h = bh % H;
    to = b * os0 + h * os1;
    from = b * gs0 + h * gs1 + r0 * gs2;
  }, [&](int64_t row, int rpb, int c) {
    float4 x[kRowUnroll][2];
#pragma unroll
    for (int k = 0; k < kRowUnroll; ++k)
      if (row + k * rpb < C) {
        const float4* src = reinterpret_cast<const float4*>(g + from + (row + k * rpb) * gs2 + 8 * c);
        x[k][0] = src[0];
        x[k][1] = src[1];
      }
#pragma unroll
    for (int k = 0; k < kRowUnroll; ++k)
      if (row + k * rpb < C) {
        float4 a = x[k][0], e = x[k][1];
        a.x *= scaler; a.y *= scaler; a.z *= scaler; a.w *= scaler;
        e.x *= scaler; e.y *= scaler; e.z *= scaler; e.w *= scaler;
        const int64_t off = to + (row + k * rpb) * os2 + 8 * c;
        if (kBf16) {
          typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
          const bf16x8 v = {(__bf16)a.x, (__bf16)a.y, (__bf16)a.z, (__bf16)a.w, (__bf16)e.x, (__bf16)e.y, (__bf16)e.z, (__bf16)e.w};
          *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(out) + off) = v;
        } else {
          float4* d = reinterpret_cast<float4*>(static_cast<float*>(out) + off);
          d[0] = a;
          d[1] = e;
        }
      }
  });
}

// workgroups for `nrows` rows of `u` units each of n_bh (batch, head) pairs and n_tensors tensors; the kernels' stride
// loops cover what a grid dimension cannot hold
dim3 rows_grid(int64_t nrows, int u, int n_bh, int n_tensors) {
  const int64_t per = (int64_t)(256 / u) * kRowUnroll;
  const int64_t x = (nrows + per - 1) / per;
  return dim3((unsigned)(x < (1 << 20) ? x : (1 << 20)), (unsigned)(n_bh < 32768 ? n_bh : 32768), (unsigned)n_tensors);
}

}  // namespace

// The launchers take a pair of tensors (gK and gV, keys and values); a NULL member is skipped.
int launch_kvgrad_zero(float* ga, float* gb, int B, int H, int D, const int64_t gs[3], int64_t r0, int64_t r1,
                       hipStream_t s) {
  if (!ga) { ga = gb; gb = nullptr; }
  if (r1 == r0 || !ga) return SECO_OK;
  {
    ProfScope prof(kKernelKvgrad, s);
    hipLaunchKernelGGL(kvgrad_kernel<false>, rows_grid(r1 - r0, D / 4, B * H, gb ? 2 : 1), dim3(256), 0, s, ga, gb, nullptr,
                       nullptr, 0.f, B * H, H, D / 4, gs[0], gs[1], gs[2], r0, r1 - r0);
  }
  return launch_status();
}

int launch_kvgrad_axpy(float* da, float* db, const float* sa, const float* sb, float scale, int B, int H, int D,
                       const int64_t gs[3], int64_t r0, int64_t r1, hipStream_t s) {
  if (!da) { da = db; sa = sb; db = nullptr; sb = nullptr; }
  if (r1 == r0 || !da) return SECO_OK;
  {
    ProfScope prof(kKernelKvgrad, s);
    hipLaunchKernelGGL(kvgrad_kernel<true>, rows_grid(r1 - r0, D / 4, B * H, db ? 2 : 1), dim3(256), 0, s, da, db, sa, sb,
                       scale, B * H, H, D / 4, gs[0], gs[1], gs[2], r0, r1 - r0);
  }
  return launch_status();
}

int launch_rows_copy(void* da, void* db, const void* sa, const void* sb, int eb, int B, int H, int C, int D,
                     const int64_t dst_s[3], const int64_t src_s[3], int64_t r0, hipStream_t s) {
  const int per16 = 16 / eb;                  // elements per 16-byte word; strides and D are multiples of it
  const int v16 = D / per16;
  if (!da) { da = db; sa = sb; db = nullptr; sb = nullptr; }
  if (!da) return SECO_OK;
  {
    ProfScope prof(kKernelKvgrad, s);
    hipLaunchKernelGGL(rows_copy_kernel, rows_grid(C, v16, B * H, db ? 2 : 1), dim3(256), 0, s, static_cast<u32x4*>(da),
                       static_cast<u32x4*>(db), static_cast<const u32x4*>(sa), static_cast<const u32x4*>(sb), B * H, H, C,
                       v16, dst_s[0] / per16, dst_s[1] / per16, dst_s[2] / per16, src_s[0] / per16, src_s[1] / per16,
                       src_s[2] / per16, r0);
  }
  return launch_status();
}

int launch_readout(void* oa, void* ob, const float* ga, const float* gb, float scaler, bool bf16, int B, int H, int C,
                   int D, const int64_t out_s[3], const int64_t gs[3], int64_t r0, hipStream_t s) {
  if (!oa) { oa = ob; ga = gb; ob = nullptr; gb = nullptr; }
  if (!oa) return SECO_OK;
  {
    ProfScope prof(kKernelKvgrad, s);
    const dim3 grid = rows_grid(C, D / 8, B * H, ob ? 2 : 1);
    if (bf16)
      hipLaunchKernelGGL(readout_kernel<true>, grid, dim3(256), 0, s, oa, ob, ga, gb, scaler, B * H, H, C, D / 8,
                         out_s[0], out_s[1], out_s[2], gs[0], gs[1], gs[2], r0);
    else
      hipLaunchKernelGGL(readout_kernel<false>, grid, dim3(256), 0, s, oa, ob, ga, gb, scaler, B * H, H, C, D / 8,
                         out_s[0], out_s[1], out_s[2], gs[0], gs[1], gs[2], r0);
  }
  return launch_status();
}

template <typename T> struct Quad;                               // four consecutive elements, one memory access
template <> struct Quad<float> {
  float4 v;
  __device__ float get(int j) const { return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w; }
  __device__ static Quad of(const float* f) { return {make_float4(f[0], f[1], f[2], f[3])}; }
};
template <> struct Quad<__bf16> {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 v;
  __device__ float get(int j) const { return (float)v[j]; }
  __device__ static Quad of(const float* f) { return {bf16x4{(__bf16)f[0], (__bf16)f[1], (__bf16)f[2], (__bf16)f[3]}}; }
};

// Rotary position embedding of rows: out[b, h, r, :] = R(sign * theta(pos0 + r)) (scale * in[b, h, r, :]), pairs
// (i, i + D/2), theta_i = pos * base^(-2 i / D).  A thread takes four consecutive i of one row (both halves) for
// kRopeHeads heads: angles and sines (fp64; one rounding of the result) depend on the row and i only, and computing
// them once per head made the 2048 x 32-head rotation 21 us of fp64 arithmetic for 33 MB of data.  In / out element
// types are template parameters so that the same kernel serves the cache append (storage type -> storage type, rows at
// r0 of the destination), the gradient read-out (fp32 -> storage type, rows at r0 of the source) and the plain rotation.
// A second tensor pair with the same strides (the values of an append, the value gradient of a read-out) rides along
// as blockIdx.z == 1: the same rows, scaled and converted but not rotated, so that keys and values take one pass and
// one launch.
constexpr int kRopeHeads = 4;
template <typename TIn, typename TOut>
__global__ __launch_bounds__(256) void rope_rows_kernel(TOut* out, const TIn* in, TOut* plain_out, const TIn* plain_in,
                                                        int B, int H, int C,   // (out may be in)
                                                        int D, int64_t os0, int64_t os1, int64_t os2, int64_t is0,
                                                        int64_t is1, int64_t is2, int64_t out_r0, int64_t in_r0,
                                                        int64_t pos0, RopePowers powers, float sign, float scale,
                                                        int plain_from) {
  const int q4 = D / 8;                                   // groups of 4 pairs per row
  const bool plain = (int)blockIdx.z >= plain_from;       // plain_from: 1 with a rotated pair present, else 0
  if (plain) {
    out = plain_out;
    in = plain_in;
  }
  const int rpb = 256 / q4, lr = threadIdx.x / q4, grp = threadIdx.x - lr * q4;
  const int row = blockIdx.x * rpb + lr;
  if (lr >= rpb || row >= C) return;
  const int h_groups = (H + kRopeHeads - 1) / kRopeHeads;
  const TIn* src;
  TOut* dst;
  int h0;
  Quad<TIn> x[kRopeHeads][2];
  auto load = [&](int y) {
    const int b = y / h_groups;
    h0 = (y - b * h_groups) * kRopeHeads;
    src = in + b * is0 + h0 * is1 + (in_r0 + row) * is2 + grp * 4;
    dst = out + b * os0 + h0 * os1 + (out_r0 + row) * os2 + grp * 4;
#pragma unroll
    for (int k = 0; k < kRopeHeads; ++k)
      if (h0 + k < H) {
        x[k][0] = *reinterpret_cast<const Quad<TIn>*>(src + k * is1);
        x[k][1] = *reinterpret_cast<const Quad<TIn>*>(src + k * is1 + D / 2);
      }
  };
  int y = blockIdx.y;
  load(y);                                                // in flight during the fp64 arithmetic
  double sn[4], cs[4];
  if (!plain) {                                           // (uniform over the workgroup)
    rope_sines(pos0 + row, grp, powers, sn, cs);
#pragma unroll
    for (int j = 0; j < 4; ++j) sn[j] *= (double)sign;
  }
  while (true) {
#pragma unroll
    for (int k = 0; k < kRopeHeads; ++k)
      if (h0 + k < H) {
        float lo[4], hi[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          lo[j] = x[k][0].get(j) * scale;
          hi[j] = x[k][1].get(j) * scale;
          if (!plain) {
            const double a = (double)lo[j], c = (double)hi[j];
            lo[j] = (float)(a * cs[j] - c * sn[j]);
            hi[j] = (float)(c * cs[j] + a * sn[j]);
          }
        }
        *reinterpret_cast<Quad<TOut>*>(dst + k * os1) = Quad<TOut>::of(lo);
        *reinterpret_cast<Quad<TOut>*>(dst + k * os1 + D / 2) = Quad<TOut>::of(hi);
      }
    y += gridDim.y;
    if (y >= B * h_groups) break;
    load(y);
  }
}

// What a decoder layer does between its joint projection and the attention, in one launch: the query heads of qkv [B, C, (Hq + 2
// Hkv) D] rotated in place, the key heads rotated and the value heads copied to rows row0 .. of the cache; or, on the way
// back (INV), the query gradients turned back in place and the rows of gK (turned back) and gV to the key and value
// columns.  blockIdx.y: head groups of the queries, then of the keys, then of the values.  (As two launches, queries and
// cache, 512 rows of 8/2 heads take 4 us each, of which 3 are the launch and the first loads.)
// One head group of one row: this thread's four pairs of kRopeHeads heads.
template <typename TIn, typename TOut>
__device__ __forceinline__ void rope_group(TOut* dst, const TIn* src, int64_t os1, int64_t is1, int heads, int D, int grp, int64_t pos,
                                           const RopePowers& powers, double sign, bool plain) {
  Quad<TIn> x[kRopeHeads][2];
#pragma unroll
  for (int k = 0; k < kRopeHeads; ++k)
    if (k < heads) {
      x[k][0] = *reinterpret_cast<const Quad<TIn>*>(src + k * is1);
      x[k][1] = *reinterpret_cast<const Quad<TIn>*>(src + k * is1 + D / 2);
    }
  double sn[4], cs[4];
  if (!plain) {
    rope_sines(pos, grp, powers, sn, cs);
#pragma unroll
    for (int j = 0; j < 4; ++j) sn[j] *= sign;
  }
#pragma unroll
  for (int k = 0; k < kRopeHeads; ++k)
    if (k < heads) {
      float lo[4], hi[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        lo[j] = x[k][0].get(j);
        hi[j] = x[k][1].get(j);
        if (!plain) rope_pair(lo[j], hi[j], sn[j], cs[j]);
      }
      *reinterpret_cast<Quad<TOut>*>(dst + k * os1) = Quad<TOut>::of(lo);
      *reinterpret_cast<Quad<TOut>*>(dst + k * os1 + D / 2) = Quad<TOut>::of(hi);
    }
}
template <typename T, typename TG, bool INV>
__global__ __launch_bounds__(256) void rope_qkv_kernel(T* qkv, TG* k, TG* v, int Hq, int Hkv, int C, int D, int64_t ks0, int64_t ks1,
                                                       int64_t ks2, int64_t row0, RopePowers powers, int n_q, int n_kv) {
  const int q4 = D / 8, rpb = 256 / q4, lr = threadIdx.x / q4, grp = threadIdx.x - lr * q4, row = blockIdx.x * rpb + lr;
  if (lr >= rpb || row >= C) return;
  const bool is_q = (int)blockIdx.y < n_q, plain = (int)blockIdx.y >= n_q + n_kv;
  const int y = is_q ? blockIdx.y : (int)blockIdx.y - n_q - (plain ? n_kv : 0);
  const int H = is_q ? Hq : Hkv, groups = (H + kRopeHeads - 1) / kRopeHeads, b = y / groups, h0 = (y - b * groups) * kRopeHeads;
  const int heads = min(kRopeHeads, H - h0);
  const int64_t pos = row0 + row;
  const double sign = INV ? -1.0 : 1.0;
  T* here = qkv + ((int64_t)b * C + row) * ((int64_t)(Hq + 2 * Hkv) * D) + (int64_t)(h0 + (is_q ? 0 : plain ? Hq + Hkv : Hq)) * D + grp * 4;
  if (is_q) {
    rope_group(here, (const T*)here, D, D, heads, D, grp, pos, powers, sign, false);
  } else {
    TG* there = (plain ? v : k) + b * ks0 + h0 * ks1 + (row0 + row) * ks2 + grp * 4;
    if constexpr (INV)
      rope_group(here, (const TG*)there, D, ks1, heads, D, grp, pos, powers, sign, plain);
    else
      rope_group(there, (const T*)here, ks1, D, heads, D, grp, pos, powers, sign, plain);
  }
}

int launch_rope_rows(void* out, const void* in, void* plain_out, const void* plain_in, int in_kind, int out_kind, int B,
                     int H, int C, int D, const int64_t out_s[3], const int64_t in_s[3], int64_t out_r0, int64_t in_r0,
                     int64_t pos0, float base, bool inverse, float scale, hipStream_t s) {
  if (!out && !plain_out) return SECO_OK;
  const RopePowers powers = rope_powers(D, base);
  const float sign = inverse ? -1.f : 1.f;
  {
    ProfScope prof(kKernelKvgrad, s);
    // grid.z: one slice of workgroups per tensor pair present (the rotated pair first)
    const int plain_from = out ? 1 : 0;
    const int rpb = 256 / (D / 8), n_hg = B * ((H + kRopeHeads - 1) / kRopeHeads);
    const dim3 grid((C + rpb - 1) / rpb, n_hg < 32768 ? n_hg : 32768, (out ? 1u : 0u) + (plain_out ? 1u : 0u));
#define SECO_ROPE_LAUNCH(TI, TO)                                                                                       \
  hipLaunchKernelGGL((rope_rows_kernel<TI, TO>), grid, dim3(256), 0, s, static_cast<TO*>(out),                         \
                     static_cast<const TI*>(in), static_cast<TO*>(plain_out), static_cast<const TI*>(plain_in), B, H,   \
                     C, D, out_s[0], out_s[1], out_s[2], in_s[0], in_s[1], in_s[2], out_r0, in_r0, pos0, powers, sign,     \
                     scale, plain_from)
    if (in_kind == SECO_BF16 && out_kind == SECO_BF16) SECO_ROPE_LAUNCH(__bf16, __bf16);
    else if (in_kind == SECO_F32 && out_kind == SECO_BF16) SECO_ROPE_LAUNCH(float, __bf16);
    else SECO_ROPE_LAUNCH(float, float);
#undef SECO_ROPE_LAUNCH
  }
  return launch_status();
}

}  // namespace seco

extern "C" int dec_rope_qkv(int dtype, int inverse, void* qkv, void* k, void* v, const int64_t* kv_stride, int64_t B, int64_t Hq,
                            int64_t Hkv, int64_t C, int64_t D, int64_t row0, float base, void* stream) {
  using namespace seco;
  if (!qkv || !k || !v || !kv_stride) return SECO_ERR_NULL;
  if (dtype != SECO_F32 && dtype != SECO_BF16) return SECO_ERR_DTYPE;
  const int64_t n_q = B * ((Hq + kRopeHeads - 1) / kRopeHeads), n_kv = B * ((Hkv + kRopeHeads - 1) / kRopeHeads);
  if (B < 1 || Hq < 1 || Hkv < 1 || C < 1 || D < 8 || row0 < 0) return SECO_ERR_SHAPE;
  if (dtype == SECO_BF16 ? D != 128 : D % 8 != 0 || D > 256) return SECO_ERR_HEAD_DIM;
  if (!(base > 1.f) || !std::isfinite(base)) return SECO_ERR_RANGE;
  if (n_q + 2 * n_kv > 65535 || C > (int64_t)1 << 30 || B > 65535) return SECO_ERR_TOO_LARGE;
  const int64_t per = dtype == SECO_BF16 && !inverse ? 8 : 4;       // elements per 16 bytes of a cache or gradient row
  for (int i = 0; i < 3; ++i)
    if (kv_stride[i] < 0 || kv_stride[i] % per != 0) return SECO_ERR_ALIGN;
  if (((uintptr_t)qkv | (uintptr_t)k | (uintptr_t)v) & 15u) return SECO_ERR_ALIGN;
  const int rpb = 256 / (int)(D / 8);
  const dim3 grid((unsigned)((C + rpb - 1) / rpb), (unsigned)(n_q + 2 * n_kv));
  hipStream_t s = static_cast<hipStream_t>(stream);
  const RopePowers powers = rope_powers((int)D, base);
#define SECO_QKV_LAUNCH(T, TG, INV)                                                                                              \
  hipLaunchKernelGGL((rope_qkv_kernel<T, TG, INV>), grid, dim3(256), 0, s, static_cast<T*>(qkv), static_cast<TG*>(k),              \
                     static_cast<TG*>(v), (int)Hq, (int)Hkv, (int)C, (int)D, kv_stride[0], kv_stride[1], kv_stride[2], row0, powers, \
                     (int)n_q, (int)n_kv)
  ProfScope prof(kKernelKvgrad, s);
  if (dtype == SECO_BF16) {
    if (inverse) SECO_QKV_LAUNCH(__bf16, float, true);
    else SECO_QKV_LAUNCH(__bf16, __bf16, false);
  } else {
    if (inverse) SECO_QKV_LAUNCH(float, float, true);
    else SECO_QKV_LAUNCH(float, float, false);
  }
#undef SECO_QKV_LAUNCH
  return launch_status();
}

namespace seco {

#define SECO_MERGE_LAUNCH(kernel)                                                                             \
  const int64_t R = (int64_t)p.B * p.Hq * p.C;                                                                \
  ProfScope prof(kKernelMerge, s);                                                                            \
  const dim3 tpb(256);                                                                                        \
  if (p.n_splits <= 2) hipLaunchKernelGGL((kernel<1, 2>), dim3((unsigned)((R + 7) / 8)), tpb, 0, s, p);       \
  else if (p.n_splits <= 4) hipLaunchKernelGGL((kernel<1, 4>), dim3((unsigned)((R + 7) / 8)), tpb, 0, s, p);  \
  else if (p.n_splits <= 8) hipLaunchKernelGGL((kernel<1, 8>), dim3((unsigned)((R + 7) / 8)), tpb, 0, s, p);  \
  else if (p.n_splits <= 16) hipLaunchKernelGGL((kernel<2, 8>), dim3((unsigned)((R + 3) / 4)), tpb, 0, s, p); \
  else if (p.n_splits <= 32) hipLaunchKernelGGL((kernel<4, 8>), dim3((unsigned)((R + 1) / 2)), tpb, 0, s, p); \
  else hipLaunchKernelGGL((kernel<8, 8>), dim3((unsigned)R), tpb, 0, s, p);

int launch_fwd_merge(const AttnParams& p, hipStream_t s) {
  SECO_MERGE_LAUNCH(fwd_merge_kernel)
  return launch_status();
}

int launch_dq_merge(const AttnParams& p, hipStream_t s) {
  SECO_MERGE_LAUNCH(dq_merge_kernel)
  return launch_status();
}
#undef SECO_MERGE_LAUNCH

}  // namespace seco
