// Merges of partial results: rows of the split kernels, shared-out column tiles of the dK/dV pass.
#pragma once
#include "seco_internal.h"

namespace seco {
namespace {

// Merge of the partial rows of the split kernels (n_splits <= 64 of 128 fp32 each).  GP groups of 32 threads (a thread:
// 4 consecutive head_dim elements) share a row, each taking the splits sp = group, group + GP, .., at most 8 of them, so
// that all its loads are in flight at once; the groups' sums meet in LDS and are added in group order (fixed order:
// reproducible).  What bounds it is the partials' traffic (33 MB for a 32-row chunk of 32 heads in 64 splits): with one
// group per row and a loop over the splits every load waited for the one before, 23 us for that chunk; now 8.
// Launchers choose GP = the power of two from which a group has at most K = 8 splits (K less for the fewest splits).
typedef float f32x4 __attribute__((ext_vector_type(4)));
// requests the group's partials (clamped, never behind a condition that differs over the lanes: the compiler would wait for
// each load before the next one)
template <int GP, int K>
__device__ __forceinline__ void load_partials(const float* part, int n_splits, int64_t R, int64_t rowid, int group, int d4,
                                              f32x4 (&x)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k)
    x[k] = *reinterpret_cast<const f32x4*>(part + (min(group + k * GP, n_splits - 1) * R + rowid) * 128 + 4 * d4);
}
template <int GP, int K, typename Weight>
__device__ __forceinline__ bool merge_partials(const f32x4 (&x)[K], int n_splits, int group, Weight weight, float4& acc) {
  __shared__ float4 sh[GP > 1 ? 256 : 1];
  acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const float w = weight(k);                     // (a cross-lane read: every lane takes part)
    if (group + k * GP < n_splits && w != 0.f) {   // weight 0: an empty partial, never written
      acc.x += w * x[k][0];
      acc.y += w * x[k][1];
      acc.z += w * x[k][2];
      acc.w += w * x[k][3];
    }
  }
  if (GP == 1) return true;
  sh[threadIdx.x] = acc;
  __syncthreads();
  if (group != 0) return false;
#pragma unroll
  for (int k = 1; k < GP; ++k) {
    const float4 y = sh[threadIdx.x + 32 * k];     // the groups of a row are adjacent in the workgroup
    acc.x += y.x;
    acc.y += y.y;
    acc.z += y.z;
    acc.w += y.w;
  }
  return true;
}
// element offset of row `rowid` = (b * Hq + h) * C + row of a strided [B, Hq, C, 128] tensor
__device__ __forceinline__ int64_t row_offset(const AttnParams& p, int64_t rowid, const int64_t s[3]) {   // (less than 2^31 rows)
  const int bh = over((int)rowid, p.by_C), row = (int)rowid - bh * p.C, b = over(bh, p.by_Hq);
  return b * s[0] + (bh - b * p.Hq) * s[1] + (int64_t)row * s[2];
}
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Merge of the split dQ: dQ = scale * (sum of the partials), rounded to bf16.
template <int GP, int K>
__device__ __forceinline__ void dq_merge_body(const AttnParams& p, int block) {
  const int64_t R = (int64_t)p.B * p.Hq * p.C;
  const int group = (threadIdx.x >> 5) % GP, l32 = threadIdx.x & 31;
  const int64_t mine = (int64_t)block * (8 / GP) + (threadIdx.x >> 5) / GP;
  const int64_t rowid = min(mine, R - 1);
  f32x4 x[K];
  load_partials<GP, K>(p.part, p.n_splits, R, rowid, group, l32, x);
  float4 acc;
  const bool store = merge_partials<GP, K>(x, p.n_splits, group, [](int) { return 1.f; }, acc);
  if (!store || mine >= R) return;
  const bf16x4 v = {(__bf16)(acc.x * p.scale), (__bf16)(acc.y * p.scale), (__bf16)(acc.z * p.scale), (__bf16)(acc.w * p.scale)};
  *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.d_q) + row_offset(p, rowid, p.qs) + 4 * l32) = v;
}

// gK/gV of the shared-out column tiles: g += w * (sum of the shares, in order).  One thread per four consecutive
// elements of a (tile, dV or dK) pair.
template <int COLS>
__device__ __forceinline__ void tail_merge_body(const AttnParams& p, const SegTable& seg, const TailSplit& ts, int block) {
  constexpr int kBlocks = COLS * 128 / 4 / 256;       // workgroups per (tile, dV or dK)
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int quad = (block % kBlocks) * 256 + threadIdx.x, role = (block / kBlocks) & 1;
  const int st = block / (2 * kBlocks);          // shared tile, counted over all units
  const int unit = st / ts.plan.n_shared, pos = st - unit * ts.plan.n_shared;
  const int tile = seg.tile_begin[seg.n] - ts.plan.n_tiles + pos;
  int si = 0;
  while (si + 1 < seg.n && tile >= seg.tile_begin[si + 1]) ++si;
  const int row = seg.col_begin[si] + (tile - seg.tile_begin[si]) * COLS + quad / 32;
  if (row >= seg.col_end[si]) return;
  const float wf = role == 0 ? seg.weight[si] : seg.weight[si] * p.scale;
  const int kvh = unit % p.Hkv, b = unit / p.Hkv;
  float* g = (role == 0 ? p.gv : p.gk) + b * p.gs[0] + kvh * p.gs[1] + (int64_t)row * p.gs[2] + (quad % 32) * 4;
  const f32x4 old = *reinterpret_cast<const f32x4*>(g);
  const int n_slots = ts.plan.first[ts.plan.n_shared], slot = ts.plan.first[pos], hs = ts.plan.first[pos + 1] - slot;
  const float* src = ts.part + (((int64_t)unit * n_slots + slot) * 2 + role) * (int64_t)(COLS * 128) + (int64_t)quad * 4;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  for (int h = 0; h < hs; h += 4) {                   // four shares in flight; past the last one: its address again, dropped
    f32x4 x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = *reinterpret_cast<const f32x4*>(src + (int64_t)min(h + i, hs - 1) * 2 * COLS * 128);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (h + i < hs) sum += x[i];
  }
  *reinterpret_cast<f32x4*>(g) = old + wf * sum;
}

template <int COLS>
unsigned tail_merge_grid(const AttnParams& p, const TailSplit& ts) {
  return (unsigned)(p.B * p.Hkv * ts.plan.n_shared * 2 * (COLS / 8));
}

}  // namespace
}  // namespace seco
