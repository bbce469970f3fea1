// The 8-wavefront forward for calls between one and two rounds of row tiles: those beyond the first round have their cache
// rows divided among several workgroups (its own translation unit, as fwd4_split_bf16.hip), and the merge of the shares.
// Bound as the whole tiles are (matrix cores and exponentials); what it removes is the idle chip behind the first round.
// 1100 rows of 32 heads on 8 after 9000: 268 us undivided, 196 now (192 shares in one short round, 12.6 MB of partial sums).
#include "fwd8_kernel.h"

namespace seco {
namespace {

// O = sum of the shares, weighted by exp2(reference - largest reference), over the sum of the weighted sums; LSE.  A thread:
// four elements of a row, all shares in flight.
__global__ __launch_bounds__(256) void fwd_shares_merge_kernel(AttnParams p, int n_cut) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const int tile = blockIdx.x >> 4, unit = tile / n_cut, pos = tile - unit * n_cut, lr = (blockIdx.x & 15) * 8 + (threadIdx.x >> 5);
  const int v = (n_cut - 1 - pos) * BM + lr, hg = v / p.Cpad, row = v - hg * p.Cpad, d = (threadIdx.x & 31) * 4;
  if (hg >= p.G || row >= p.C) return;
  const int64_t first = (int64_t)tile * p.n_splits * BM + lr;
  f32x4 x[kMaxRowShares];
  f32x2 ml[kMaxRowShares];
#pragma unroll
  for (int k = 0; k < kMaxRowShares; ++k) {
    const int64_t r = first + (int64_t)min(k, p.n_splits - 1) * BM;
    ml[k] = reinterpret_cast<const f32x2*>(p.part_ml)[r];
    x[k] = *reinterpret_cast<const f32x4*>(p.part + r * kHeadDim + d);
  }
  float M = -INFINITY, L = 0.f;                // (finite: column 0 is always visible)
#pragma unroll
  for (int k = 0; k < kMaxRowShares; ++k) M = fmaxf(M, ml[k][0]);
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < kMaxRowShares; ++k)
    if (k < p.n_splits) {
      const float w = fast_exp2(ml[k][0] - M);
      L += w * ml[k][1];
      sum += w * x[k];
    }
  const int kvh = unit % p.Hkv, b = unit / p.Hkv, h = kvh * p.G + hg;
  const float inv = 1.f / L;
  const bf16x4 out = {(__bf16)(sum[0] * inv), (__bf16)(sum[1] * inv), (__bf16)(sum[2] * inv), (__bf16)(sum[3] * inv)};
  *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.o_out) + b * p.os[0] + (int64_t)h * p.os[1] + row * p.os[2] + d) = out;
  if (d == 0) p.lse[((int64_t)b * p.Hq + h) * p.C + row] = (M + __log2f(L)) * kLn2;
}

}  // namespace

int launch_fwd8_shares_bf16(const AttnParams& p, int n_mtiles, hipStream_t s) {
  const int n_cut = n_mtiles - p.rows_whole;
  const int rc = launch_fwd8<kShares>(p, n_mtiles, p.B * p.Hkv * (p.rows_whole + n_cut * p.n_splits), s);
  if (rc) return rc;
  ProfScope prof(kKernelMerge, s);
  hipLaunchKernelGGL(fwd_shares_merge_kernel, dim3(p.B * p.Hkv * n_cut * 16), dim3(256), 0, s, p, n_cut);
  return launch_status();
}

}  // namespace seco
