// dQ of one chunk, bf16: the launch shapes of the kernel in bwd_dq_body.h.
#include <algorithm>

#include "bwd_dq_kernel.h"

namespace seco {
namespace {

template <int KH, int SPLIT>
int launch(const AttnParams& p, const SegTable& seg, bool sparse, int n_mtiles, int total, hipStream_t s) {
  return sparse ? launch_dq_kernel<KH, SPLIT, true, DqProducts16>(p, seg, n_mtiles, total, s)
                : launch_dq_kernel<KH, SPLIT, false, DqProducts16>(p, seg, n_mtiles, total, s);
}

// Row tiles that were divided (kShares): dQ = scale * (sum of the shares, in order).  A thread: four elements of a row.
__global__ __launch_bounds__(256) void dq_shares_merge_kernel(AttnParams p, int n_cut) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int tile = blockIdx.x >> 4, unit = tile / n_cut, pos = tile - unit * n_cut, lr = (blockIdx.x & 15) * 8 + (threadIdx.x >> 5);
  const int v = (n_cut - 1 - pos) * BM + lr, hg = v / p.Cpad, row = v - hg * p.Cpad, d = (threadIdx.x & 31) * 4;
  if (hg >= p.G || row >= p.C) return;
  const float* src = p.part + ((int64_t)tile * p.n_splits * BM + lr) * kHeadDim + d;
  f32x4 x[kMaxRowShares], sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < kMaxRowShares; ++k) x[k] = *reinterpret_cast<const f32x4*>(src + (int64_t)min(k, p.n_splits - 1) * BM * kHeadDim);
#pragma unroll
  for (int k = 0; k < kMaxRowShares; ++k)
    if (k < p.n_splits) sum += x[k];
  const int kvh = unit % p.Hkv, b = unit / p.Hkv;
  const bf16x4 out = {(__bf16)(sum[0] * p.scale), (__bf16)(sum[1] * p.scale), (__bf16)(sum[2] * p.scale), (__bf16)(sum[3] * p.scale)};
  *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.d_q) + b * p.qs[0] + (int64_t)(kvh * p.G + hg) * p.qs[1] + row * p.qs[2] + d) = out;
}

}  // namespace

// runs == nullptr: all visible cache rows, weight 1.  The pass is left for the dK/dV launcher, which may be able to run
// both at once.
int launch_dq_bf16(const AttnParams& p, const SegTable* runs, hipStream_t s) {
  if (!p.pending) return launch_dq_bf16_now(p, runs, true, s);
  p.pending->dq = true;
  p.pending->sparse = runs != nullptr;
  if (runs) p.pending->runs = *runs;
  return SECO_OK;
}

int launch_dq_bf16_now(const AttnParams& p, const SegTable* runs, bool alone, hipStream_t s) {
  SegTable none = {};
  const SegTable& seg = runs ? *runs : none;
  // (over selected columns: as many shares as those are worth, not the whole cache)
  const int n_splits = runs && p.n_splits > 1 ? std::min(p.n_splits, split_count(split_plan(p.B, p.Hkv, p.G, p.C), visited_tiles(p, *runs) * 128)) : p.n_splits;
  if (n_splits > 1) {
    const SplitPlan plan = split_plan(p.B, p.Hkv, p.G, p.C);
    AttnParams ps = p;
    ps.n_splits = n_splits;
    const int total = plan.items * n_splits;
    int rc = launch<2, kDivided>(ps, seg, runs != nullptr, plan.n_mtiles, total, s);
    return rc ? rc : launch_dq_merge(ps, s);
  }
  const int n_mtiles = (p.C + BM - 1) / BM;
  const int total = p.B * p.Hq * n_mtiles;
  if (!runs) {
    const SplitPlan plan = split_plan(p.B, p.Hkv, p.G, p.C);
    const RowShares rs = row_shares(p.B * p.Hkv, plan.n_mtiles, total, p.q_start, p.C, p.tail_bytes / (BM * kHeadDim * sizeof(float)), kDqTime);
    if (rs.shares > 1) {
      AttnParams ps = p;
      ps.rows_whole = rs.whole;
      ps.n_splits = rs.shares;
      ps.part = p.tail_part;
      const int n_cut = plan.n_mtiles - rs.whole;
      const int rc = launch_dq_kernel<2, kShares, false, DqProducts16>(ps, seg, plan.n_mtiles, p.B * p.Hkv * (rs.whole + n_cut * rs.shares), s);
      if (rc) return rc;
      ProfScope prof(kKernelMerge, s);
      hipLaunchKernelGGL(dq_shares_merge_kernel, dim3(p.B * p.Hkv * n_cut * 16), dim3(256), 0, s, ps, n_cut);
      return launch_status();
    }
  }
  if (total >= 2 * device_cus()) return launch<1, kWholeTiles>(p, seg, runs != nullptr, n_mtiles, total, s);
  return alone && dq_leaves_cus(total, (int64_t)p.B * p.Hq * p.C) ? launch_dq32_bf16(p, runs, n_mtiles, total, s) : launch<2, kWholeTiles>(p, seg, runs != nullptr, n_mtiles, total, s);
}

}  // namespace seco
