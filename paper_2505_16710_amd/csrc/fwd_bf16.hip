// Forward of one chunk, bf16: which kernel a call takes, and the 8-wavefront kernel's plain instantiation.
#include "fwd8_kernel.h"

namespace seco {

int launch_fwd_bf16(const AttnParams& p, hipStream_t s) {
  // (p.part: partial results of a divided cache; with p.tail_bytes, of the row tiles beyond one round)
  const int max_splits = p.part && p.tail_bytes == 0 ? split_plan(p.B, p.Hkv, p.G, p.C).max_splits : 1;
  if (fwd_small_pays(p, max_splits)) return launch_fwd_small_bf16(p, max_splits, s);
  if (p.n_splits > 1) {
    const SplitPlan plan = split_plan(p.B, p.Hkv, p.G, p.C);
    int rc = launch_fwd8_split_bf16(p, plan.n_mtiles, plan.items * p.n_splits, s);
    return rc ? rc : launch_fwd_merge(p, s);
  }
  const int n_mtiles = (p.C + BM - 1) / BM;
  const int total = p.B * p.Hq * n_mtiles;
  if (p.tail_bytes > 0) {
    const SplitPlan plan = split_plan(p.B, p.Hkv, p.G, p.C);
    const RowShares rs = row_shares(p.B * p.Hkv, plan.n_mtiles, total, p.q_start, p.C, p.tail_bytes / (BM * kHeadDim * sizeof(float)), kFwdTime);
    if (rs.shares > 1) {
      AttnParams ps = p;
      ps.rows_whole = rs.whole;
      ps.n_splits = rs.shares;
      return launch_fwd8_shares_bf16(ps, plan.n_mtiles, s);
    }
  }
  // fewer row tiles than two per CU: use the 8-wavefront shape so that every SIMD still has two wavefronts
  return total < 2 * device_cus() ? launch_fwd8<kWholeTiles>(p, n_mtiles, total, s) : launch_fwd4_bf16(p, n_mtiles, total, s);
}

}  // namespace seco
