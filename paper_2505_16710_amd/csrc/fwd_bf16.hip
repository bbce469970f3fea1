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
  // Row tiles for two workgroups of four wavefronts on every CU; or for two on three CUs of five, against caches long enough that
  // what the other CUs idle is less than what that kernel is the faster by (us, 8 -> 4 wavefronts; 1664, 1792, 1920 rows at 9000 of
  // 32/8 heads 264 -> 255, 275 -> 266, 288 -> 279, 1920 at 30000 858 -> 829; but 1500 at 9000 232 -> 242, 1920 at 1000 65 ->
  // 68).  There the tiles that share a CU have to be of much the same length, or a long and a short one: a chunk of at most half of
  // what precedes it (6700 at 6700 of 8/8 275 -> 281), one KV head to an XCD (16 of them and batches, 1750 rows at 5000 171 -> 174).
  const int cus = device_cus();
  if (total >= 2 * cus || (5 * total >= 8 * cus && p.q_start >= 2400 && p.q_start >= 2 * p.C && p.B * p.Hkv <= 8))
    return launch_fwd4_bf16(p, n_mtiles, total, s);
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
  // fewer: the 8-wavefront shape, so that every SIMD still has two wavefronts
  return launch_fwd8<kWholeTiles>(p, n_mtiles, total, s);
}

}  // namespace seco
