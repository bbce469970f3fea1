// dQ and dK/dV of a short call in one launch.
//
// A backward call with few rows and cache tiles is two passes of 10 - 25 us one after the other, each on a part of the chip
// and each with 6 - 9 us before its first product and behind its last.  The passes do not need each other's results: all
// that dK/dV takes from dQ are the row statistics, which are cheap enough to be computed twice for a short call (from the
// O and dO rows of a stage; OWN in bwd_dkdv_body.h).  So the workgroups of both are one grid, a third as many launches deep.
// Kernel times of a call with its merges, two launches -> one, in us (Hq/Hkv, chunk at position):
//   8/8  32 at 0     18.0 -> 10.5     32/8 128 at 1024   41.7 -> 30.3
//   8/8  32 at 1024  25.4 -> 16.8     32/8 256 at 0      34.6 -> 23.3
//   8/8 128 at 512   26.9 -> 17.7     32/8 256 at 2048   65.8 -> 54.2
//   16/2 184 at 736  43.6 -> 31.2
// What bounds it now: one workgroup's prologue, 1 - 10 iterations and epilogue, at one workgroup per CU.
#include <algorithm>

#include "bwd_dkdv_body.h"
#include "bwd_dq_body.h"

namespace seco {
namespace {

using Cfg = DkdvCfg<kColTileBf16 / 32, SECO_DKDV_RB>;
constexpr int kNcb = kColTileBf16 / 32, kDqSmem = 4 * BNW * 2 * kRowBytes;
constexpr int kSmem = Cfg::kSmemBytes > kDqSmem ? Cfg::kSmemBytes : kDqSmem;
static_assert(Cfg::kThreads == 512, "both passes in workgroups of 8 wavefronts");

// The first first_grid workgroups are those of dK/dV (kv_first: the pass with the longer workgroups) or of dQ; both numbers are rounded up to whole XCD rounds.
template <bool SPLIT>
__global__ __launch_bounds__(512, 2) void bwd_fused_bf16_kernel(AttnParams p, SegTable seg, TailSplit ts, int n_mtiles,
                                                                int kv_total, int dq_total, int first_grid, int kv_first) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds_char* smem = (lds_char*)smem_raw;
  const bool first = (int)blockIdx.x < first_grid, kv = first == (kv_first != 0);
  const int item = xcd_item(first ? blockIdx.x : blockIdx.x - first_grid, kv ? kv_total : dq_total);
  if (item < 0) return;
  if (kv) {
    RowRuns none;
    none.n = 0;
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x / (64 * kNcb)) == 0)
      dkdv_bf16_body<kNcb, SECO_DKDV_RB, false, 0, true>(p, seg, ts, none, item, smem);
    else
      dkdv_bf16_body<kNcb, SECO_DKDV_RB, false, 1, true>(p, seg, ts, none, item, smem);
  } else {
    dq_bf16_body<2, SPLIT, false>(p, seg, n_mtiles, item, smem);
  }
}

template <bool SPLIT>
int launch(const AttnParams& p, const SegTable& seg, const TailSplit& ts, int n_mtiles, int kv_total, int dq_total, bool kv_first,
           hipStream_t s) {
  auto kern = bwd_fused_bf16_kernel<SPLIT>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), kSmem)) return SECO_ERR_LAUNCH;
  const int first = xcd_grid(kv_first ? kv_total : dq_total), second = xcd_grid(kv_first ? dq_total : kv_total);
  {
    ProfScope prof(kKernelDkdv, s);
    hipLaunchKernelGGL(kern, dim3(first + second), dim3(512), kSmem, s, p, seg, ts, n_mtiles, kv_total, dq_total, first,
                       kv_first ? 1 : 0);
    if (ts.plan.n_shared > 0) launch_tail_merge(p, seg, ts.part, ts.plan, s);
  }
  return launch_status();
}

}  // namespace

// Taken when both passes fit the chip at one workgroup per CU and the longer of them, with the extra work, is expected to
// end before the two would one after the other: with more workgroups than CUs the two halves of the grid would queue
// behind each other on some CUs (16/2 heads, chunk 704 at 5632: 7% slower in one launch).  dQ may take fewer shares of a
// row tile than it would alone, so that both fit.
int launch_bwd_fused_bf16(const AttnParams& p, const SegTable& seg, bool& launched, hipStream_t s) {
  launched = false;
  const int cus = device_cus(), n_units = p.B * p.Hkv, n_ctiles = seg.tile_begin[seg.n];
  if (n_ctiles == 0 || (int64_t)n_units * n_ctiles > cus) return SECO_OK;
  RowRuns none;
  none.n = 0;
  const TailSplit ts = tail_split<Cfg, false>(p, seg, none, n_units, p.tail_part, p.tail_slots);
  const int kv_total = n_units * (n_ctiles - ts.plan.n_tiles + ts.plan.n_entries);
  // Longest share of iterations (the first tile sees the most rows), and with it the time of a dK/dV workgroup, in 0.1 us as
  // measured: 80 + 16.5 per iteration, 18 with the row statistics; a dQ workgroup 75 + 28 per tile of 128 cache rows.
  const int rt0 = std::max(0, seg.col_begin[0] - p.q_start) / 64;
  const int iters = ((p.C + 63) / 64 - rt0) * p.G;
  const int shares = ts.plan.n_shared > 0 && ts.plan.n_tiles == n_ctiles ? ts.plan.first[1] : 1;
  const int each = (iters + shares - 1) / shares;
  const int tiles = (p.q_start + p.C + 127) / 128;
  const SplitPlan plan = split_plan(p.B, p.Hkv, p.G, p.C);
  const int mtiles = (p.C + BM - 1) / BM;
  // dQ with n workgroups per row tile, all workgroups of both passes side by side
  auto dq_wgs = [&](int n) { return n > 1 ? (int64_t)plan.items * n : (int64_t)p.B * p.Hq * mtiles; };
  auto dq_time = [&](int n) { return 75 + 28 * ((tiles + n - 1) / n); };
  auto merge_time = [&](int n) { return n > 1 ? 40 + (int)(3 * dq_wgs(n) / 10) : 0; };
  int best = 0, best_t = dq_time(p.n_splits) + merge_time(p.n_splits) + 80 + 33 * each / 2 + 20;   // one after the other
  for (int n = 1; n <= p.n_splits; ++n) {
    const int t = std::max(dq_time(n), 85 + 18 * each) + merge_time(n);
    if (dq_wgs(n) + kv_total <= cus && t < best_t) {
      best = n;
      best_t = t;
    }
  }
  if (best == 0) return SECO_OK;
  launched = true;
  AttnParams pd = p;
  pd.n_splits = best;
  const bool kv_first = 85 + 18 * each >= dq_time(best);
  const int rc = best > 1 ? launch<true>(pd, seg, ts, plan.n_mtiles, kv_total, (int)dq_wgs(best), kv_first, s)
                          : launch<false>(pd, seg, ts, mtiles, kv_total, (int)dq_wgs(1), kv_first, s);
  return rc || best == 1 ? rc : launch_dq_merge(pd, s);
}

}  // namespace seco
