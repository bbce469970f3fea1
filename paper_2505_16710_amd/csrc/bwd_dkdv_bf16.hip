// dK/dV of one chunk, bf16: the launch of the kernel in bwd_dkdv_body.h and the merge of shared-out column tiles.
#include "bwd_dkdv_kernel.h"
#include "bwd_plan.h"
#include "merge_body.h"

namespace seco {
namespace {

template <int COLS>
__global__ __launch_bounds__(256) void dkdv_tail_merge_kernel(AttnParams p, SegTable seg, TailSplit ts) {
  tail_merge_body<COLS>(p, seg, ts, blockIdx.x);
}

// Which products: those that take the least power where the pass keeps the CUs busy, else, with the clock as high as it goes, those
// that leave the vector instructions the most room (us, 32x32x16 against 16x16x32; 1088 rows at 8704 of 16/2 heads, 154 column
// tiles of 136 iterations: 186 against 196; 1095 at 1694 of 32/8 102 / 110, 2327 at 2894 of 16/4 195 / 212; but, busy to 0.85, 1355 at
// 6418 of 32/4 292 / 269).  The line lies between calls at 0.70 and 0.77 that lose 3 % on their other sides.
constexpr float kBusy = 0.74f;

template <Rows MODE>
int launch(const AttnParams& p, const SegTable& seg, const TailSplit& ts, const RowRuns& rr, bool p16, hipStream_t s) {
  ProfScope prof(kKernelDkdv, s);     // the merge of the divided tiles counts as part of the dK/dV pass
  const int rc = p16 ? launch_dkdv_kernel<MODE, Products16>(p, seg, ts, rr, s) : launch_dkdv32_bf16(p, seg, ts, rr, MODE, s);
  if (rc || ts.plan.n_shared == 0) return rc;
  hipLaunchKernelGGL(dkdv_tail_merge_kernel<kColTileBf16>, dim3(tail_merge_grid<kColTileBf16>(p, ts)), dim3(256), 0, s, p, seg, ts);
  return launch_status();
}

}  // namespace

int launch_dkdv_bf16(const AttnParams& p, const SegTable& seg, hipStream_t s) {
  const bool dq = p.pending && p.pending->dq;
  if (dq) p.pending->dq = false;
  const SegTable* runs = dq && p.pending->sparse ? &p.pending->runs : nullptr;
  if (seg.tile_begin[seg.n] == 0) return dq ? launch_dq_bf16_now(p, runs, true, s) : SECO_OK;
  // (where dQ visits selected columns or lies over O, the sums of gK / gV are divided as they would be otherwise: the same bits)
  const BwdPlan plan = plan_bwd<Cfg>(p, seg, dq);
  if (dq && plan.dq_splits > 0 && !dq_over_inputs(p, 2)) {
    AttnParams pf = p;
    pf.n_splits = runs ? sparse_shares(p, *runs, plan.dq_splits) : plan.dq_splits;
    return launch_bwd_fused_bf16(pf, seg, plan.ts, plan.kv_first, plan.joined, runs, s);
  }
  int rc = dq ? launch_dq_bf16_now(p, runs, plan.dq_splits == 0, s) : SECO_OK;
  RowRuns none;
  none.n = 0;
  if (rc) return rc;
  const bool p16 = plan.dq_splits == 0 && plan.busy >= kBusy;
  return plan.joined ? launch<kJoined>(p, seg, plan.ts, none, p16, s) : launch<kAll>(p, seg, plan.ts, none, p16, s);
}

int launch_dkdv_rows_bf16(const AttnParams& p, const SegTable& seg, const RowRuns& rr, hipStream_t s) {
  if (seg.tile_begin[seg.n] == 0 || rr.n == 0) return SECO_OK;
  int n_rows = 0;
  for (int i = 0; i < rr.n; ++i) n_rows += rr.end[i] - rr.begin[i];
  TailSplit ts;
  ts.part = p.tail_part;
  float time, busy;
  ts.plan = share_plan(tile_iterations<Cfg, true>(p, seg, rr), p.B * p.Hkv, seg.tile_begin[seg.n], p.G, n_rows, slots_in(p.tail_bytes), time, &busy);
  return launch<kRuns>(p, seg, ts, rr, busy >= kBusy, s);
}

}  // namespace seco
