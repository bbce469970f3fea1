// dK/dV of one chunk, bf16: the launch of the kernel in bwd_dkdv_body.h and the merge of shared-out column tiles.
#include "bwd_dkdv_body.h"
#include "bwd_plan.h"
#include "merge_body.h"

namespace seco {
namespace {

template <int NCB, int RB, bool ROWS, class Products>
__global__ __launch_bounds__(NCB * 128, 2) void dkdv_bf16_kernel(AttnParams p, SegTable seg, TailSplit ts,
                                                                  RowRuns rr, int total_items) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];   // Cfg::kSmemBytes (can exceed the 64 KiB static limit)
  lds_char* smem = (lds_char*)smem_raw;
  const int item = xcd_item(blockIdx.x, total_items, p.B * p.Hkv);
  if (item < 0) return;
  // wavefronts 0 .. NCB-1: role A, the others role B (wavefront-uniform: a scalar branch)
  const int role_u = __builtin_amdgcn_readfirstlane((int)threadIdx.x / (64 * NCB));
  if (role_u == 0)
    dkdv_bf16_body<NCB, RB, ROWS, 0, Products>(p, seg, ts, rr, item, smem);
  else
    dkdv_bf16_body<NCB, RB, ROWS, 1, Products>(p, seg, ts, rr, item, smem);
}

template <int COLS>
__global__ __launch_bounds__(256) void dkdv_tail_merge_kernel(AttnParams p, SegTable seg, TailSplit ts) {
  tail_merge_body<COLS>(p, seg, ts, blockIdx.x);
}

using Cfg = DkdvCfg<kColTileBf16 / 32, SECO_DKDV_RB>;

template <bool ROWS, class Products>
int launch(const AttnParams& p, const SegTable& seg, const TailSplit& ts, const RowRuns& rr, hipStream_t s) {
  const int total = p.Hkv * p.B * (seg.tile_begin[seg.n] - ts.plan.n_tiles + ts.plan.n_entries);
  auto kern = dkdv_bf16_kernel<kColTileBf16 / 32, SECO_DKDV_RB, ROWS, Products>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), Cfg::kSmemBytes)) return SECO_ERR_LAUNCH;
  {
    ProfScope prof(kKernelDkdv, s);   // the merge of the divided tiles counts as part of the dK/dV pass
    hipLaunchKernelGGL(kern, dim3(xcd_grid(total, p.B * p.Hkv)), dim3(Cfg::kThreads), Cfg::kSmemBytes, s, p, seg, ts, rr, total);
    if (ts.plan.n_shared > 0)
      hipLaunchKernelGGL(dkdv_tail_merge_kernel<kColTileBf16>, dim3(tail_merge_grid<kColTileBf16>(p, ts)), dim3(256), 0, s, p, seg, ts);
  }
  return launch_status();
}

}  // namespace

int launch_dkdv_bf16(const AttnParams& p, const SegTable& seg, hipStream_t s) {
  const bool dq = p.pending && p.pending->dq;
  if (dq) p.pending->dq = false;
  const SegTable* runs = dq && p.pending->sparse ? &p.pending->runs : nullptr;
  if (seg.tile_begin[seg.n] == 0) return dq ? launch_dq_bf16_now(p, runs, s) : SECO_OK;
  // (where dQ visits selected columns or lies over O, the sums of gK / gV are divided as they would be otherwise: the same bits)
  const BwdPlan plan = plan_bwd<Cfg>(p, seg, dq);
  if (dq && plan.dq_splits > 0 && !dq_over_inputs(p, 2)) {
    AttnParams pf = p;
    pf.n_splits = runs ? sparse_shares(p, *runs, plan.dq_splits) : plan.dq_splits;
    return launch_bwd_fused_bf16(pf, seg, plan.ts, plan.kv_first, runs, s);
  }
  int rc = dq ? launch_dq_bf16_now(p, runs, s) : SECO_OK;
  RowRuns none;
  none.n = 0;
  if (rc) return rc;
  return plan.dq_splits > 0 ? launch<false, Products32>(p, seg, plan.ts, none, s) : launch<false, Products16>(p, seg, plan.ts, none, s);
}

int launch_dkdv_rows_bf16(const AttnParams& p, const SegTable& seg, const RowRuns& rr, hipStream_t s) {
  if (seg.tile_begin[seg.n] == 0 || rr.n == 0) return SECO_OK;
  int n_rows = 0;
  for (int i = 0; i < rr.n; ++i) n_rows += rr.end[i] - rr.begin[i];
  TailSplit ts;
  ts.part = p.tail_part;
  float time;
  ts.plan = share_plan(tile_iterations<Cfg, true>(p, seg, rr), p.B * p.Hkv, seg.tile_begin[seg.n], p.G, n_rows, slots_in(p.tail_bytes), time);
  return launch<true, Products16>(p, seg, ts, rr, s);
}

}  // namespace seco
