// dK/dV of one chunk, bf16: the launch of the kernel in bwd_dkdv_body.h and the merge of shared-out column tiles.
#include "bwd_dkdv_body.h"

namespace seco {
namespace {

template <int NCB, int RB, bool ROWS>
__global__ __launch_bounds__(NCB * 128, 2) void dkdv_bf16_kernel(AttnParams p, SegTable seg, TailSplit ts,
                                                                  RowRuns rr, int total_items) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];   // Cfg::kSmemBytes (can exceed the 64 KiB static limit)
  lds_char* smem = (lds_char*)smem_raw;
  const int item = xcd_item(blockIdx.x, total_items);
  if (item < 0) return;
  // wavefronts 0 .. NCB-1: role A, the others role B (wavefront-uniform: a scalar branch)
  const int role_u = __builtin_amdgcn_readfirstlane((int)threadIdx.x / (64 * NCB));
  if (role_u == 0)
    dkdv_bf16_body<NCB, RB, ROWS, 0>(p, seg, ts, rr, item, smem);
  else
    dkdv_bf16_body<NCB, RB, ROWS, 1>(p, seg, ts, rr, item, smem);
}

// gK/gV of the shared-out column tiles: g += w * (sum of the shares, in order).  One thread per four consecutive
// elements of a (tile, dV or dK) pair.
template <int COLS>
__global__ __launch_bounds__(256) void dkdv_tail_merge_kernel(AttnParams p, SegTable seg, TailSplit ts, int n_units) {
  constexpr int kBlocks = COLS * 128 / 4 / 256;       // workgroups per (tile, dV or dK)
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int quad = (blockIdx.x % kBlocks) * 256 + threadIdx.x, role = (blockIdx.x / kBlocks) & 1;
  const int st = blockIdx.x / (2 * kBlocks);          // shared tile, counted over all units
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

}  // namespace

void launch_tail_merge(const AttnParams& p, const SegTable& seg, float* part, const SharePlan& plan, hipStream_t s) {
  const int n_units = p.Hkv * p.B;
  TailSplit ts;
  ts.part = part;
  ts.plan = plan;
  hipLaunchKernelGGL(dkdv_tail_merge_kernel<kColTileBf16>, dim3((unsigned)(n_units * plan.n_shared * 2 * (kColTileBf16 / 8))),
                     dim3(256), 0, s, p, seg, ts, n_units);
}

template <int NCB, int RB, bool ROWS>
int launch_cfg(const AttnParams& p, const SegTable& seg, const RowRuns& rr, hipStream_t s) {
  using Cfg = DkdvCfg<NCB, RB>;
  const int n_units = p.Hkv * p.B, n_ctiles = seg.tile_begin[seg.n];
  const TailSplit ts = tail_split<Cfg, ROWS>(p, seg, rr, n_units, p.tail_part, p.tail_slots);
  const int total = n_units * (n_ctiles - ts.plan.n_tiles + ts.plan.n_entries);
  auto kern = dkdv_bf16_kernel<NCB, RB, ROWS>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), Cfg::kSmemBytes)) return SECO_ERR_LAUNCH;
  {
    ProfScope prof(kKernelDkdv, s);   // the merge of the divided tiles counts as part of the dK/dV pass
    hipLaunchKernelGGL(kern, dim3(xcd_grid(total)), dim3(Cfg::kThreads), Cfg::kSmemBytes, s, p, seg, ts, rr, total);
    if (ts.plan.n_shared > 0) launch_tail_merge(p, seg, ts.part, ts.plan, s);
  }
  return launch_status();
}

int launch_dkdv_bf16(const AttnParams& p, const SegTable& seg, hipStream_t s) {
  if (p.pending && p.pending->dq) {
    p.pending->dq = false;
    bool launched = false;
    int rc = launch_bwd_fused_bf16(p, seg, launched, s);
    if (rc || launched) return rc;
    if ((rc = launch_dq_bf16_now(p, nullptr, s))) return rc;
  }
  if (seg.tile_begin[seg.n] == 0) return SECO_OK;
  RowRuns none;
  none.n = 0;
  return launch_cfg<kColTileBf16 / 32, SECO_DKDV_RB, false>(p, seg, none, s);
}

int launch_dkdv_rows_bf16(const AttnParams& p, const SegTable& seg, const RowRuns& rr, hipStream_t s) {
  if (seg.tile_begin[seg.n] == 0 || rr.n == 0) return SECO_OK;
  return launch_cfg<kColTileBf16 / 32, SECO_DKDV_RB, true>(p, seg, rr, s);
}

}  // namespace seco
