// The dK/dV kernel of a launch of its own, in either shape of the products (a translation unit each: bwd_dkdv_bf16.hip,
// bwd_dkdv32_bf16.hip).
#pragma once
#include "bwd_dkdv_body.h"

namespace seco {
namespace {

using Cfg = DkdvCfg<kColTileBf16 / 32, SECO_DKDV_RB>;

template <int NCB, int RB, Rows MODE, class Products>
__global__ __launch_bounds__(NCB * 128, 2) void dkdv_bf16_kernel(AttnParams p, SegTable seg, TailSplit ts,
                                                                  RowRuns rr, int total_items) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];   // Cfg::kSmemBytes (can exceed the 64 KiB static limit)
  lds_char* smem = (lds_char*)smem_raw;
  const int item = xcd_item(blockIdx.x, total_items, p.B * p.Hkv);
  if (item < 0) return;
  // wavefronts 0 .. NCB-1: role A, the others role B (wavefront-uniform: a scalar branch)
  const int role_u = __builtin_amdgcn_readfirstlane((int)threadIdx.x / (64 * NCB));
  if (role_u == 0)
    dkdv_bf16_body<NCB, RB, MODE, 0, Products>(p, seg, ts, rr, item, smem);
  else
    dkdv_bf16_body<NCB, RB, MODE, 1, Products>(p, seg, ts, rr, item, smem);
}

template <Rows MODE, class Products>
int launch_dkdv_kernel(const AttnParams& p, const SegTable& seg, const TailSplit& ts, const RowRuns& rr, hipStream_t s) {
  AttnParams pl = p;
  const int per_unit = for_column_tiles(pl, seg, ts), total = p.Hkv * p.B * per_unit;
  auto kern = dkdv_bf16_kernel<kColTileBf16 / 32, SECO_DKDV_RB, MODE, Products>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), Cfg::kSmemBytes)) return SECO_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, dim3(xcd_grid(total, p.B * p.Hkv)), dim3(Cfg::kThreads), Cfg::kSmemBytes, s, pl, seg, ts, rr, total);
  return launch_status();
}

}  // namespace
}  // namespace seco
