// The dQ kernel of a launch of its own, in either shape of the products (a translation unit each: bwd_dq_bf16.hip,
// bwd_dq32_bf16.hip).
#pragma once
#include "bwd_dq_body.h"

namespace seco {
namespace {

template <int KH, int SPLIT, bool SPARSE, class Products>
__global__ __launch_bounds__(256 * KH, 2) void dq_bf16_kernel(AttnParams p, SegTable seg, int n_mtiles, int total_items) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  const int item = SPLIT == kShares ? shares_item(blockIdx.x, p.B * p.Hkv * p.rows_whole, total_items)
                                     : xcd_item(blockIdx.x, total_items, SPLIT == kDivided ? 8 : p.B * p.Hkv);
  if (item < 0) return;
  dq_bf16_body<KH, SPLIT, SPARSE, Products>(p, seg, n_mtiles, item, (lds_char*)smem_raw);
}

template <int KH, int SPLIT, bool SPARSE, class Products>
int launch_dq_kernel(const AttnParams& p, const SegTable& seg, int n_mtiles, int total, hipStream_t s) {
  constexpr int smem = 4 * BNW * KH * kRowBytes;
  auto kern = dq_bf16_kernel<KH, SPLIT, SPARSE, Products>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  {
    ProfScope prof(kKernelDq, s);
    const int units = SPLIT == kWholeTiles ? p.B * p.Hkv : 8, first = SPLIT == kShares ? p.B * p.Hkv * p.rows_whole : 0;
    hipLaunchKernelGGL(kern, dim3(xcd_grid(first, units) + xcd_grid(total - first, units)), dim3(256 * KH), smem, s, for_launch(p, n_mtiles), seg, n_mtiles, total);
  }
  return launch_status();
}

}  // namespace
}  // namespace seco
