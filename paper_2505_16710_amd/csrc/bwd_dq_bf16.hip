// dQ of one chunk, bf16: the launch shapes of the kernel in bwd_dq_body.h.
#include "bwd_dq_body.h"

namespace seco {
namespace {

template <int KH, bool SPLIT, bool SPARSE>
__global__ __launch_bounds__(256 * KH, 2) void dq_bf16_kernel(AttnParams p, SegTable seg, int n_mtiles, int total_items) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  const int item = xcd_item(blockIdx.x, total_items);
  if (item < 0) return;
  dq_bf16_body<KH, SPLIT, SPARSE>(p, seg, n_mtiles, item, (lds_char*)smem_raw);
}

template <int KH, bool SPLIT, bool SPARSE>
int launch_kh(const AttnParams& p, const SegTable& seg, int n_mtiles, int total, hipStream_t s) {
  constexpr int smem = 4 * BNW * KH * kRowBytes;
  auto kern = dq_bf16_kernel<KH, SPLIT, SPARSE>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  {
    ProfScope prof(kKernelDq, s);
    hipLaunchKernelGGL(kern, dim3(xcd_grid(total)), dim3(256 * KH), smem, s, p, seg, n_mtiles, total);
  }
  return launch_status();
}

}  // namespace

// runs == nullptr: all visible cache rows, weight 1.  A small dense pass is left for the dK/dV launcher, which may be able
// to run both at once.
int launch_dq_bf16(const AttnParams& p, const SegTable* runs, hipStream_t s) {
  if (p.pending && !runs) {
    p.pending->dq = true;
    return SECO_OK;
  }
  return launch_dq_bf16_now(p, runs, s);
}

int launch_dq_bf16_now(const AttnParams& p, const SegTable* runs, hipStream_t s) {
  SegTable none = {};
  const SegTable& seg = runs ? *runs : none;
  if (p.n_splits > 1) {
    const SplitPlan plan = split_plan(p.B, p.Hkv, p.G, p.C);
    const int total = plan.items * p.n_splits;
    int rc = runs ? launch_kh<2, true, true>(p, seg, plan.n_mtiles, total, s)
                  : launch_kh<2, true, false>(p, seg, plan.n_mtiles, total, s);
    return rc ? rc : launch_dq_merge(p, s);
  }
  const int n_mtiles = (p.C + BM - 1) / BM;
  const int total = p.B * p.Hq * n_mtiles;
  if (total < 2 * device_cus())
    return runs ? launch_kh<2, false, true>(p, seg, n_mtiles, total, s) : launch_kh<2, false, false>(p, seg, n_mtiles, total, s);
  return runs ? launch_kh<1, false, true>(p, seg, n_mtiles, total, s) : launch_kh<1, false, false>(p, seg, n_mtiles, total, s);
}

}  // namespace seco
