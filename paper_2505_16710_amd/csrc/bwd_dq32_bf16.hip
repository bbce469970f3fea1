// dQ of one chunk, bf16, in whole row tiles with 32x32x16 products: for launches that leave CUs without work (launch_dq_bf16_now).
// A translation unit of its own for its scheduler strategy, see build.py.
#include "bwd_dq_kernel.h"

namespace seco {

int launch_dq32_bf16(const AttnParams& p, const SegTable* runs, int n_mtiles, int total, hipStream_t s) {
  return runs ? launch_dq_kernel<2, kWholeTiles, true, DqProducts32>(p, *runs, n_mtiles, total, s)
              : launch_dq_kernel<2, kWholeTiles, false, DqProducts32>(p, SegTable{}, n_mtiles, total, s);
}

}  // namespace seco
