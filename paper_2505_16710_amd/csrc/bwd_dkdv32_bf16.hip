// dK/dV of one chunk, bf16, with 32x32x16 products: for launches that leave many CUs without work (launch_dkdv_bf16).  A
// translation unit of its own for its scheduler strategy, see build.py: max-memory-clause; max-ilp 3 - 7 % slower.
#include "bwd_dkdv_kernel.h"

namespace seco {

int launch_dkdv32_bf16(const AttnParams& p, const SegTable& seg, const TailSplit& ts, const RowRuns& rr, Rows mode, hipStream_t s) {
  if (mode == kRuns) return launch_dkdv_kernel<kRuns, Products32>(p, seg, ts, rr, s);
  return mode == kJoined ? launch_dkdv_kernel<kJoined, Products32>(p, seg, ts, rr, s) : launch_dkdv_kernel<kAll, Products32>(p, seg, ts, rr, s);
}

}  // namespace seco
