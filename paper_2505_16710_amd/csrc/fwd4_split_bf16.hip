// The short-chunk forward: the 8-wavefront kernel (4 row blocks x 2 column halves) with the cache divided among workgroups.
// (Its own translation unit: instantiated next to the plain one, neither keeps its instruction schedule.)
#include "fwd8_kernel.h"

namespace seco {

int launch_fwd8_split_bf16(const AttnParams& p, int n_mtiles, int total, hipStream_t s) { return launch_fwd8<kDivided>(p, n_mtiles, total, s); }

}  // namespace seco
