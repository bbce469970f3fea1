// Which work item a workgroup takes, by XCD (host arithmetic and the kernels' side of it).  Workgroup ids go round-robin over the 8 XCDs, each
// with its own L2 and 32 CUs; a kernel's grid is the matching xcd_grid.  (An MI355X as one device.  Divided into several it has fewer of
// both: the same items, placed as they come.  Decided from a kernel argument instead, dK/dV's pass takes 1 % longer.)
#pragma once
#include <hip/hip_runtime.h>

namespace seco {

constexpr int kXcds = 8, kXcdCus = 32;

// XCD x takes the contiguous item range [x * per_xcd, (x+1) * per_xcd): the workgroups that stream one KV head stay on one L2.
__host__ __device__ __forceinline__ int xcd_item(int block, int total_items) {
  const int per_xcd = (total_items + 7) >> 3;
  const int item = (block & 7) * per_xcd + (block >> 3);
  return item < total_items ? item : -1;
}
inline int xcd_grid(int total_items) { return ((total_items + 7) / 8) * 8; }

// The same for the items of a launch that come as equal runs, one for each of `units` (batch, KV head) pairs, the long ones of a run
// first, and are more than one for each CU: one, two or four units have eight, four or two XCDs each, and the items of a unit are
// dealt to its XCDs in turn.  As ranges one XCD had a unit's long items and another its short ones, or one its whole column tiles
// and another its shares: forward of 7000 rows at 0 of 8/2 heads 166 -> 110 us, 3602 of 16/2 90 -> 63; backward of 2135 at 1572 of
// 16/2 232 -> 184, two sequences of 1439 at 8039 811 -> 637.  With a CU for every item ranges are the faster (1000 rows at 0 of 32/4
// 19.5 against 20.2), and for row tiles that are divided (all, 128 at 16000 of 16/2: 27.8 against 31.2; those beyond a round, 1500 at
// 3000 of 32/4: 105 against 107): units 8.  (The launch of both passes of the backward keeps ranges as well: 1 - 2 % slower dealt.)
__host__ __device__ __forceinline__ bool xcds_share_units(int total_items, int units) {
  return total_items > kXcds * kXcdCus && (units == 1 || units == 2 || units == 4);
}
__host__ __device__ __forceinline__ int xcd_item(int block, int total_items, int units) {
  if (!xcds_share_units(total_items, units)) return xcd_item(block, total_items);
  const int lg = units >> 1, xcd = block & 7, of_unit = 3 - lg;        // (log2 of the units, and of a unit's XCDs)
  const int per_unit = total_items >> lg, in = ((block >> 3) << of_unit) + (xcd & ((1 << of_unit) - 1));
  return in < per_unit ? (xcd >> of_unit) * per_unit + in : -1;
}
inline int xcd_grid(int total_items, int units) {
  if (!xcds_share_units(total_items, units)) return xcd_grid(total_items);
  const int lg = units >> 1, of_unit = 3 - lg;
  return ((total_items >> lg) + (1 << of_unit) - 1) >> of_unit << 3;
}

// The first n_first items, then the others: each part divided evenly among the XCDs (grid: the two parts' together).
__host__ __device__ __forceinline__ int shares_item(int block, int n_first, int total_items) {
  const int grid = (n_first + 7) / 8 * 8;
  if (block < grid) return xcd_item(block, n_first);
  const int i = xcd_item(block - grid, total_items - n_first);
  return i < 0 ? -1 : n_first + i;
}

}  // namespace seco
