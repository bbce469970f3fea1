// Division by a number that the host knows, by the method of Granlund and Montgomery (Division by Invariant Integers using
// Multiplication, 1994): q = (m n / 2^32 + n) / 2^l, exact for 0 <= n < 2^31 and d >= 1 (l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1).  Three scalar instructions, where a division by a kernel argument is a chain of about 35
// through the vector unit's reciprocal.  A workgroup finds out what it is to do by five to nine of them, one behind the other, in front
// of its first load: 2.6 us from a dQ workgroup's start to its first requests, 2.1 with these.  Over random calls together with
// 32-bit row offsets from scalar addresses: forward 2.6 % faster (1 % slower to 8 % faster), backward 1.7 %; calls of a millisecond the same.
#pragma once
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace seco {

struct Div {
  uint32_t m, l;
};
inline Div make_div(int d) {
  Div x{0, 0};
  while (((uint64_t)1 << x.l) < (uint64_t)d) ++x.l;
  x.m = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << x.l) - (uint64_t)d)) / (uint64_t)d + 1);
  return x;
}
// n / d
__host__ __device__ __forceinline__ int over(int n, Div x) {
  return (int)(((uint32_t)(((uint64_t)x.m * (uint32_t)n) >> 32) + (uint32_t)n) >> x.l);
}

}  // namespace seco
