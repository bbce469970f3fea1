// Angles of the rotary position embedding, in fp64, and the rotation of a pair.
#pragma once
#include <cmath>

#include <hip/hip_runtime.h>

namespace seco {
namespace {

// base^(-2 i / D) for i = 4 grp + j is a product of powers the host has computed: pow[k] = base^(-8 2^k / D) for bit k of
// grp, and step = base^(-2 / D), j times (an fp64 exp2 per element pair was half of the kernel's arithmetic).
struct RopePowers {
  double pow[6], step;
};
inline RopePowers rope_powers(int D, float base) {
  RopePowers powers;
  powers.step = exp2(-2.0 / D * log2((double)base));
  for (int k = 0; k < 6; ++k) powers.pow[k] = exp2(-8.0 * (1 << k) / D * log2((double)base));
  return powers;
}

// Sine and cosine in fp64: the nearest multiple n of pi/2 is taken off in two fused steps (pi/2 as the sum of two
// doubles, so that the remainder is good to an ulp of 1 for |n| up to 2^40), and on the remaining |x| <= pi/4 the Taylor
// series up to x^15 and x^16 are exact to 1e-16.
__device__ __forceinline__ void sincos_f64(double theta, double& sn, double& cs) {
  const double n = rint(theta * 0.63661977236758134308);        // 2 / pi
  double x = fma(-n, 1.57079632679489655800, theta);
  x = fma(-n, 6.12323399573676603587e-17, x);
  const double y = x * x;
  double ps = -1.0 / 1307674368000.0, pc = 1.0 / 20922789888000.0;
  ps = fma(ps, y, 1.0 / 6227020800.0);
  pc = fma(pc, y, -1.0 / 87178291200.0);
  ps = fma(ps, y, -1.0 / 39916800.0);
  pc = fma(pc, y, 1.0 / 479001600.0);
  ps = fma(ps, y, 1.0 / 362880.0);
  pc = fma(pc, y, -1.0 / 3628800.0);
  ps = fma(ps, y, -1.0 / 5040.0);
  pc = fma(pc, y, 1.0 / 40320.0);
  ps = fma(ps, y, 1.0 / 120.0);
  pc = fma(pc, y, -1.0 / 720.0);
  ps = fma(ps, y, -1.0 / 6.0);
  pc = fma(pc, y, 1.0 / 24.0);
  pc = fma(pc, y, -0.5);
  const double s0 = fma(x * y, ps, x), c0 = fma(y, pc, 1.0);
  const int q = (int)(n - 4.0 * floor(0.25 * n));                // n mod 4
  const double a = q & 1 ? c0 : s0, b = q & 1 ? s0 : c0;
  sn = q & 2 ? -a : a;
  cs = (q + 1) & 2 ? -b : b;
}

// of position pos and the pairs 4 grp .. 4 grp + 3
__device__ __forceinline__ void rope_sines(int64_t pos, int grp, const RopePowers& powers, double (&sn)[4], double (&cs)[4]) {
  double theta = (double)pos;
#pragma unroll
  for (int k = 0; k < 6; ++k) theta *= grp >> k & 1 ? powers.pow[k] : 1.0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    sincos_f64(theta, sn[j], cs[j]);
    theta *= powers.step;
  }
}
__device__ __forceinline__ void rope_pair(float& lo, float& hi, double sn, double cs) {
  const double a = (double)lo, c = (double)hi;
  lo = (float)(a * cs - c * sn);
  hi = (float)(c * cs + a * sn);
  // (rounded to fp32 and then to the storage type, as rope_rows_kernel does: the compiler would take the two steps
  // as one, and two of 524288 elements differ)
  asm("" : "+v"(lo), "+v"(hi));
}

}  // namespace
}  // namespace seco
