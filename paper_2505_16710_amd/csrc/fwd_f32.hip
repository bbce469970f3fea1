// Forward of one chunk, fp32: O = softmax(s Q K^T) V and LSE (f32_tiles.h; a translation unit of its own: compiled together, a
// change to one of the two kernels gives the other a spill).
#include <type_traits>

#include "f32_tiles.h"

namespace seco {
namespace {

// sum of this lane's squares: infinite or NaN where an element is, or lies beyond 2^64
template <int NT>
__device__ __forceinline__ float squares(const Acc<NT>& x) {
  f32x4 t = zero4();
#pragma unroll
  for (int n = 0; n < Acc<NT>::kF; ++n)
#pragma unroll
    for (int j = 0; j < 4; ++j) t += x.full[n][j] * x.full[n][j];
#pragma unroll
  for (int m = 0; m < Acc<NT>::kR; ++m) t += x.rest[m] * x.rest[m];
  return (t[0] + t[1]) + (t[2] + t[3]);
}

// O = softmax(s Q K^T) V and LSE, of O the columns of NO of the NT blocks (fwd_nt).  The next block's K and V are requested before the present one is worked on.
template <int NT, int NO, int NW>
__global__ __launch_bounds__(NW * 64, NT <= 12 ? 2 : 1) void fwd_f32_kernel(AttnArgs p) {
  constexpr int kParts = (NT + NO - 1) / NO;
  constexpr bool kAhead = NT <= 8;                      // (longer rows do not leave the registers)
  extern __shared__ float part[];                       // an image per wavefront; then its (reference, sum) per row
  float* ml = part + NW * kPart<NT>;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;
  const int turn = gridDim.x - 1 - blockIdx.x, r0 = turn / kParts * kRows, h = blockIdx.y, b = blockIdx.z, D = p.D;
  const int o0 = turn % kParts * (16 * NO), n_o = min(D - o0, 16 * NO);   // this workgroup's columns of O
  if (n_o <= 0) return;
  const float* K = static_cast<const float*>(p.k) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const float* V = static_cast<const float*>(p.v) + b * p.kvs[0] + (h / p.G) * p.kvs[1] + o0;
  const int64_t row = p.kvs[2];
  const int qpos = p.q_start + r0 + i, kv_end = p.q_start + min(r0 + kRows, p.C);
  float* own = part + w * kPart<NT>;
  Block<NT> kb;
  Cols<NO> vx;
  const Pieces<NT> pk(lane, row, D);
  const uint32_t v_off = (uint32_t)(4 * g) * (uint32_t)row;   // elements
  auto load_k = [&](int c0) { pk.load(kb, K + c0 * row, row, kv_end - c0); };
  auto load_v = [&](int c0) {
    const float* from = V + c0 * row;
    if (c0 + kRows <= kv_end)
      vx.load([&](int r) { return from + r * row + v_off; }, n_o, i);
    else
      vx.load([&](int r) { return V + min(c0 + 4 * g + r, kv_end - 1) * row; }, n_o, i);
  };
  f32x4 qf[NT];
  {
    // (every wavefront brings Q for itself: a barrier here sets them all on the same phase, 15.4 us instead of 14.8)
    Block<NT> qb;
    Pieces<NT>(lane, p.qs[2], D).load(qb, static_cast<const float*>(p.q) + b * p.qs[0] + h * p.qs[1] + r0 * p.qs[2], p.qs[2], p.C - r0);
    if (kAhead && w * 16 < kv_end) load_k(w * 16), load_v(w * 16);
    pk.put(own, qb, lane);
    rows_of<NT>(own, i, g, qf);
    mask_kept<NT>(D, g, qf);
  }
  const float c = p.scale * kLog2e;
  // m: the row's reference in log2 units (-inf before it has seen anything), ref: the same with 0 for -inf; l: this lane's
  // share of the row's sum.  The reference only guards against overflow, so it moves only when a score lies more than
  // `slack` above it.  (Vector instructions and fp32 products take turns on a SIMD, whichever wavefront they come from, so
  // every instruction of the loop counts: with the maximum and the rescaling in every block a call over 1024 rows took
  // 15.5 us, 14.8 without.)  Weights of up to 2^32 take as much from the range of V: a wavefront whose sums come near the end
  // of fp32 starts over with the running maximum, under which they end only where rows times |V| do.  (To look for that costs
  // 0.0 - 0.2 us of calls of 6 - 25 us, 0.3 of 40; at the longest rows up to 2 %: 8 heads of 256, 700 rows at 200: 74 -> 75.)
  constexpr float kSlack = 32.f;
  float m, ref, l;
  Acc<NO> o;
  // ahead: the first block's K and V have been requested, and the next ones are while a block is worked on
  auto blocks = [&](auto ahead, float slack) {
    constexpr bool kNext = decltype(ahead)::value;
    m = -INFINITY, ref = 0.f, l = 0.f;
    o.clear();
#pragma unroll 1
    for (int c0 = w * 16; c0 < kv_end; c0 += NW * 16) {
      if (!kNext) load_k(c0);
      const bool more = kNext && c0 + NW * 16 < kv_end;
      f32x4 s;
      {
        f32x4 kx[NT];
        pk.put(own, kb, lane);
        if (more) load_k(c0 + NW * 16);
        rows_of<NT>(own, i, g, kx);
        s = score<NT>(kx, qf);
      }
      if (!kNext) {                                     // (behind the products: K, its row form and V do not fit together)
        asm volatile("" : "+v"(s) : : "memory");
        load_v(c0);
      }
      s *= c;
      if (c0 + kRows > p.q_start + r0) {                // a block on the diagonal
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = c0 + 4 * g + r <= qpos ? s[r] : -INFINITY;
      }
      float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
      if (__builtin_amdgcn_ballot_w64(mx > m + slack)) {
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32)));
        ref = mx == -INFINITY ? 0.f : mx;
        const float alpha = fast_exp2(m - ref);
        m = mx;
        l *= alpha;
        o.scale(alpha);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[r] = fast_exp2(s[r] - ref);
        l += s[r];
      }
      o.add(vx, s);
      if (more) load_v(c0 + NW * 16);
    }
  };
  auto near_end = [&]() { return __builtin_expect(__builtin_amdgcn_ballot_w64(!(squares(o) <= __FLT_MAX__)) != 0, 0); };
  if constexpr (kAhead) {                               // (a second loop: as one, with its first loads inside, it spills)
    blocks(std::true_type(), kSlack);
    if (near_end()) blocks(std::false_type(), 0.f);
  } else {
    for (float slack = kSlack;; slack = 0.f) {
      blocks(std::false_type(), slack);
      if (slack == 0.f || !near_end()) break;
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  o.store(own, i, g);
  if (g == 0) {
    ml[(w * kRows + i) * 2] = m;
    ml[(w * kRows + i) * 2 + 1] = l;
  }
  __syncthreads();
  // a wavefront finishes whole rows: its lane (i, g) adds the partials of wavefronts g NW / 4 .. of elements 4 i ..
  for (int r = w; r < min(kRows, p.C - r0); r += NW) {
    float M = -INFINITY, a[NW / 4], L = 0.f;
#pragma unroll
    for (int v = 0; v < NW / 4; ++v) a[v] = ml[((g * (NW / 4) + v) * kRows + r) * 2], M = fmaxf(M, a[v]);
    M = fmaxf(M, __shfl_xor(M, 16));
    M = fmaxf(M, __shfl_xor(M, 32));                    // finite: column 0 is always visible
#pragma unroll
    for (int v = 0; v < NW / 4; ++v) {
      a[v] = fast_exp2(a[v] - M);
      L += a[v] * ml[((g * (NW / 4) + v) * kRows + r) * 2 + 1];
    }
    L += __shfl_xor(L, 16);
    L += __shfl_xor(L, 32);
    float* out = static_cast<float*>(p.o_out) + b * p.os[0] + h * p.os[1] + (r0 + r) * p.os[2] + o0;
#pragma unroll
    for (int d0 = 0; d0 < 16 * NO; d0 += 64) {
      const int d = d0 + 4 * i;
      f32x4 acc = zero4();
#pragma unroll
      for (int v = 0; v < NW / 4; ++v) acc += a[v] * load4(part + (g * (NW / 4) + v) * kPart<NT> + r * kPartRow<NO> + min(d, 16 * NO - 4));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[j] += __shfl_xor(acc[j], 16);
        acc[j] += __shfl_xor(acc[j], 32);
      }
      if (g == 0 && d < n_o) *reinterpret_cast<f32x4*>(out + d) = acc * (1.f / L);
    }
    if (lane == 0 && o0 == 0) p.lse[((int64_t)b * p.Hq + h) * p.C + r0 + r] = (M + __log2f(L)) * kLn2;
  }
}

// Wavefronts per workgroup: as many as the register file holds of the kernel at that head_dim.
template <int NT> constexpr int kFwdWaves = NT <= 4 ? 16 : NT <= 8 ? 8 : 4;

template <int NT, int NO>
int fwd_launch(const AttnParams& p, hipStream_t s) {
  constexpr int NW = kFwdWaves<NT>, smem = NW * (kPart<NT> + 2 * kRows) * 4;
  auto kern = fwd_f32_kernel<NT, NO, NW>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  ProfScope prof(kKernelFwd, s);
  hipLaunchKernelGGL(kern, dim3((p.C + kRows - 1) / kRows * ((NT + NO - 1) / NO), p.Hq, p.B), dim3(NW * 64), smem, s, p);
  return launch_status();
}
// Few row tiles: two or four workgroups for each, on CUs that had none, which all compute its scores but only a part of the
// columns of O, whose products are half of the work.  As long as that leaves every workgroup a CU: beyond, the scores computed
// again cost more than they save (88 tiles of head_dim 64 by four: 24 us, by two 17.3, whole 18.7).  4 heads of 64, 256 rows
// at 768: 14.9 -> 11.7 us; 3 heads of 128, 76 rows at 560: 18.2 -> 13.8; 4 of 256, 200 at 400: 37.5 -> 25.0.
// Not where O is written over an input: each of them would read query rows that another has overwritten.
template <int NT>
int fwd_nt(const AttnParams& p, hipStream_t s) {
  const int64_t n = (int64_t)((p.C + kRows - 1) / kRows) * p.Hq * p.B, cus = device_cus();
  if (o_over_inputs(p, sizeof(float))) return fwd_launch<NT, NT>(p, s);
  if (n * 4 <= cus) return fwd_launch<NT, (NT + 3) / 4>(p, s);
  if (n * 2 <= cus) return fwd_launch<NT, (NT + 1) / 2>(p, s);
  return fwd_launch<NT, NT>(p, s);
}
}  // namespace

int launch_fwd_f32(const AttnParams& p, hipStream_t s) { SECO_F32_DISPATCH(fwd_nt, p, s) }

}  // namespace seco
