// What the fp32 kernels for chunked causal attention share (fwd_f32.hip; kernels_f32.hip: dQ and dK/dV): the fp32 matrix
// instruction (v_mfma_f32_16x16x4_f32: fp32 products and sums, 157 TFLOP/s on this GPU), for any head_dim that is a multiple
// of 4 up to 256.
//
// The fp32 configuration is small (cfg1: 4 heads, 256-row chunks, 1024 tokens), so what bounds it is how much of the
// GPU a call can occupy and the length of the dependent chains, not bandwidth: a workgroup owns only 16 query rows
// (forward, dQ) or 16 cache rows (dK/dV), its wavefronts divide the other dimension among themselves, and their partial
// results are combined through LDS in wavefront order (one writer per element, fixed order: reproducible).
//
// Operand forms (lane l, i = l % 16, g = l / 16; a contraction may visit its index in any order, so each lane takes
// four consecutive elements with one load and instruction j uses the j-th):
//   row form  X[r0 + i][16 t + 4 g + j]   contraction over head_dim, instruction (t, j)
//   col form  X[r0 + 4 g + r][64 n + 4 i + j]   contraction over rows, instruction r; output (n, j)
// A score tile computed as (rows of X) x (rows of Y) leaves lane l with Y row i and X rows 4 g + r, r = 0..3: exactly
// the second operand of the col form.  An output tile holds head_dim 64 n + 16 g + 4 r + j for the lane's row i.
// What is left behind the groups of 64 is taken in blocks of 16, one element per lane (head_dim 80: 20 products per block of
// 16 rows and operand instead of 32).
//
// A wavefront copies 16 rows with its lanes along the rows (a "block"), 1 KiB per instruction, and turns them in its own
// LDS into the forms it needs.  Loaded in row form straight from memory, 16 neighbouring lanes touch 16 rows, which the
// address unit takes one by one: 16 bytes per clock and CU instead of 64, and all three kernels waited for that (4 heads of
// head_dim 64, 256 rows at position 768: forward 17.2 -> 14.8 us, backward 22.0 -> 18.3; 97 rows at 900: 16.9 -> 14.7 and 21.0 ->
// 18.2).  What bounds them now: the products and vector instructions of the CUs that have a row tile (2 us per 256 cache
// rows of products alone), and 4 - 6 us of launch, first loads and last sums.
// Positions past head_dim repeat the row's last four elements and are multiplied by zero (row form) or dropped (col form);
// rows past the end repeat the last one and are masked.
#pragma once
#include "mfma_tiles.h"
#include "seco_internal.h"

namespace seco {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kRows = 16;   // rows a workgroup owns
// blocks of 16 that every head_dim that NT blocks are used for (SECO_F32_DISPATCH) fills; past head_dim lie later ones
template <int NT> constexpr int kWhole = NT <= 2 ? 0 : NT <= 4 ? 2 : NT <= 5 ? 4 : NT <= 8 ? 5 : NT <= 12 ? 8 : 12;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// LDS image of 16 rows: rows of 16 NT floats, padded by 4
template <int NT> constexpr int kPartRow = 16 * NT + 4;
template <int NT> constexpr int kPart = kRows * kPartRow<NT>;

// ---- a wavefront's copy of 16 rows: lane l takes the 16-byte pieces l, l + 64, ..
template <int NT> struct Block { f32x4 v[NT]; };
// This lane's pieces.  Where a row is a power of two pieces long, piece l + 64 j lies kStep j rows below piece l.
template <int NT> struct Pieces {
  static constexpr bool kEven = 64 % (4 * NT) == 0;
  static constexpr bool kFixed = kEven || NT <= 8;      // offsets kept (twelve of them do not leave the registers)
  static constexpr int kStep = 64 / (4 * NT), kN = kEven ? 1 : kFixed ? NT : 0;
  int lane, D;
  uint32_t off[kN > 0 ? kN : 1];   // bytes from the first row, in a matrix of the given stride
  __device__ __forceinline__ int row(int j) const { return (lane + 64 * j) / (4 * NT); }
  __device__ __forceinline__ int col(int j) const { return min((lane + 64 * j) % (4 * NT) * 4, D - 4); }   // element
  __device__ __forceinline__ Pieces(int lane_, int64_t stride, int D_) : lane(lane_), D(D_) {
#pragma unroll
    for (int j = 0; j < kN; ++j) off[j] = ((uint32_t)row(j) * (uint32_t)stride + (uint32_t)col(j)) * 4u;
  }
  // rows base, base + stride, ..; n of them (at least one): rows past them repeat the last.  (All scalar but the lane.)
  __device__ __forceinline__ void load(Block<NT>& b, const float* base, int64_t stride, int n) const {
    if (kFixed && n >= kRows) {
      const char* from = reinterpret_cast<const char*>(base);
      int step = kEven ? kStep * 4 * (int)stride : 0;
      asm volatile("" : "+s"(step));       // (its multiples are not worth registers of their own throughout a loop)
#pragma unroll
      for (int j = 0; j < NT; ++j) b.v[j] = *reinterpret_cast<const f32x4*>(from + (int64_t)j * step + off[kEven ? 0 : j % (kN > 0 ? kN : 1)]);
    } else {
#pragma unroll
      for (int j = 0; j < NT; ++j) b.v[j] = load4(base + min(row(j), n - 1) * stride + col(j));
    }
  }
  __device__ __forceinline__ void put(float* own, const Block<NT>& b, int lane) const {
#pragma unroll
    for (int j = 0; j < NT; ++j)
      *reinterpret_cast<f32x4*>(own + (lane + 64 * j) / (4 * NT) * kPartRow<NT> + (lane + 64 * j) % (4 * NT) * 4) = b.v[j];
    asm volatile("" : : : "memory");     // (read back by other lanes; a wavefront's LDS accesses are in order)
  }
};
// row form of a block in LDS
template <int NT>
__device__ __forceinline__ void rows_of(const float* own, int i, int g, f32x4 (&x)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) x[t] = load4(own + i * kPartRow<NT> + 16 * t + 4 * g);
  asm volatile("" : : : "memory");
}
// ... to be kept as the second operand of a score tile: zero past head_dim
template <int NT>
__device__ __forceinline__ void mask_kept(int D, int g, f32x4 (&x)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) x[t][j] = 16 * t + 4 * g < D ? x[t][j] : 0.f;
}
// (two chains: a tile's products are dependent, 32 cycles each)
template <int NT>
__device__ __forceinline__ f32x4 score(const f32x4 (&x)[NT], const f32x4 (&kept)[NT]) {
  f32x4 s[2] = {zero4(), zero4()};
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j & 1] = mfma4(x[t][j], kept[t][j], s[j & 1]);
  return s[0] + s[1];
}
// 16 rows in col form
template <int NT> struct Cols {
  static constexpr int kF = NT / 4, kR = NT % 4;
  f32x4 full[4][kF > 0 ? kF : 1];
  float rest[4][kR > 0 ? kR : 1];
  // row(r): of this lane's rows 4 g + r, from its first element on; width: elements that are there
  template <typename Row> __device__ __forceinline__ void load(const Row& row, int width, int i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int n = 0; n < kF; ++n) full[r][n] = load4(row(r) + min(64 * n + 4 * i, width - 4));
#pragma unroll
      for (int m = 0; m < kR; ++m) rest[r][m] = row(r)[min(64 * kF + 16 * m + i, width - 1)];
    }
  }
  // of a block in LDS
  __device__ __forceinline__ void of(const float* own, int i, int g) {
    load([&](int r) { return own + (4 * g + r) * kPartRow<NT>; }, 16 * NT, i);
    asm volatile("" : : : "memory");
  }
};
// 16 rows of results: element 64 n + 16 g + 4 r + j of the lane's row i in full[n][j][r], 64 kF + 16 m + 4 g + r in rest[m][r]
template <int NT> struct Acc {
  static constexpr int kF = NT / 4, kR = NT % 4;
  f32x4 full[kF > 0 ? kF : 1][4];
  f32x4 rest[kR > 0 ? kR : 1];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int n = 0; n < kF; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) full[n][j] = zero4();
#pragma unroll
    for (int m = 0; m < kR; ++m) rest[m] = zero4();
  }
  __device__ __forceinline__ void scale(float f) {
#pragma unroll
    for (int n = 0; n < kF; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) full[n][j] *= f;
#pragma unroll
    for (int m = 0; m < kR; ++m) rest[m] *= f;
  }
  __device__ __forceinline__ void add(const Cols<NT>& x, const f32x4& w) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int n = 0; n < kF; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) full[n][j] = mfma4(x.full[r][n][j], w[r], full[n][j]);
#pragma unroll
      for (int m = 0; m < kR; ++m) rest[m] = mfma4(x.rest[r][m], w[r], rest[m]);
    }
  }
  // into an LDS image
  __device__ __forceinline__ void store(float* own, int i, int g) const {
    float* row = own + i * kPartRow<NT>;
#pragma unroll
    for (int n = 0; n < kF; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x4 v = {full[n][0][r], full[n][1][r], full[n][2][r], full[n][3][r]};
        *reinterpret_cast<f32x4*>(row + 64 * n + 16 * g + 4 * r) = v;
      }
#pragma unroll
    for (int m = 0; m < kR; ++m) *reinterpret_cast<f32x4*>(row + 64 * kF + 16 * m + 4 * g) = rest[m];
  }
};

}  // namespace

// head_dim in blocks of 16: the sizes in use exactly, others by the next larger one
#define SECO_F32_DISPATCH(F, ...)                       \
  switch ((p.D + 15) / 16) {                            \
    case 1: case 2: return F<2>(__VA_ARGS__);           \
    case 3: case 4: return F<4>(__VA_ARGS__);           \
    case 5: return F<5>(__VA_ARGS__);                   \
    case 6: case 7: case 8: return F<8>(__VA_ARGS__);   \
    case 9: case 10: case 11: case 12: return F<12>(__VA_ARGS__); \
    default: return F<16>(__VA_ARGS__);                 \
  }

}  // namespace seco
