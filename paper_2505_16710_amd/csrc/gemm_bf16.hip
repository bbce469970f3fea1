// Matrix products of the decoder around the attention (chunk_loop.py), bf16 with fp32 accumulation, in the three forms
// a projection needs: forward C = A B, data gradient C = A B^T, weight gradient C (+)= A^T B, with the SiLU of the MLP
// and its derivative in the epilogue of the product they follow.
//
// What bounds them: at the row counts of a chunk (512 rows, 1 - 4 thousand columns) a product is 1 - 4 GFLOP, a few
// microseconds of matrix work on 256 CUs, so launch cost and latency count, not the matrix pipe.  A call of the
// library product through the framework took 17 - 19 us of host time, twice its kernel; a launch here takes 3.  Above
// about 10 GMAC the framework's kernels are faster, and the training step takes those (worth() in chunk_step_ext.cpp).
//
// A workgroup (2 x 2 or 2 x 4 wavefronts, or two groups of the former that take the steps in turn) owns a BM x BN tile of C
// and walks the contraction in steps of 64 through a ring of kStages LDS slots filled by direct global -> LDS copies,
// kStages - 1 steps ahead, with one barrier per step.  An operand whose
// contraction runs along its rows in memory ("KC") is staged as rows of 64 contraction elements, one whose rows are
// contracted ("KR") as panels of 64 of its columns; either way an LDS row is 128 bytes whose eight 16-byte chunks
// are XOR-ed with a function of the row such that row reads (ds_read_b128, 16 rows) and transpose reads
// (ds_read_b64_tr_b16, 4 rows x 64 bytes) meet no bank conflict.  Both kinds of read deliver contraction slot s of
// lane group g as element 8 g + s, so that any two operands can meet.  The tile leaves through LDS in rows of 16-byte stores.
#include <algorithm>
#include <type_traits>

#include "decoder.h"
#include "mfma_tiles.h"
#include "rope.h"
#include "seco_internal.h"

namespace seco {
namespace {

constexpr int kStep = 64, kRow = 128;   // contraction elements per step; bytes per LDS row
enum Epilogue { kStore, kAdd, kSilu, kSiluBwd, kQkv };

struct GemmArgs {
  const char* a;
  const char* b;
  __bf16* c;
  __bf16* c2;       // kSilu: silu(C); kSiluBwd: the u that C is the gradient of silu at
  int M, N, K, lda, ldb, ldc, tiles_m, tiles_n;
  int split_m, part_m, part_n;       // an XCD's part of the tiles (place_tiles); split_m 0: runs of them
};
// kQkv: C is the joint projection [B C, (Hq + 2 Hkv) 128], whose query heads leave rotated; the key heads go rotated, the value heads
// as they are, to rows row0 .. of the cache
struct QkvArgs : GemmArgs {
  __bf16 *k, *v;
  int64_t ks[3], row0;
  int chunk, Hq, Hkv;
  Div by_chunk;
  RopePowers powers;
};
template <int EPI> using ArgsOf = std::conditional_t<EPI == kQkv, QkvArgs, GemmArgs>;

__device__ __forceinline__ int flip(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }

// Copies of one operand by W wavefronts: instruction i of a wavefront brings the staged rows 8 (wave + W i) .. + 7.
// GAP (KR): columns left out in the middle of a panel
template <bool KC, int BO, int W = 4, int GAP = 0> struct Stage {
  static constexpr int kCopies = BO / (8 * W);
  uint32_t off[kCopies];      // this lane's source, relative to the step's base
  // o0: first outer index of the tile, n_outer: how many there are (KR: a multiple of 8); rows / chunks past the end repeat the last
  __device__ void init(int o0, int n_outer, int ld, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      const int lr = 8 * (wave + W * i) + (lane >> 3);
      if (KC) {
        off[i] = (uint32_t)min(o0 + lr, n_outer - 1) * (uint32_t)(ld * 2) + (((lane & 7) ^ flip(lr)) << 4);
      } else {
        const int krow = lr & 63;
        const int chunk = (lane & 7) ^ flip(krow);
        off[i] = (uint32_t)krow * (uint32_t)(ld * 2) + (uint32_t)min(o0 + (lr & ~63) + (chunk << 3) + (chunk >> 2) * GAP, n_outer - 8) * 2u;
      }
    }
  }
  __device__ void copy(const char* base, uint32_t lds_wave) const {   // lds_wave: the operand's slot + 8 wave rows
#pragma unroll
    for (int i = 0; i < kCopies; ++i) dma16_sbase(base, off[i], lds_wave + i * 8 * W * kRow);
  }
};

// The last contraction rows of two KR operands, when they do not fill a step: through registers, zeros behind the end.
template <int BO>
__device__ __forceinline__ void stage_rest(lds_char* dst, const char* base, int rows, int o0, int n_outer, int ld) {
  for (int c = threadIdx.x; c < BO * 8; c += blockDim.x) {
    const int lr = c >> 3, krow = lr & 63, col = min(o0 + (lr & ~63) + ((c & 7) << 3), n_outer - 8);
    bf16x8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (__bf16)0.f;
    if (krow < rows) v = *reinterpret_cast<const bf16x8*>(base + ((int64_t)krow * ld + col) * 2);
    *reinterpret_cast<SECO_LDS bf16x8*>(dst + lr * kRow + (((c & 7) ^ flip(krow)) << 4)) = v;
  }
}

// Operand of the 32-wide block `blk` of a staged tile for 16 contraction elements, t = 0 .. 3
template <bool KC> struct Frag {
  int lo, hi;
  int chunk_t[KC ? 4 : 1];
  __device__ void init(int blk, int lane, int t0 = 0) {   // t0: which of a step's 16 elements t = 0 stands for
    if (KC) {
      const int row = lane & 31;
      lo = blk * 32 * kRow + row * kRow;
#pragma unroll
      for (int t = 0; t < (KC ? 4 : 1); ++t) chunk_t[t] = lo + (((2 * (t0 + t) + (lane >> 5)) ^ flip(row)) << 4);
      hi = 0;
    } else {
      const int ii = lane & 15, row = 8 * (lane >> 5) + (ii >> 2), first = 16 * t0 * kRow;
      const int chunk = 4 * (blk & 1) + 2 * ((lane >> 4) & 1) + ((ii & 3) >> 1), sub = (ii & 1) << 3;
      lo = first + (blk >> 1) * 64 * kRow + row * kRow + ((chunk ^ flip(row)) << 4) + sub;
      hi = first + (blk >> 1) * 64 * kRow + (row + 4) * kRow + ((chunk ^ flip(row + 4)) << 4) + sub;
      chunk_t[0] = 0;
    }
  }
  __device__ __forceinline__ bf16x8 read(lds_char* tile, int t) const {
    if constexpr (KC) {
      return *reinterpret_cast<SECO_LDS bf16x8*>(tile + chunk_t[t]);
    } else {
      s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<SECO_LDS s16x4*>(tile + lo + 16 * t * kRow));
      s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<SECO_LDS s16x4*>(tile + hi + 16 * t * kRow));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      const s16x8 r = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
      return __builtin_bit_cast(bf16x8, r);
    }
  }
};

// what eight sums from element `at` of C on meet there: C itself, or u
template <int EPI> __device__ __forceinline__ bf16x8 met(const GemmArgs& g, int64_t at) {
  bf16x8 old = {};
  if constexpr (EPI == kAdd) old = *reinterpret_cast<const bf16x8*>(g.c + at);
  if constexpr (EPI == kSiluBwd) old = *reinterpret_cast<const bf16x8*>(g.c2 + at);
  return old;
}
// 1 / (1 + e^-u).  A division is eleven vector instructions, half of the epilogue's, and all wavefronts of the one round of tiles
// are in their epilogues together: 2048 x 4096 x 1024 with the SiLU 25.3 us, 24.2 by the reciprocal and a step of Newton's; back
// through it 24.7 and 23.4.  The same SiLU for every u in bf16, and the same derivative.  Below kFar, where e^-u or the reciprocal
// leave fp32's normal numbers, the division.
constexpr float kFar = -87.f;
template <bool FAR> __device__ __forceinline__ float logistic(float u) {
  const float d = 1.f + __expf(-u);
  if constexpr (FAR) return 1.f / d;
  const float y = __builtin_amdgcn_rcpf(d);
  return __builtin_fmaf(__builtin_fmaf(-d, y, 1.f), y, y);
}
// silu(u) to c2, or the gradient f behind the SiLU to C
template <int EPI, bool FAR>
__device__ __forceinline__ void emit_silu(const GemmArgs& g, int64_t at, const float (&f)[8], const bf16x8& u) {
  bf16x8 x;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float v = (float)u[e], s = logistic<FAR>(v);
    x[e] = EPI == kSilu ? (__bf16)(v * s) : (__bf16)((float)(__bf16)f[e] * (s * (1.f + v * (1.f - s))));
  }
  *reinterpret_cast<bf16x8*>((EPI == kSilu ? g.c2 : g.c) + at) = x;
}
// eight sums to C, from element `at` on
template <int EPI, typename F4>
__device__ __forceinline__ void emit(const GemmArgs& g, int64_t at, const F4& lo, const F4& hi, const bf16x8& old) {
  const float f[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  bf16x8 out;
#pragma unroll
  for (int e = 0; e < 8; ++e) out[e] = (__bf16)(EPI == kAdd ? (float)old[e] + f[e] : f[e]);
  if constexpr (EPI != kSiluBwd) *reinterpret_cast<bf16x8*>(g.c + at) = out;
  if constexpr (EPI == kSilu || EPI == kSiluBwd) {
    const bf16x8& u = EPI == kSilu ? out : old;
    float least = (float)u[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) least = fminf(least, (float)u[e]);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(least < kFar) != 0, 0))
      emit_silu<EPI, true>(g, at, f, u);
    else
      emit_silu<EPI, false>(g, at, f, u);
  }
}

// The columns of a tile of kQkv are pairs (c, c + 64) of one head: all of its 128, or, 64 wide, 32 from either half, so that a thread
// finds both elements of four pairs among the tile's sums (a tile of half rows reads half lines of B: 0.9 us at 512 rows).  The sines
// are computed while the first operands are on their way, which covers half of their time (0.8 us; one pair behind each step of the
// contraction all of it shows).  Product and rotation, 8/2 heads of a 1024-wide model, in two launches -> one, us: 64 rows 7.5 -> 5.2,
// 256 9.0 -> 6.5, 512 9.7 -> 7.8, 1024 12.3 -> 10.5; the product alone 4.4, 5.3, 6.2, 8.6.
template <int BN> __device__ __forceinline__ int qkv_column(int tn) { return BN == 64 ? (tn >> 1) * 128 + (tn & 1) * 32 : tn * BN; }
struct Sines {
  double sn[4], cs[4];
};
// of row r of C and the pairs from column c of a head on
__device__ __forceinline__ void qkv_sines(const QkvArgs& g, int r, int c, Sines& x) {
  const int b = over(r, g.by_chunk);
  rope_sines(g.row0 + r - b * g.chunk, c >> 2, g.powers, x.sn, x.cs);
#pragma unroll
  for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(x.sn[j]), "+v"(x.cs[j]));     // (here, not behind the products)
}
// four pairs of row r, from column col = 128 head + c on
template <typename F4>
__device__ __forceinline__ void emit_qkv(const QkvArgs& g, int r, int col, const F4& lo, const F4& hi, const Sines& x) {
  const int head = col >> 7, c = col & 127, b = over(r, g.by_chunk), kv = head - g.Hq, vh = kv - g.Hkv;
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 out[2];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float l = (float)(__bf16)lo[j], h = (float)(__bf16)hi[j];
    if (vh < 0) rope_pair(l, h, x.sn[j], x.cs[j]);
    out[0][j] = (__bf16)l;
    out[1][j] = (__bf16)h;
  }
  __bf16* to = kv < 0 ? g.c + (int64_t)r * g.ldc + col
                      : (vh < 0 ? g.k : g.v) + b * g.ks[0] + (vh < 0 ? kv : vh) * g.ks[1] + (g.row0 + r - b * g.chunk) * g.ks[2] + c;
  *reinterpret_cast<bf16x4*>(to) = out[0];
  *reinterpret_cast<bf16x4*>(to + 64) = out[1];
}

// KH groups of 2 x WN x KW wavefronts, each with a ring of kStages slots; group kh takes the steps kh, kh + KH, ..., and of each
// step the wavefronts of equal kw a KW-th.
template <int BM, int BN, int KH, int kStages, int WN, bool AKC, bool BKC, int EPI, int KW>
__device__ __forceinline__ void ring_tile(const ArgsOf<EPI>& g, int item, lds_char* smem_all) {
  constexpr int kSlot = (BM + BN) * kRow, GW = 2 * WN * KW, MB = BM / 64, NB = BN / (32 * WN);
  constexpr int kPerWave = BM / (8 * GW) + BN / (8 * GW);            // copies per wavefront and step
  constexpr int kRing = kStages * kSlot, kImage = kRing / KW;   // kImage: for a wavefront's part of the sums
  const int tid = threadIdx.x, lane = tid & 63, wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = wave_all % GW, kh = KH == 1 ? 0 : wave_all / GW;
  const int kw = KW == 1 ? 0 : wave / (2 * WN), wt = KW == 1 ? wave : wave % (2 * WN);
  lds_char* smem = smem_all + kh * kRing;
  const int tn = item / g.tiles_m, tm = item - tn * g.tiles_m;
  const int m0 = tm * BM, n0 = EPI == kQkv ? qkv_column<BN>(tn) : tn * BN;

  Stage<AKC, BM, GW> sa;
  Stage<BKC, BN, GW, EPI == kQkv && BN == 64 ? 32 : 0> sb;
  sa.init(m0, g.M, g.lda, wave, lane);
  sb.init(n0, g.N, g.ldb, wave, lane);
  const int64_t step_a = AKC ? kStep * 2 : (int64_t)kStep * g.lda * 2, step_b = BKC ? kStep * 2 : (int64_t)kStep * g.ldb * 2;
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + 8 * wave * kRow);
  const char *pa = g.a + kh * step_a, *pb = g.b + kh * step_b;   // of the next step to be copied
  const int n_full = g.K / kStep;
  const int n_steps = (n_full - kh + KH - 1) / KH;       // of this group
  auto copy = [&](int slot) {
    sa.copy(pa, lds_wave + slot * kSlot);
    sb.copy(pb, lds_wave + slot * kSlot + BM * kRow);
    pa += KH * step_a;
    pb += KH * step_b;
  };
#pragma unroll
  for (int s = 0; s < kStages - 1; ++s)
    if (s < n_steps) copy(s);

  constexpr int kPerRow = BN / 8, kRows = 64 * GW * KH / kPerRow;
  Sines sines[EPI == kQkv ? BM / kRows : 1];
  const int pairs = n0 + (tid % kPerRow) * 4;              // kQkv: this thread's first column
  if constexpr (EPI == kQkv) {
    if (n0 < (g.Hq + g.Hkv) * 128) {
#pragma unroll
      for (int i = 0; i < BM / kRows; ++i) qkv_sines(g, min(m0 + i * kRows + tid / kPerRow, g.M - 1), pairs & 127, sines[i]);
    }
  }
  Frag<AKC> fa[MB];
  Frag<BKC> fb[NB];
#pragma unroll
  for (int i = 0; i < MB; ++i) fa[i].init(wt / WN * MB + i, lane, kw * (4 / KW));
#pragma unroll
  for (int i = 0; i < NB; ++i) fb[i].init(wt % WN * NB + i, lane, kw * (4 / KW));
  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto multiply = [&](int slot) {
    lds_char* ta = smem + slot * kSlot;
    lds_char* tb = ta + BM * kRow;
#pragma unroll
    for (int t = 0; t < 4 / KW; ++t) {
      bf16x8 x[MB], y[NB];
#pragma unroll
      for (int i = 0; i < MB; ++i) x[i] = fa[i].read(ta, t);
#pragma unroll
      for (int j = 0; j < NB; ++j) y[j] = fb[j].read(tb, t);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = mfma(x[i], y[j], acc[i][j]);
    }
  };

  // where this thread's part of the tile leaves, and what it meets there: requested behind the last wait for operands, in
  // front of the last step's products
  const int col = n0 + (tid % kPerRow) * 8;
  bf16x8 old[BM / kRows];
  auto request_old = [&]() {
#pragma unroll
    for (int i = 0; i < BM / kRows; ++i) {
      const int row = min(m0 + i * kRows + tid / kPerRow, g.M - 1);
      old[i] = met<EPI>(g, (int64_t)row * g.ldc + min(col, g.N - 8));
    }
  };
  int slot = 0;
  const int n_turns = (n_full + KH - 1) / KH;            // the same for all groups: they share the barriers
  auto wait = [&](int it) {
    // step `it` has landed when at most the copies of the kStages - 2 steps behind it are outstanding
    if (it + kStages - 2 < n_steps)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((kStages - 2) * kPerWave) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" : : : "memory");
  };
  constexpr bool kMeets = EPI == kAdd || (EPI == kSiluBwd && BM == 128);
  for (int it = 0; it < n_turns - (kMeets ? 1 : 0); ++it) {
    wait(it);
    if (it + kStages - 1 < n_steps) copy(slot == 0 ? kStages - 1 : slot - 1);   // the slot every wavefront has just left
    if (KH == 1 || it < n_steps) multiply(slot);
    slot = slot + 1 == kStages ? 0 : slot + 1;
  }
  if constexpr (kMeets) {
    if (n_turns > 0) wait(n_turns - 1);
    request_old();
    if (n_turns > 0 && (KH == 1 || n_turns - 1 < n_steps)) multiply(slot);
  }
  if constexpr (!AKC && !BKC) {
    if (const int rest = g.K - n_full * kStep; rest > 0) {
      __syncthreads();
      stage_rest<BM>(smem_all, g.a + n_full * step_a, rest, m0, g.M, g.lda);
      stage_rest<BN>(smem_all + BM * kRow, g.b + n_full * step_b, rest, n0, g.N, g.ldb);
      __syncthreads();
      if (kh == 0) multiply(0);
    }
  }

  __syncthreads();
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  constexpr int kTurnRow = BM * (BN + 4) * 4 <= kImage ? (BN + 4) * 4 : BN * 4;   // padded where there is room
  static_assert(BM * kTurnRow <= kImage && kImage % 16 == 0, "the tile fits");
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        *reinterpret_cast<SECO_LDS float*>(smem + kw * kImage + ((wt / WN * MB + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * kTurnRow +
                                           ((wt % WN * NB + j) * 32 + (lane & 31)) * 4) = acc[i][j][r];
  __syncthreads();
  if (col >= g.N) return;
#pragma unroll
  for (int i = 0; i < BM / kRows; ++i) {
    const int lr = i * kRows + tid / kPerRow, row = m0 + lr;
    if (row >= g.M) break;
    constexpr int kBetween = EPI == kQkv ? BN * 2 : 16;       // bytes between a thread's two quads of a row
    lds_char* src = smem_all + lr * kTurnRow + (tid % kPerRow) * (EPI == kQkv ? 16 : 32);
    f32x4 lo = *reinterpret_cast<SECO_LDS f32x4*>(src), hi = *reinterpret_cast<SECO_LDS f32x4*>(src + kBetween);
#pragma unroll
    for (int v = 1; v < KH * KW; ++v) {
      lo += *reinterpret_cast<SECO_LDS f32x4*>(src + v * kImage);
      hi += *reinterpret_cast<SECO_LDS f32x4*>(src + v * kImage + kBetween);
    }
    if constexpr (EPI == kQkv) {
      emit_qkv(g, row, pairs, lo, hi, sines[i]);
      continue;
    }
    const int64_t at = (int64_t)row * g.ldc + col;
    emit<EPI>(g, at, lo, hi, kMeets ? old[i] : met<EPI>(g, at));
  }
}

// A product with few tiles and, often, a long contraction (the projections back to the residual stream: 512 x 1024 x 4096):
// tiles of 32 x 64 (BM 32), and every wavefront takes steps of the contraction for the whole tile, w, w + NW, .., on its own, in LDS
// of its own: no barrier before the sums of the wavefronts meet.  What bounds 64 x 64 tiles there is LDS (2 KiB read per
// MFMA) on half of the CUs; here an operand is read from LDS once (1.5 KiB per MFMA), twice the CUs work, and the copies of
// all wavefronts are in flight at once.
// BM 64: an operand is read for twice as many products, by half as many workgroups (taller_beside).
template <int BM> struct KSlot {      // a wavefront's operands, or its part of the sums
  static constexpr int kTurnRow = (64 + 4) * 4, kBytes = std::max((BM + 64) * kRow, BM * kTurnRow);
};
template <int NW, int BM, bool AKC, bool BKC, int EPI>
__device__ __forceinline__ void k_tile(const ArgsOf<EPI>& g, int item, lds_char* smem_all) {
  constexpr int BN = 64, MB = BM / 32, kSlot = KSlot<BM>::kBytes, kTurnRow = KSlot<BM>::kTurnRow;
  static_assert(BM * 8 <= 64 * NW, "a thread for eight columns of a row");
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  lds_char* smem = smem_all + w * kSlot;
  const int tn = item / g.tiles_m, tm = item - tn * g.tiles_m;
  const int m0 = tm * BM, n0 = EPI == kQkv ? qkv_column<BN>(tn) : tn * BN;
  Stage<AKC, BM, 1> sa;
  Stage<BKC, BN, 1, EPI == kQkv ? 32 : 0> sb;
  sa.init(m0, g.M, g.lda, 0, lane);
  sb.init(n0, g.N, g.ldb, 0, lane);
  const int64_t step_a = AKC ? kStep * 2 : (int64_t)kStep * g.lda * 2, step_b = BKC ? kStep * 2 : (int64_t)kStep * g.ldb * 2;
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
  const char *pa = g.a + w * step_a, *pb = g.b + w * step_b;
  const int n_steps = g.K / kStep;
  auto copy = [&]() {
    sa.copy(pa, lds);
    sb.copy(pb, lds + BM * kRow);
    pa += NW * step_a;
    pb += NW * step_b;
  };
  if (w < n_steps) copy();
  Sines sines;
  const int pairs = n0 + (threadIdx.x & 7) * 4;
  if constexpr (EPI == kQkv)
    if (n0 < (g.Hq + g.Hkv) * 128 && w < BM / 8) qkv_sines(g, min(m0 + (int)(threadIdx.x >> 3), g.M - 1), pairs & 127, sines);
  Frag<AKC> fa[MB];
  Frag<BKC> fb[2];
#pragma unroll
  for (int i = 0; i < MB; ++i) fa[i].init(i, lane);
  fb[0].init(0, lane);
  fb[1].init(1, lane);
  f32x16 acc[MB][2];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  for (int it = w; it < n_steps; it += NW) {
    dma_wait_all();
    bf16x8 x[MB][4], y[2][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int i = 0; i < MB; ++i) x[i][t] = fa[i].read(smem, t);
      y[0][t] = fb[0].read(smem + BM * kRow, t);
      y[1][t] = fb[1].read(smem + BM * kRow, t);
    }
    // (all operands are in registers before the next copy overwrites them)
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[0][2]), "+v"(x[0][3]), "+v"(y[0][0]), "+v"(y[0][1]), "+v"(y[0][2]),
                 "+v"(y[0][3]), "+v"(y[1][0]), "+v"(y[1][1]), "+v"(y[1][2]), "+v"(y[1][3]) : : "memory");
    if constexpr (MB == 2) asm volatile("" : "+v"(x[1][0]), "+v"(x[1][1]), "+v"(x[1][2]), "+v"(x[1][3]) : : "memory");
    if (it + NW < n_steps) copy();
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma(x[i][t], y[j][t], acc[i][j]);
  }
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        *reinterpret_cast<SECO_LDS float*>(smem + (32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * kTurnRow + (j * 32 + (lane & 31)) * 4) =
            acc[i][j][r];
  __syncthreads();
  const int lr = threadIdx.x >> 3, col = n0 + (threadIdx.x & 7) * 8;
  if (lr >= BM || m0 + lr >= g.M || col >= g.N) return;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    lds_char* src = smem_all + v * kSlot + lr * kTurnRow + (threadIdx.x & 7) * (EPI == kQkv ? 16 : 32);
    lo += *reinterpret_cast<SECO_LDS f32x4*>(src);
    hi += *reinterpret_cast<SECO_LDS f32x4*>(src + (EPI == kQkv ? 128 : 16));
  }
  if constexpr (EPI == kQkv) {
    emit_qkv(g, m0 + lr, pairs, lo, hi, sines);
    return;
  }
  const int64_t at = (int64_t)(m0 + lr) * g.ldc + col;
  emit<EPI>(g, at, lo, hi, met<EPI>(g, at));
}

// A way to work a product: workgroups of kThreads with kSmem bytes of LDS, one per item
template <int BM, int BN, int KH, int ST, int WN, bool AKC, bool BKC, int EPI, int KW = 1> struct Ring {
  using Args = ArgsOf<EPI>;
  static constexpr int kThreads = 128 * WN * KW * KH, kSmem = KH * ST * (BM + BN) * kRow, kBM = BM, kBN = BN;
  static __device__ __forceinline__ void run(const Args& g, int item, lds_char* smem) {
    ring_tile<BM, BN, KH, ST, WN, AKC, BKC, EPI, KW>(g, item, smem);
  }
};
template <int NW, bool AKC, bool BKC, int EPI, int BM = 32> struct ByK {
  using Args = ArgsOf<EPI>;
  static constexpr int kThreads = 64 * NW, kSmem = NW * KSlot<BM>::kBytes, kBM = BM, kBN = 64;
  static __device__ __forceinline__ void run(const Args& g, int item, lds_char* smem) { k_tile<NW, BM, AKC, BKC, EPI>(g, item, smem); }
};
// Which tiles the XCDs take (workgroups whose ids are equal mod 8 share an L2).  Runs of the tiles, column by column: an XCD
// reads all rows of A and an eighth of B's columns.  Or split_m x 8 / split_m parts of part_m x part_n tiles, one for each XCD,
// where that reads less than two thirds of it and leaves no XCD more tiles than an even share; with less to win the runs are as
// fast or faster (512 x 1024 x 4096, 512 rows and columns for 640: 11.5 against 12.2 us).  Returns the grid.
// us, runs -> parts: added to 4096 x 1024 over 2048 rows 24.2 -> 21.2, over 512 9.9 -> 8.6; 2048 x 1024 x 4096 25.6 -> 24.4;
// 2048 x 1024 x 1536, rows of both contracted, 13.4 -> 12.4.
template <typename T> int place_tiles(GemmArgs& g) {
  g.tiles_m = (g.M + T::kBM - 1) / T::kBM;
  g.tiles_n = (g.N + T::kBN - 1) / T::kBN;
  const int64_t total = (int64_t)g.tiles_m * g.tiles_n, even = (total + 7) / 8;
  int64_t least = (2 * (std::min<int64_t>(g.tiles_m, even) * T::kBM + (even + g.tiles_m - 1) / g.tiles_m * T::kBN) + 2) / 3;
  g.split_m = 0;
  for (int sm = 2; sm <= 8; sm *= 2) {
    const int64_t pm = (g.tiles_m + sm - 1) / sm, pn = (g.tiles_n + 8 / sm - 1) / (8 / sm), reads = pm * T::kBM + pn * T::kBN;
    if (pm * pn > even || reads >= least) continue;
    least = reads;
    g.split_m = sm;
    g.part_m = (int)pm;
    g.part_n = (int)pn;
  }
  return g.split_m ? 8 * g.part_m * g.part_n : xcd_grid((int)total);
}
__device__ __forceinline__ int tile_of(const GemmArgs& g, int block) {
  if (g.split_m == 0) return xcd_item(block, g.tiles_m * g.tiles_n);
  const int xcd = block & 7, i = block >> 3, in = i / g.part_m;
  const int tm = (xcd & (g.split_m - 1)) * g.part_m + (i - in * g.part_m), tn = xcd / g.split_m * g.part_n + in;
  return tm < g.tiles_m && tn < g.tiles_n ? tn * g.tiles_m + tm : -1;
}

template <typename T>
__global__ __launch_bounds__(T::kThreads, 2) void gemm_kernel(typename T::Args g) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  const int item = tile_of(g, blockIdx.x);
  if (item >= 0) T::run(g, item, (lds_char*)smem_raw);
}
template <typename T> int launch(typename T::Args g, hipStream_t s) {
  auto kern = gemm_kernel<T>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), T::kSmem)) return SECO_ERR_LAUNCH;
  const int grid = place_tiles<T>(g);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(T::kThreads), T::kSmem, s, g);
  return launch_status();
}
// Which tile: measured over 64 .. 2048 rows against matrices of 1024 x 1024 .. 4096 x 1024 (us; K: contraction length).
// LDS reads bound the small tiles (2 KiB per MFMA at 64 x 64, 1 KiB at 128 x 128), idle CUs the large ones.
//  - forward and data gradient whose 32 x 64 tiles fit one round: those, the contraction divided among eight wavefronts (512 x
//    1024 x 4096: 11.3 against 14.5 with 64 x 64 tiles, 512 x 1024 x 1024: 5.2 / 5.8, 320 x 1536 x 1024: 5.1 / 5.8; in two rounds
//    they lose: 640 x 1024 x 1024 8.2 / 5.8; twelve wavefronts 11.6 and 5.5.  What bounds the long one now is what the L2s
//    deliver: 196 MB in 8.5 us; beside a weight gradient 64 x 64, taller_beside);
//  - over 1.25 128 x 128 tiles per CU: those, four wavefronts and two slots, so that two workgroups share a CU
//    (2048 x 4096 x 1024: 25; 31 with eight wavefronts, 35 with 64 x 64 tiles);
//  - from 0.55 per CU on: 128 x 128, eight wavefronts side by side, three slots (added to a 4096 x 1024 product over 512 rows:
//    9.5; in two groups with two slots, which turn and add twice the sums through LDS, 10.5, and 11.4 while what the sums
//    are added to was only requested when they were there);
//  - 64 x 64 tiles that fit one round: those, two groups, three slots (512 x 1024 x 4096: 14.6; 18.5 with one group);
//  - more of them: 128 x 64 for a long contraction of rows of A (2048 x 1024 x 4096: 25 against 27 with 64 x 128), forward with the
//    steps halved between wavefronts that hold 64 x 64 of the tile, two thirds of the LDS reads and two more images to add (as
//    64 x 32 of whole steps -> so: 2048 x 1024 x 4096 26.9 -> 24.1, 1500 rows 23.0 -> 21.8; the data gradient 24.2 / 24.6; 128 x 128 tiles
//    so halved 12.8 -> 12.3 at 2048 x 1536 x 1024, 5.0 -> 5.6 at 1536 x 1536 x 192); else, where
//    the rows of B are contracted, 64 x 128, eight wavefronts side by side, three slots: a third less from L2 than 64 x 64 with two
//    slots and two workgroups per CU (1024 x 1536 over 512 rows: 5.7 against 6.3, 512 x 4096 x 1024 with the SiLU: 9.9 / 10.4;
//    2048 x 1024 over 2048: 13.7 / 14.9 with 128 x 64); else those (512 x 4096 x 1024 back through the SiLU: 9.5; 10.2 with 64 x 128).
template <typename T> struct Way { using type = T; };
template <bool AKC, bool BKC, int EPI, typename F> int with_way(const GemmArgs& g, const F& f) {
  const int64_t m64 = (g.M + 63) / 64, n64 = (g.N + 63) / 64, big = ((m64 + 1) / 2) * ((n64 + 1) / 2), cus = device_cus();
  if constexpr (AKC)
    if ((g.M + 31) / 32 * n64 <= cus) return f(Way<ByK<8, AKC, BKC, EPI>>());
  if (4 * big > 5 * cus) return f(Way<Ring<128, 128, 1, 2, 2, AKC, BKC, EPI>>());
  if (20 * big >= 11 * cus) return f(Way<Ring<128, 128, 1, 3, 4, AKC, BKC, EPI>>());
  if (m64 * n64 <= cus) return f(Way<Ring<64, 64, 2, 3, 2, AKC, BKC, EPI>>());
  if constexpr (AKC)
    if (g.K >= 2048) return f(Way<Ring<128, 64, 2, 3, BKC ? 2 : 1, AKC, BKC, EPI, BKC ? 1 : 2>>());
  if constexpr (!BKC)
    return f(Way<Ring<64, 128, 1, 3, 4, AKC, BKC, EPI>>());
  else
    return f(Way<Ring<64, 64, 2, 2, 2, AKC, BKC, EPI>>());
}
template <bool AKC, bool BKC, int EPI> int pick(const GemmArgs& g, hipStream_t s) {
  return with_way<AKC, BKC, EPI>(g, [&](auto way) { return launch<typename decltype(way)::type>(g, s); });
}

// Both gradients of a layer's product in one launch.  Each fills the chip once or less for a few microseconds: what is saved is
// the end of the one and the start of the other, 1.5 - 3 us.  512 rows, apart -> together: 1024 x 4096 19.5 -> 17.7, 4096 x 1024
// with the SiLU's derivative 18.9 -> 17.6, 1024 x 1536 12.1 -> 10.3, 1024 x 1024 10.1 -> 8.6; 320 rows 17.5 -> 14.5, 16.6 -> 14.0,
// -, 9.5 -> 7.7.
// weight_first: which workgroups go in front.  Those of the weight gradient take rows / 64 steps, the others' time does not
// depend on the rows: the longer ones first (512 rows, 4096 x 1024: 17.6 against 18.8; 320: 15.1 against 14.0).  data_first: taller_beside.
template <typename A, typename B>
__global__ __launch_bounds__(512, 2) void gemm_pair_kernel(GemmArgs a, GemmArgs b, int first_grid, int weight_first) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  const bool first = (int)blockIdx.x < first_grid, weight = first == (weight_first != 0);
  const int block = first ? blockIdx.x : blockIdx.x - first_grid;
  if (weight) {
    if (const int item = tile_of(b, block); item >= 0) B::run(b, item, (lds_char*)smem_raw);
  } else {
    if (const int item = tile_of(a, block); item >= 0) A::run(a, item, (lds_char*)smem_raw);
  }
}
template <typename A, typename B> int launch_pair(GemmArgs a, GemmArgs b, hipStream_t s, bool data_first = false) {
  static_assert(A::kThreads == 512 && B::kThreads == 512, "workgroups of one size");
  constexpr int smem = A::kSmem > B::kSmem ? A::kSmem : B::kSmem;
  auto kern = gemm_pair_kernel<A, B>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  const int ga = place_tiles<A>(a), gb = place_tiles<B>(b), weight_first = b.K >= 448 && !data_first;
  hipLaunchKernelGGL(kern, dim3(ga + gb), dim3(512), smem, s, a, b, weight_first ? gb : ga, weight_first);
  return launch_status();
}
// taller_pays of the tiles: a data gradient in 32 x 64 or 64 x 64, beside a weight gradient in bm x bn
inline bool taller_beside(const GemmArgs& a, const GemmArgs& b, int bm, int bn) {
  const int64_t n64 = (a.N + 63) / 64;
  return taller_pays(a.M, a.K, (a.M + 31) / 32 * n64, (a.M + 63) / 64 * n64, (int64_t)((b.M + bm - 1) / bm) * ((b.N + bn - 1) / bn));
}
constexpr int kApart = 1;           // (no seco_status)
// In one launch where the data gradient takes one of the small tiles and as many of its workgroups share a CU as by itself
// (64 x 64 tiles with two slots: two; larger products would gain less than 5 %).  kApart: not
// EPI_W: what becomes of the weight gradient: kAdd, or kStore for a step's first chunk
template <int EPI, int EPI_W> int pair(const GemmArgs& a, const GemmArgs& b, hipStream_t s) {
  using Wide = Ring<128, 128, 1, 3, 4, false, false, EPI_W>;
  using Two = Ring<64, 64, 2, 2, 2, true, true, EPI>;
  return with_way<true, true, EPI>(a, [&](auto way_a) {
    using A = typename decltype(way_a)::type;
    if constexpr (A::kThreads == 512 && A::kBM <= 64) {
      return with_way<false, false, EPI_W>(b, [&](auto way_b) {
        using B = typename decltype(way_b)::type;
        if constexpr (std::is_same_v<A, ByK<8, true, true, EPI>> && B::kThreads == 512)
          if (taller_beside(a, b, B::kBM, B::kBN))
            return launch_pair<ByK<8, true, true, EPI, 64>, B>(a, b, s, true);        // (the same sums)
        if constexpr (!std::is_same_v<A, Two> && B::kThreads == 512)
          return launch_pair<A, B>(a, b, s);
        else if constexpr (std::is_same_v<A, Two> && std::is_same_v<B, Wide>)
          return launch_pair<A, Ring<128, 128, 1, 2, 4, false, false, EPI_W>>(a, b, s);     // (the same sums)
        else if constexpr (std::is_same_v<A, Two> && 2 * B::kSmem <= 160 * 1024 && B::kThreads == 512)
          return launch_pair<A, B>(a, b, s);
        else
          return kApart;
      });
    } else {
      return kApart;
    }
  });
}

}  // namespace
}  // namespace seco

extern "C" int dec_gemm_supported(int form, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
  const int64_t big = (int64_t)1 << 30;
  if (M < 1 || N < 8 || K < 1 || N % 8 || lda % 8 || ldb % 8 || ldc % 8) return 0;
  if (form == DEC_GEMM_TN ? (M < 8 || M % 8) : K % 64) return 0;
  // offsets inside an operand are 32-bit: outer indices times row length (KC), 64 rows (KR)
  const int64_t ra = form == DEC_GEMM_TN ? 64 : M, rb = form == DEC_GEMM_NT ? N : 64;
  return M < big && N < big && K < big && ra * lda < big && rb * ldb < big && ((M + 63) / 64) * ((N + 63) / 64) < big;
}

extern "C" int dec_gemm(int form, int epilogue, const void* a, const void* b, void* c, void* c2, int64_t M, int64_t N, int64_t K,
                        int64_t lda, int64_t ldb, int64_t ldc, void* stream) {
  using namespace seco;
  if (!dec_gemm_supported(form, M, N, K, lda, ldb, ldc)) return SECO_ERR_SHAPE;
  if (!a || !b || !c || ((epilogue == DEC_GEMM_SILU || epilogue == DEC_GEMM_SILU_BWD) && !c2)) return SECO_ERR_NULL;
  if (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)c2) & 15u) return SECO_ERR_ALIGN;
  const GemmArgs g{static_cast<const char*>(a), static_cast<const char*>(b), static_cast<__bf16*>(c), static_cast<__bf16*>(c2),
                   (int)M, (int)N, (int)K, (int)lda, (int)ldb, (int)ldc, 0, 0, 0, 0, 0};
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (form == DEC_GEMM_NN && epilogue == DEC_GEMM_STORE) return pick<true, false, kStore>(g, s);
  if (form == DEC_GEMM_NN && epilogue == DEC_GEMM_SILU) return pick<true, false, kSilu>(g, s);
  if (form == DEC_GEMM_NT && epilogue == DEC_GEMM_STORE) return pick<true, true, kStore>(g, s);
  if (form == DEC_GEMM_NT && epilogue == DEC_GEMM_SILU_BWD) return pick<true, true, kSiluBwd>(g, s);
  if (form == DEC_GEMM_TN && epilogue == DEC_GEMM_STORE) return pick<false, false, kStore>(g, s);
  if (form == DEC_GEMM_TN && epilogue == DEC_GEMM_ADD) return pick<false, false, kAdd>(g, s);
  return SECO_ERR_SHAPE;
}

static int gemm_grads(bool first, const void* dy, const void* w, void* dx, void* u, const void* x, void* dw, int64_t M, int64_t K, int64_t n,
                      void* stream) {
  using namespace seco;
  if (!dec_gemm_supported(DEC_GEMM_NT, M, K, n, n, n, K) || !dec_gemm_supported(DEC_GEMM_TN, K, n, M, K, n, n)) return SECO_ERR_SHAPE;
  if (!dy || !w || !dx || !x || !dw) return SECO_ERR_NULL;
  if (((uintptr_t)dy | (uintptr_t)w | (uintptr_t)dx | (uintptr_t)u | (uintptr_t)x | (uintptr_t)dw) & 15u) return SECO_ERR_ALIGN;
  const GemmArgs a{static_cast<const char*>(dy), static_cast<const char*>(w), static_cast<__bf16*>(dx), static_cast<__bf16*>(u),
                   (int)M, (int)K, (int)n, (int)n, (int)n, (int)K, 0, 0, 0, 0, 0};
  const GemmArgs b{static_cast<const char*>(x), static_cast<const char*>(dy), static_cast<__bf16*>(dw), nullptr,
                   (int)K, (int)n, (int)M, (int)K, (int)n, (int)n, 0, 0, 0, 0, 0};
  hipStream_t s = static_cast<hipStream_t>(stream);
  int rc = first ? (u ? pair<kSiluBwd, kStore>(a, b, s) : pair<kStore, kStore>(a, b, s)) : u ? pair<kSiluBwd, kAdd>(a, b, s) : pair<kStore, kAdd>(a, b, s);
  if (rc != kApart) return rc;
  rc = u ? pick<true, true, kSiluBwd>(a, s) : pick<true, true, kStore>(a, s);
  return rc ? rc : first ? pick<false, false, kStore>(b, s) : pick<false, false, kAdd>(b, s);
}
extern "C" int dec_gemm_grads(const void* dy, const void* w, void* dx, void* u, const void* x, void* dw, int64_t M, int64_t K, int64_t n,
                              void* stream) {
  return gemm_grads(false, dy, w, dx, u, x, dw, M, K, n, stream);
}
extern "C" int dec_gemm_qkv(const void* h, const void* w, void* qkv, void* k, void* v, const int64_t* kv_stride, int64_t B, int64_t Hq,
                            int64_t Hkv, int64_t C, int64_t K, int64_t row0, float base, void* stream) {
  using namespace seco;
  if (!h || !w || !qkv || !k || !v || !kv_stride) return SECO_ERR_NULL;
  if (B < 1 || Hq < 1 || Hkv < 1 || C < 1 || row0 < 0) return SECO_ERR_SHAPE;
  if (!(base > 1.f) || !std::isfinite(base)) return SECO_ERR_RANGE;
  const int64_t big = (int64_t)1 << 30;
  if (B > 65535 || C > big || Hq > 65535 || Hkv > 65535) return SECO_ERR_TOO_LARGE;
  const int64_t M = B * C, N = (Hq + 2 * Hkv) * 128;
  for (int i = 0; i < 3; ++i)
    if (kv_stride[i] < 0 || kv_stride[i] % 8 != 0) return SECO_ERR_ALIGN;
  if (((uintptr_t)h | (uintptr_t)w | (uintptr_t)qkv | (uintptr_t)k | (uintptr_t)v) & 15u) return SECO_ERR_ALIGN;
  if (!dec_gemm_supported(DEC_GEMM_NN, M, N, K, K, N, N)) return SECO_ERR_SHAPE;
  QkvArgs g;
  static_cast<GemmArgs&>(g) = {static_cast<const char*>(h), static_cast<const char*>(w), static_cast<__bf16*>(qkv), nullptr,
                               (int)M, (int)N, (int)K, (int)K, (int)N, (int)N, 0, 0, 0, 0, 0};
  g.k = static_cast<__bf16*>(k);
  g.v = static_cast<__bf16*>(v);
  for (int i = 0; i < 3; ++i) g.ks[i] = kv_stride[i];
  g.row0 = row0;
  g.chunk = (int)C;
  g.Hq = (int)Hq;
  g.Hkv = (int)Hkv;
  g.by_chunk = make_div((int)C);
  g.powers = rope_powers(128, base);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int rc = with_way<true, false, kQkv>(g, [&](auto way) {
    using T = typename decltype(way)::type;
    if constexpr (T::kBM <= 64)
      return launch<T>(g, s);
    else
      return kApart;             // (a thread of the large tiles would hold the sines of four rows or more)
  });
  if (rc != kApart) return rc;
  if (const int st = pick<true, false, kStore>(g, s)) return st;
  return dec_rope_qkv(SECO_BF16, 0, qkv, k, v, kv_stride, B, Hq, Hkv, C, 128, row0, base, stream);
}
extern "C" int dec_gemm_first_grads(const void* dy, const void* w, void* dx, void* u, const void* x, void* dw, int64_t M, int64_t K, int64_t n,
                                    void* stream) {
  return gemm_grads(true, dy, w, dx, u, x, dw, M, K, n, stream);
}
