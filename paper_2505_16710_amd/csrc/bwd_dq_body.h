// dQ of one chunk, bf16 matrix cores: dQ = s * dS K over ALL visible cache rows, with
// P = exp(S - LSE), dS = P * (dO V^T - delta), delta = rowsum(dO * O) (computed in this kernel's prologue).  (SpaCO keeps dQ exact: a selected chunk's
// graph is rebuilt against every earlier cache, Alg. 2.)
//
// Same row-parallel decomposition as the forward, in the same two workgroup shapes: a workgroup
// owns 128 query rows of one head, a wavefront 32 of them; K and V tiles stream through
// swizzled, double-buffered LDS, copied global -> LDS directly one tile ahead; with KH = 2 (8 wavefronts, 128-row tiles) the two wavefronts
// of a row block take one 64-row half of every tile each and their partial dQ are added
// through LDS at the end.  Scores are again computed transposed (S^T = K Q^T, dP^T = V dO^T)
// so that LSE and delta are one or two values per lane and dS^T feeds dQ^T += K^T dS^T from registers;
// K^T comes from the same K tile through the LDS transpose read.
//
// Bound: power on long calls, as the forward, and products of 16x16x32 for the same reason (half the accumulator traffic of
// 32x32x16): 2048 rows at 30720 of 32/8 heads 1278 -> 1236 us (2.03 GHz and the matrix pipe 59 % busy, before 1.81 and 66 %),
// 1024 at 15360 345 -> 320, two sequences of 777 at 9324 366 -> 351.  Operands are read kAhead pairs of products ahead, held
// there by a scheduling barrier per pair (2, 3, 4: within 1 % here, in the launch with dK/dV 2 is the fastest).  Writing dS of one block of 32 cache rows under the products
// of the other (48 registers of scores for 32) spills 26 registers and more, which costs a third.
//
// Column-weighted dQ (SPARSE = true): the tiles are taken from a by-value table of runs of cache rows, each with
// one positive weight w, instead of from all visible rows: dQ = s * sum over the runs of w * dS K.  A tile starts
// where its run starts (not on a multiple of the tile height), rows past the run's end are masked like rows above
// the diagonal, and the weight costs nothing per element: P * w = exp2(S - (LSE - log2 w)), one logarithm per
// tile.  With every chunk sampled with probability pi and weighted 1 / pi this is an unbiased estimate of dQ
// whose cost does not grow with the number of unvisited rows.
//
// Short chunks (SPLIT = kDivided): as in the forward, the rows of the G heads of a KV head are packed into one row
// space and the visible cache rows of a row tile are divided among n_splits workgroups; each writes its partial
// dQ (fp32, unscaled) to the workspace and dq_merge_kernel adds the partials in split order.
//
// Between one and two rounds of workgroups (SPLIT = kShares): packed row tiles too, but only those beyond the first round
// are divided (row_shares in seco_internal.h); the others are written as they are.
#pragma once
#include "mfma_tiles.h"
#include "seco_internal.h"

namespace seco {
namespace {

constexpr int BM = 128;
constexpr int BNW = 64;   // cache rows per wavefront and tile
constexpr int kAhead = 2; // operand reads in flight ahead of the products

// The products of a wavefront, in either shape of the matrix instructions: what a lane holds of its 32 query rows.
// 16x16x32: two rows, 16 apart, and of each of their fragments every fourth chunk of head_dim.
struct DqProducts16 {
  static constexpr bool k16 = true;
  static constexpr int kRows = 2;
  using Acc = f32x4[8][2];
  int r_off[4], t_off[8];                      // lane-dependent parts of the LDS operand addresses, constant for the whole kernel
  __device__ __forceinline__ DqProducts16(int lane, int base) {
#pragma unroll
    for (int t = 0; t < 4; ++t) r_off[t] = row16_lane_off(t, lane) + base;
#pragma unroll
    for (int db = 0; db < 8; ++db) t_off[db] = tr16_lane_off(db, lane) + base;
  }
  static __device__ __forceinline__ void frags(bf16x8 (&f)[8], const bf16x8 (&x)[8], lds_char* own, int lane) { rows16_to_frags(f, x, own, lane); }
  static __device__ __forceinline__ void clear(Acc& acc) {
#pragma unroll
    for (int db = 0; db < 8; ++db) acc[db][0] = acc[db][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // delta of the lane's rows: O (as load_rows32 brings it) times dO (the same, and its fragments)
  static __device__ __forceinline__ void row_dots(float (&d)[kRows], const bf16x8 (&o)[8], const bf16x8 (&)[8], const bf16x8 (&dof)[8], lds_char* own, int lane) {
    bf16x8 of[8];
    rows16_to_frags(of, o, own, lane);
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) d[qb] = row16_dot(of + 4 * qb, dof + 4 * qb, lane);
  }
  static __device__ __forceinline__ f32x4 piece(const Acc& acc, int i) { return acc[i >> 1][i & 1]; }
  static __device__ __forceinline__ void add(Acc& acc, int i, f32x4 x) { acc[i >> 1][i & 1] += x; }
  static __device__ __forceinline__ void store_part(const Acc& acc, float* base, int n_rows, lds_char* own) { store_part16(acc, base, n_rows, own); }
  static __device__ __forceinline__ void store(const Acc& acc, float scale, __bf16* base, int64_t stride, int row0, int n_rows, lds_char* own8k) {
    store_rows16([&](int db, int qb, int i) { return acc[db][qb][i] * scale; }, base, stride, row0, n_rows, own8k);
  }
};
// 32x32x16: one row, every second chunk.  For launches of whole row tiles that leave CUs without work (dq_leaves_cus): with the clock
// as high as it goes what counts is the room for vector instructions (see Products32 in bwd_dkdv_body.h).
struct DqProducts32 {
  static constexpr bool k16 = false;
  static constexpr int kRows = 1;
  using Acc = f32x16[4];
  int r_off[8];
  TrOff t_off[4];
  __device__ __forceinline__ DqProducts32(int lane, int base) {
#pragma unroll
    for (int t = 0; t < 8; ++t) r_off[t] = row8_lane_off(lane & 31, 2 * t + (lane >> 5)) + base;
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      t_off[db] = tr8_lane_off(db, lane);
      t_off[db].lo += base;
      t_off[db].hi += base;
    }
  }
  static __device__ __forceinline__ void frags(bf16x8 (&f)[8], const bf16x8 (&x)[8], lds_char* own, int lane) { rows32_to_frags(f, x, own, lane); }
  static __device__ __forceinline__ void clear(Acc& acc) {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
  }
  static __device__ __forceinline__ void row_dots(float (&d)[kRows], const bf16x8 (&o)[8], const bf16x8 (&d_o)[8], const bf16x8 (&)[8], lds_char* own, int lane) {
    bf16x8 of[8], df[8];                       // (the operands of 16x16x32: the same bits)
    rows16_to_frags(of, o, own, lane);
    rows16_to_frags(df, d_o, own, lane);
    const float lo = row16_dot(of, df, lane), hi = row16_dot(of + 4, df + 4, lane);
    d[0] = lane & 16 ? hi : lo;
  }
  static __device__ __forceinline__ f32x4 piece(const Acc& acc, int i) {
    const f32x16& x = acc[i >> 2];
    const int r = 4 * (i & 3);
    return f32x4{x[r], x[r + 1], x[r + 2], x[r + 3]};
  }
  static __device__ __forceinline__ void add(Acc& acc, int i, f32x4 x) {
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i >> 2][4 * (i & 3) + r] += x[r];
  }
  static __device__ __forceinline__ void store(const Acc& acc, float scale, __bf16* base, int64_t stride, int row0, int n_rows, lds_char* own8k) {
    store_rows32([&](int db, int r) { return acc[db][r] * scale; }, base, stride, row0, n_rows, own8k);
  }
};

// seg (SPARSE only): runs of cache rows in ascending order, each with a positive weight
// smem: 4 * kTileBytes, [buf][K|V]
// FUSED: inside the kernel that holds dK/dV too, where scalar registers are short (opaque)
template <int KH, int SPLIT, bool SPARSE, class Products, bool FUSED = false>
__device__ __forceinline__ void dq_bf16_body(const AttnParams& p, const SegTable& seg, int n_mtiles, int item, lds_char* smem) {
  static_assert(!SPLIT || KH == 2, "the split variant uses the 8-wavefront shape");
  static_assert(Products::k16 || (KH == 2 && !SPLIT), "32x32x16: whole row tiles of 8 wavefronts");
  constexpr int BN = BNW * KH;
  constexpr int kTileBytes = BN * kRowBytes;
  // (the wavefront index through readfirstlane: the compiler then knows that it, and every tile coordinate and branch
  // condition derived from it, is uniform over the wavefront and keeps them in scalar registers)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kRows = Products::kRows, kLaneRows = 32 / kRows;     // query rows of a lane; lanes of a wavefront with rows of their own
  const int g = lane / kLaneRows, pg = Products::k16 ? pi4(g) : g;
  const int rb = wave & 3, kh = (KH == 1 && !SPARSE) ? 0 : wave >> 2;
  int b, kvh, h, mt, m0, sp = 0;              // m0: first chunk-local row of this wavefront
  int n_sp = 1, slot = 0;                     // shares of this row tile; kShares: where this one's sums go
  if constexpr (SPLIT) {
    int rest;
    if constexpr (SPLIT == kDivided) {
      n_sp = p.n_splits;
      const int tiles = over(item, p.by_splits);
      sp = item - tiles * n_sp;
      rest = over(tiles, p.by_tiles);
      mt = n_mtiles - 1 - (tiles - rest * n_mtiles);
    } else {
      const int n_cut = n_mtiles - p.rows_whole, n_first = p.B * p.Hkv * p.rows_whole;   // (the whole tiles come first)
      if (item < n_first) {
        rest = item / p.rows_whole;
        mt = n_mtiles - 1 - (item - rest * p.rows_whole);
      } else {
        n_sp = p.n_splits;
        slot = item - n_first;
        rest = slot / (n_cut * n_sp);
        const int e = slot - rest * (n_cut * n_sp);
        sp = e % n_sp;
        mt = n_cut - 1 - e / n_sp;
      }
    }
    b = over(rest, p.by_Hkv);
    kvh = rest - b * p.Hkv;
    const int v0 = mt * BM + rb * 32;          // packed row: head v0 / Cpad of the group, row v0 % Cpad
    int hg = over(v0, p.by_Cpad);
    m0 = v0 - hg * p.Cpad;
    if (hg >= p.G) {                           // past the last head of the group: idle wavefront (m0 >= C)
      hg = p.G - 1;
      m0 = p.Cpad;
    }
    h = kvh * p.G + hg;
  } else {
    // (launches of their own are long and bound by power: behind plain divisions the loop's registers come out so that it is 0.5 %
    // faster)
    const int tiles = FUSED ? over(item, p.by_G) : item / p.G, hg = item - tiles * p.G, rest = FUSED ? over(tiles, p.by_tiles) : tiles / n_mtiles;
    mt = n_mtiles - 1 - (tiles - rest * n_mtiles);
    b = FUSED ? over(rest, p.by_Hkv) : rest / p.Hkv;
    kvh = rest - b * p.Hkv;
    h = kvh * p.G + hg;
    m0 = mt * BM + rb * 32;
  }

  const int kv_len = p.q_start + p.C;
  const int row = m0 + lane % kLaneRows;       // this lane's first row; a second one is 16 on
  const int qpos = p.q_start + row;
  // Q, dO, O, the row's LSE and (below) the first K/V tile are all requested before the first of them is waited for:
  // a workgroup starts with one memory round trip
  bf16x8 qr[8], dor[8], orow[8];
  {
    const int64_t ob = b * p.os[0] + h * p.os[1];
    load_rows32(qr, static_cast<const __bf16*>(p.q) + b * p.qs[0] + h * p.qs[1], p.qs[2], m0, p.C - 1, lane);
    load_rows32(dor, static_cast<const __bf16*>(p.d_o) + ob, p.os[2], m0, p.C - 1, lane);
    load_rows32(orow, static_cast<const __bf16*>(p.o) + ob, p.os[2], m0, p.C - 1, lane);
  }
  const float* lse_h = p.lse + ((int64_t)b * p.Hq + h) * p.C;
  float lse[kRows];
#pragma unroll
  for (int qb = 0; qb < kRows; ++qb) lse[qb] = lse_h[min(row + 16 * qb, p.C - 1)];
  const float c = p.scale * kLog2e;

  const __bf16* kbase = static_cast<const __bf16*>(p.k) + b * p.kvs[0] + kvh * p.kvs[1];
  const __bf16* vbase = static_cast<const __bf16*>(p.v) + b * p.kvs[0] + kvh * p.kvs[1];
  int wg_kv_end;                               // columns any row of the workgroup sees
  if constexpr (SPLIT) {
    int rows_end = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int v = mt * BM + r * 32, hh = over(v, p.by_Cpad), mm = v - hh * p.Cpad;
      if (hh < p.G && mm < p.C) rows_end = max(rows_end, min(mm + 32, p.C));
    }
    wg_kv_end = rows_end ? p.q_start + rows_end : 0;
  } else {
    wg_kv_end = p.q_start + min((mt + 1) * BM, p.C);
  }
  // SPARSE: position in the run table = (run, first cache row of the tile, end of the run clipped to the rows
  // this workgroup sees); runs that start at or past that limit have no tiles
  struct Cur { int si, col, end; };
  auto run_at = [&](int si) { return Cur{si, seg.col_begin[si], min(seg.col_end[si], wg_kv_end)}; };
  auto advance = [&](Cur x) {
    x.col += BN;
    if (x.col >= x.end && x.si + 1 < seg.n) x = run_at(x.si + 1);
    return x;
  };
  int n_tiles = (wg_kv_end + BN - 1) / BN;
  if constexpr (SPARSE) {
    n_tiles = 0;
    for (int si = 0; si < seg.n; ++si) {
      const int len = min(seg.col_end[si], wg_kv_end) - seg.col_begin[si];
      if (len > 0) n_tiles += (len + BN - 1) / BN;
    }
  }
  const int wave_kv_end = m0 < p.C ? p.q_start + min(m0 + 32, p.C) : 0;
  int n_begin = 0, n_end = n_tiles;            // tiles of this workgroup
  if constexpr (SPLIT) {
    const int per = SPLIT == kDivided ? over(n_tiles + n_sp - 1, p.by_splits) : 0;
    n_begin = sp * per;
    n_end = min(n_tiles, n_begin + per);       // may be empty: the partial written below is then all zero
    if constexpr (SPLIT == kShares) {          // (never empty: there are at least as many tiles as shares)
      n_begin = sp * n_tiles / n_sp;
      n_end = (sp + 1) * n_tiles / n_sp;
    }
  }

  // asynchronous global -> LDS copy of one K and one V tile: each wavefront copies 4 groups of 4 rows of each.
  // The per-lane byte offsets inside a tile never change; a tile that lies entirely inside the cache is copied
  // from a scalar base address with no vector arithmetic, the last (ragged) one with clamped per-lane addresses.
  uint32_t lane_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) lane_off[i] = dma_lane_offset(4 * (wave + 4 * KH * i), p.kvs[2] * 2, lane);
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + wave * 4 * kRowBytes);
  auto copy_tile = [&](int col, int buf) {      // col: first cache row of the tile
    if (col + BN <= kv_len) {
      const __bf16* kt_src = kbase + (int64_t)col * p.kvs[2];
      const __bf16* vt_src = vbase + (int64_t)col * p.kvs[2];
      const uint32_t lds = FUSED ? opaque(lds_wave) : lds_wave;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t dst = lds + buf * 2 * kTileBytes + i * (16 * KH * kRowBytes);
        dma16_sbase(kt_src, lane_off[i], dst);
        dma16_sbase(vt_src, lane_off[i], dst + kTileBytes);
      }
    } else {                                   // rows past the cache's end repeat its last one
      const __bf16* kt_src = kbase + (int64_t)col * p.kvs[2];
      const __bf16* vt_src = vbase + (int64_t)col * p.kvs[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t dst = lds_wave + buf * 2 * kTileBytes + i * (16 * KH * kRowBytes);
        const uint32_t past = max(4 * (wave + 4 * KH * i) + (lane >> 4) + col - (kv_len - 1), 0);
        const uint32_t off = lane_off[i] - __umul24(past, (uint32_t)p.kvs[2] * 2u);
        dma16_sbase(kt_src, off, dst);
        dma16_sbase(vt_src, off, dst + kTileBytes);
      }
    }
  };

  // (dense variants: the wavefront's half of the tile, for KH = 2, is part of the per-lane offsets, so that a tile's
  // base is a compile-time constant in the unrolled loop below)
  const Products pr(lane, SPARSE ? 0 : kh * BNW * kRowBytes);
  typename Products::Acc dq;
  Products::clear(dq);

  Cur cur{0, n_begin * BN, 0};
  if constexpr (SPARSE) {
    cur = run_at(0);
    for (int i = 0; i < n_begin && i < n_tiles; ++i) cur = advance(cur);
  }
  Cur nxt = cur;
  if (n_begin < n_end) copy_tile(cur.col, 0);
  bf16x8 qf[8], dof[8];
  lds_char* own = smem + 2 * kTileBytes + wave * 8192;      // of the second tile buffer, which is empty until the loop
  Products::frags(qf, qr, own, lane);
  Products::frags(dof, dor, own, lane);
  // delta = rowsum(dO * O).  It is also written to the workspace for the
  // dK/dV kernel that follows on the same stream, negated, together with -LSE / s (the log-sum-exp in units of the unscaled dot
  // product): the two values that kernel starts its MFMA chains from.
  float lse_c[kRows], delta[kRows];
  Products::row_dots(delta, orow, dor, dof, own, lane);
#pragma unroll
  for (int qb = 0; qb < kRows; ++qb) {
    lse_c[qb] = lse[qb] * kLog2e;
    if (kh == 0 && sp == 0 && g == 0 && row + 16 * qb < p.C) {
      const int64_t kept = ((int64_t)b * p.Hq + h) * p.stat_stride + p.stat_off + row + 16 * qb;
      p.delta[kept] = -delta[qb];
      p.nlse2[kept] = -lse[qb] / p.scale;
    }
  }
  dma_wait_all();
  __syncthreads();

  if constexpr (SPARSE) {
    for (int n = n_begin; n < n_end; ++n) {
      const int buf = (n - n_begin) & 1;
#include "bwd_dq_tile_step.inc"
    }
  } else {
    for (int n0 = n_begin; n0 < n_end; n0 += 2) {
      {
        constexpr int buf = 0;
        const int n = n0;
#include "bwd_dq_tile_step.inc"
      }
      if (n0 + 1 >= n_end) break;
      {
        constexpr int buf = 1;
        const int n = n0 + 1;
#include "bwd_dq_tile_step.inc"
      }
    }
  }

  if (KH == 2) {
    // add the partial dQ of the two column halves of each row block through LDS
    lds_char* slot = smem + rb * (17 * 1024);
    if (kh == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i) *reinterpret_cast<SECO_LDS f32x4*>(slot + (i * 64 + lane) * 16) = Products::piece(dq, i);
    }
    __syncthreads();
    if (kh == 1 || m0 >= p.C) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) Products::add(dq, i, *reinterpret_cast<SECO_LDS f32x4*>(slot + (i * 64 + lane) * 16));
  }

  if constexpr (SPLIT == kShares) {
    if (n_sp > 1) {                            // all 32 rows: the merge takes those that exist
      Products::store_part(dq, p.part + ((int64_t)slot * BM + rb * 32) * kHeadDim, 32, smem + rb * (17 * 1024));
      return;
    }
  }
  if constexpr (SPLIT == kDivided) {
    float* po = p.part + ((int64_t)sp * p.B * p.Hq * p.C + ((int64_t)b * p.Hq + h) * p.C + m0) * kHeadDim;
    Products::store_part(dq, po, p.C - m0, smem + rb * (17 * 1024));
    return;
  }

  Products::store(dq, p.scale, static_cast<__bf16*>(p.d_q) + b * p.qs[0] + h * p.qs[1], p.qs[2], m0, p.C,
                  KH == 2 ? smem + rb * (17 * 1024) : smem + wave * 8192);
}

}  // namespace
}  // namespace seco
