// Forward of one chunk, bf16 matrix cores (Eq. 1 at the attention layer):
// O = softmax(s Q K^T) V over cache rows [0, q_start + C) with the causal rule
// col <= q_start + row, plus the per-row log-sum-exp.
//
// Decomposition.  A workgroup owns 128 query rows of one head; a wavefront owns 32 of them and
// keeps Q^T fragments, the running max / sum and the O^T accumulator (128 x 32, fp32) in
// registers.  K and V tiles stream through swizzled LDS tiles shared by the workgroup, copied
// global -> LDS directly ahead of their use.  Two shapes of workgroup:
//   4 wavefronts (fwd4_bf16.hip): tiles of 64 cache rows, 80 KiB of LDS -> two workgroups per CU; used when a
//       call has two row tiles per CU or close to it (launch_fwd_bf16);
//   8 wavefronts (this header): tiles of 128 cache rows in two buffers of a K and a V tile; wavefront (rb, kh)
//       handles row block rb and the kh-th 64-row half of every tile, and the two partial (max, sum, O) of a
//       row block are merged through LDS at the end.  One such workgroup fills a CU with two wavefronts per
//       SIMD, which is what calls with few row tiles need (a 1024-row chunk of a 32-head layer has only 256
//       row tiles for 256 CUs).
//
// Short chunks (SPLIT = kDivided).  With chunks of 32 .. 512 rows (the sizes of the paper's chunk-size study,
// Sec. 6.3) a call has far fewer row tiles than the GPU has CUs and every tile would stream the whole cache
// alone.  The split variant therefore (a) packs the rows of the G query heads that share a KV head into one row
// space of G * roundup(C, 32) rows, so that a workgroup's K/V tiles serve several heads, and (b) divides the
// visible cache rows of a row tile among n_splits workgroups (split_count); each writes its un-normalised partial O with
// its reference maximum and sum (fp32) to the workspace, and fwd_merge_kernel combines the partials in split order.
// (With the 4-wavefront kernel here twice as many partials were written and merged: 32 rows x 32 heads against 16K cache
// rows 32.1 us, now 24.2; 256 rows against 2304 29.1, now 24.6.)
//
// Between one and two rounds of workgroups (SPLIT = kShares): packed row tiles too, but only those beyond the first round are
// divided (row_shares in seco_internal.h); the others are written as they are.
//
// The score tile is computed transposed, S^T = K Q^T, so that a lane owns one query row
// (C layout: lane = column): row max / row sum are in-lane reductions plus one exchange with
// lane^32, the rescale of O^T is a per-lane scalar, and P^T feeds the second product
// O^T += V^T P^T straight from registers.  V^T comes from the row-major V tile through the
// LDS transpose read.
#pragma once
#include "mfma_tiles.h"
#include "seco_internal.h"

namespace seco {
namespace {

constexpr int BM = 128;  // query rows per workgroup
constexpr int BNW = 64;  // cache rows per wavefront and tile
constexpr float kBig = 1099511627776.f;   // 2^40: a tile's exponentials may sum to this before the reference moves

// 8-wavefront shape (see the head of the file)
template <int SPLIT>
__global__ __launch_bounds__(512, 2) void fwd8_bf16_kernel(AttnParams p, int n_mtiles, int total_items) {
  constexpr int KH = 2;
  constexpr int BN = BNW * KH;                 // cache rows per tile
  constexpr int kTileBytes = BN * kRowBytes;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];   // 4 * kTileBytes: [buf][K|V]
  lds_char* smem = (lds_char*)smem_raw;

  const int item = SPLIT == kShares ? shares_item(blockIdx.x, p.B * p.Hkv * p.rows_whole, total_items)
                                     : xcd_item(blockIdx.x, total_items, SPLIT == kDivided ? 8 : p.B * p.Hkv);
  if (item < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, g = lane >> 5;
  const int rb = wave & 3, kh = wave >> 2;
  int b, kvh, h, mt, m0, sp = 0;              // m0: first chunk-local row of this wavefront
  int n_sp = 1, share_slot = 0;                // shares of this row tile; kShares: where this one's sums go
  if constexpr (SPLIT) {
    // item -> (batch, kv head, row tile of the packed row space, split)
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
        share_slot = item - n_first;
        rest = share_slot / (n_cut * n_sp);
        const int e = share_slot - rest * (n_cut * n_sp);
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
    // item -> (batch, kv head, row tile (heavy first), head within the group)
    const int tiles = over(item, p.by_G), hg = item - tiles * p.G, rest = over(tiles, p.by_tiles);
    mt = n_mtiles - 1 - (tiles - rest * n_mtiles);
    b = over(rest, p.by_Hkv);
    kvh = rest - b * p.Hkv;
    h = kvh * p.G + hg;
    m0 = mt * BM + rb * 32;
  }

  const int kv_len = p.q_start + p.C;
  const int row = m0 + l32;                    // this lane's row
  const int qpos = p.q_start + row;            // its global position
  bf16x8 qr[8];
  load_rows32(qr, static_cast<const __bf16*>(p.q) + b * p.qs[0] + h * p.qs[1], p.qs[2], m0, p.C - 1, lane);

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
  const int n_tiles = (wg_kv_end + BN - 1) / BN;
  const int wave_kv_end = m0 < p.C ? p.q_start + min(m0 + 32, p.C) : 0;  // columns this wavefront sees
  int n_begin = 0, n_end = n_tiles;            // tiles of this workgroup
  auto part_row_of = [&]() { return (int64_t)sp * p.B * p.Hq * p.C + ((int64_t)b * p.Hq + h) * p.C + row; };
  if constexpr (SPLIT == kShares) {            // (never empty: there are at least as many tiles as shares)
    n_begin = sp * n_tiles / n_sp;
    n_end = (sp + 1) * n_tiles / n_sp;
  }
  if constexpr (SPLIT == kDivided) {
    const int per = over(n_tiles + p.n_splits - 1, p.by_splits);
    n_begin = sp * per;
    n_end = min(n_tiles, n_begin + per);
    if (n_begin >= n_end) {                    // nothing to do for this split: an empty partial (max = -inf)
      if (kh == 0 && row < p.C && g == 0) {
        const int64_t part_row = part_row_of();
        p.part_ml[2 * part_row] = -INFINITY;
        p.part_ml[2 * part_row + 1] = 0.f;
      }
      return;
    }
  }

  // asynchronous global -> LDS copy of one K and one V tile: each wavefront copies 4 groups of 4 rows of each.
  // The per-lane byte offsets inside a tile never change; a tile that lies entirely inside the cache is copied
  // from a scalar base address with no vector arithmetic, the last (ragged) one with clamped per-lane addresses.
  uint32_t lane_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) lane_off[i] = dma_lane_offset(4 * (wave + 4 * KH * i), p.kvs[2] * 2, lane);
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + wave * 4 * kRowBytes);
  auto copy_tile = [&](int n, int buf) {
    if ((n + 1) * BN <= kv_len) {
      const __bf16* kt_src = kbase + (int64_t)n * BN * p.kvs[2];
      const __bf16* vt_src = vbase + (int64_t)n * BN * p.kvs[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t dst = lds_wave + buf * 2 * kTileBytes + i * (16 * KH * kRowBytes);
        dma16_sbase(kt_src, lane_off[i], dst);
        dma16_sbase(vt_src, lane_off[i], dst + kTileBytes);
      }
    } else {                                   // rows past the cache's end repeat its last one
      const __bf16* kt_src = kbase + (int64_t)n * BN * p.kvs[2];
      const __bf16* vt_src = vbase + (int64_t)n * BN * p.kvs[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t dst = lds_wave + buf * 2 * kTileBytes + i * (16 * KH * kRowBytes);
        const uint32_t past = max(4 * (wave + 4 * KH * i) + (lane >> 4) + n * BN - (kv_len - 1), 0);
        const uint32_t off = lane_off[i] - __umul24(past, (uint32_t)p.kvs[2] * 2u);
        dma16_sbase(kt_src, off, dst);
        dma16_sbase(vt_src, off, dst + kTileBytes);
      }
    }
  };

  f32x16 o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c = p.scale * kLog2e;

  // lane-dependent parts of the LDS operand addresses (constant for the whole kernel)
  int r_off[8];
  TrOff t_off[4];
#pragma unroll
  for (int t = 0; t < 8; ++t) r_off[t] = row8_lane_off(l32, 2 * t + g) + kh * BNW * kRowBytes;
#pragma unroll
  for (int db = 0; db < 4; ++db) {
    t_off[db] = tr8_lane_off(db, lane);
    t_off[db].lo += kh * BNW * kRowBytes + kTileBytes;
    t_off[db].hi += kh * BNW * kRowBytes + kTileBytes;
  }

  copy_tile(n_begin, 0);
  bf16x8 qf[8];
  rows32_to_frags(qf, qr, smem + 2 * kTileBytes + wave * 8192, lane);   // (the second tile buffer is empty until the loop)
  settle8(qf);
  dma_wait_all();
  __syncthreads();

  for (int n = n_begin; n < n_end; ++n) {
    const int buf = (n - n_begin) & 1;
    if (n + 1 < n_end) copy_tile(n + 1, buf ^ 1);
    const int col0 = n * BN + kh * BNW;        // first cache row of this wavefront's part of the tile
    if (col0 < wave_kv_end) {
      lds_char* kt = smem + buf * 2 * kTileBytes;
      f32x16 s[2];
#pragma unroll
      for (int kvb = 0; kvb < 2; ++kvb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kvb][r] = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) s[kvb] = mfma(lds_row8_at(kt + r_off[t], kvb * 32), qf[t], s[kvb]);
      }
      if (col0 + BNW - 1 > p.q_start + m0) {  // reaches past this wavefront's first row: causal mask
#pragma unroll
        for (int kvb = 0; kvb < 2; ++kvb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int kv = col0 + kvb * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
            if (kv > qpos) s[kvb][r] = -INFINITY;
          }
      }
      // Reference value of the row's exponentials.  A max subtraction only guards against overflow, so the
      // reference m_run is kept as it is as long as the exponentials stay representable: the (costly) row maximum
      // is computed only on a row's first visible tile and when the tile's sum of exponentials exceeds kBig = 2^40,
      // which for a whole kernel is a handful of times.  Exponentials may thus reach 2^40; bf16 and fp32 have
      // the exponent range for that, and O and the sum are rescaled together when the reference moves.
      auto tile_max = [&]() {
        float mx = s[0][0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[0][r]);
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[1][r]);
        return fmaxf(mx, __shfl_xor(mx, 32)) * c;
      };
      auto move_reference = [&](float m_new) {          // m_new >= m_run; exp2(-inf - x) = 0 on the first tile
        const float alpha = fast_exp2(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
        m_run = m_new;
      };
      if (__builtin_amdgcn_ballot_w64(m_run == -INFINITY) != 0) {      // some row has seen nothing yet
        const float m_blk = tile_max();
        if (m_run == -INFINITY && m_blk != -INFINITY) m_run = m_blk;    // (o and l_run are still zero)
      }
      // a part of a tile can be fully masked for a row (only when kh > 0 or q_start is unaligned): such a row
      // has seen nothing yet and keeps m_run = -inf; use 0 so that exp2(-inf - (-inf)) never appears
      float m_use = m_run == -INFINITY ? 0.f : m_run;
      float sum = 0.f;
      f32x16 e[2];
#pragma unroll
      for (int kvb = 0; kvb < 2; ++kvb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          e[kvb][r] = fast_exp2(__builtin_fmaf(s[kvb][r], c, -m_use));
          sum += e[kvb][r];
        }
      if (__builtin_amdgcn_ballot_w64(!(sum <= kBig)) != 0) {           // reference too low for this tile (rare)
        const float m_blk = tile_max();
        if (m_blk > m_run) move_reference(m_blk);
        m_use = m_run == -INFINITY ? 0.f : m_run;
        sum = 0.f;
#pragma unroll
        for (int kvb = 0; kvb < 2; ++kvb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            e[kvb][r] = fast_exp2(__builtin_fmaf(s[kvb][r], c, -m_use));
            sum += e[kvb][r];
          }
      }
#pragma unroll
      for (int kvb = 0; kvb < 2; ++kvb) s[kvb] = e[kvb];
      l_run += sum;
#pragma unroll
      for (int kvb = 0; kvb < 2; ++kvb)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const bf16x8 pb = pack8(s[kvb], t);
#pragma unroll
          for (int db = 0; db < 4; ++db) o[db] = mfma(lds_tr8_at(kt, t_off[db], kvb * 32 + 16 * t), pb, o[db]);
        }
    }
    dma_wait_all();
    __syncthreads();
  }

  float l_tot = l_run + __shfl_xor(l_run, 32);
  {
    // merge the two column halves of each row block: kh = 1 publishes (m, l, O), kh = 0 combines
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    lds_char* slot = smem + rb * (17 * 1024);            // 16 KiB of O + 512 B of (m, l) per row block
    if (kh == 1) {
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          f32x4 v = {o[db][4 * r4], o[db][4 * r4 + 1], o[db][4 * r4 + 2], o[db][4 * r4 + 3]};
          *reinterpret_cast<SECO_LDS f32x4*>(slot + ((db * 4 + r4) * 64 + lane) * 16) = v;
        }
      *reinterpret_cast<SECO_LDS float*>(slot + 16384 + lane * 4) = m_run;
      *reinterpret_cast<SECO_LDS float*>(slot + 16384 + 256 + lane * 4) = l_tot;
    }
    __syncthreads();
    if (kh == 1 || m0 >= p.C) return;
    const float m1 = *reinterpret_cast<SECO_LDS float*>(slot + 16384 + lane * 4);
    const float l1 = *reinterpret_cast<SECO_LDS float*>(slot + 16384 + 256 + lane * 4);
    // (finite where the workgroup starts at column 0; a share of the cache may lie past what a row sees)
    const float m = fmaxf(m_run, m1), m_sub = SPLIT && m == -INFINITY ? 0.f : m;
    float a0 = fast_exp2(m_run - m_sub), a1 = fast_exp2(m1 - m_sub);
    l_tot = l_tot * a0 + l1 * a1;
    m_run = m;
    if (SPLIT != kDivided && (SPLIT == kWholeTiles || n_sp == 1)) {
      const float inv = 1.f / l_tot;
      a0 *= inv;
      a1 *= inv;
    }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 v = *reinterpret_cast<SECO_LDS f32x4*>(slot + ((db * 4 + r4) * 64 + lane) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) o[db][4 * r4 + i] = o[db][4 * r4 + i] * a0 + v[i] * a1;
      }
  }

  if constexpr (SPLIT == kShares) {
    if (n_sp > 1) {                            // all 32 rows: the merge takes those that exist
      const int64_t part_row = (int64_t)share_slot * BM + rb * 32;
      store_part32(o, p.part + part_row * kHeadDim, 32, smem + rb * (17 * 1024));
      if (g == 0) {
        p.part_ml[2 * (part_row + l32)] = m_run;
        p.part_ml[2 * (part_row + l32) + 1] = l_tot;
      }
      return;
    }
  }
  if constexpr (SPLIT == kDivided) {
    // un-normalised partial O (relative to the reference m_run), fp32, plus (m_run, sum)
    const int64_t part_row = part_row_of();
    store_part32(o, p.part + (part_row - l32) * kHeadDim, p.C - m0, smem + rb * (17 * 1024));
    if (row < p.C && g == 0) {
      p.part_ml[2 * part_row] = m_run;
      p.part_ml[2 * part_row + 1] = l_tot;
    }
    return;
  }
  store_rows32([&](int db, int r) { return o[db][r]; },
               static_cast<__bf16*>(p.o_out) + b * p.os[0] + h * p.os[1], p.os[2], m0, p.C, smem + rb * (17 * 1024));
  if (row < p.C && g == 0) p.lse[((int64_t)b * p.Hq + h) * p.C + row] = (m_run + __log2f(l_tot)) * kLn2;
}

template <int SPLIT>
int launch_fwd8(const AttnParams& p, int n_mtiles, int total, hipStream_t s) {
  constexpr int smem = 4 * BNW * 2 * kRowBytes;
  auto kern = fwd8_bf16_kernel<SPLIT>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  {
    ProfScope prof(kKernelFwd, s);
    const int units = SPLIT == kWholeTiles ? p.B * p.Hkv : 8, first = SPLIT == kShares ? p.B * p.Hkv * p.rows_whole : 0;
    hipLaunchKernelGGL(kern, dim3(xcd_grid(first, units) + xcd_grid(total - first, units)), dim3(512), smem, s, for_launch(p, n_mtiles), n_mtiles, total);
  }
  return launch_status();
}

}  // namespace
}  // namespace seco
