// Forward of one chunk, bf16 matrix cores, 4-wavefront workgroups (Eq. 1 at the attention layer): the shape used
// when a call has two row tiles per CU or close to it (launch_fwd_bf16).  A workgroup owns 128 query rows of one head, a wavefront 32 of them;
// S^T = K Q^T so that a lane owns query rows; O^T += V^T P^T from registers.  K tiles stream through a ring of three LDS
// slots and V tiles through a ring of two, and S of tile n+1 is computed while the exponentials of tile n are taken (the
// two instruction streams are written interleaved), so that the matrix pipe runs while the vector ALU works: 5 %
// faster than computing a tile's S, softmax and PV one after the other.
//
// Bound: power.  With 32x32x16 products the matrix pipe was busy 63 % of the cycles at 1.68 GHz (long calls), and every
// schedule that kept it busier lowered the clock.  The 16x16x32 products used here take the same operands out of LDS, but
// half the accumulator traffic per operation: products alone run at 2.0 PFLOP/s against 1.75 within the same power
// (random operands, 0.2 s), with each operand out of LDS 1.6 against 1.5.  Here: 16384 rows 1934 -> 1860 us, 2048 rows at
// 30720 938 -> 922.  Operand reads are held two pairs of products ahead by scheduling barriers: left to the compiler they
// came one ahead and the kernel was 1 - 2 % slower; four ahead spill.
//
// With its order fixed so, a wavefront is nearly always ready to issue, and of the two on a SIMD the older one then gets
// all it can use: the two workgroups of a CU end one behind the other.  TURNS raises the priority over the scores and exponentials and
// lowers it over O, so that they alternate: two halves of the chip's power at a time as well (2048 rows at 15000 470 -> 455 us).
// turns_pay (seco_internal.h) says where.
//
// (A translation unit of its own, with a scheduler strategy of its own, see build.py: max-ilp; max-memory-clause 1 %
// slower, iterative-ilp 10 %.)
#include "mfma_tiles.h"
#include "seco_internal.h"

namespace seco {
namespace {

constexpr int BM = 128;  // query rows per workgroup
constexpr int BN = 64;   // cache rows per tile
constexpr float kBig = 1099511627776.f;   // 2^40: a tile's exponentials may sum to this before the reference moves

constexpr int kTileBytes = BN * kRowBytes;
constexpr int kKSlots = 3;
constexpr int kAhead = 2; // operand reads in flight ahead of the products

template <bool TURNS>
__global__ __launch_bounds__(256, 2) void fwd4_bf16_kernel(AttnParams p, int n_mtiles, int total_items) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];   // 5 * kTileBytes: K ring (3 tiles), V ring (2 tiles)
  lds_char* smem = (lds_char*)smem_raw;

  const int item = xcd_item(blockIdx.x, total_items, p.B * p.Hkv);
  if (item < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4, pg = pi4(g);
  // item -> (batch, kv head, row tile (heavy first), head within the group)
  const int tiles = over(item, p.by_G), hg = item - tiles * p.G, rest = over(tiles, p.by_tiles);
  const int mt = n_mtiles - 1 - (tiles - rest * n_mtiles);
  const int b = over(rest, p.by_Hkv), kvh = rest - b * p.Hkv, h = kvh * p.G + hg;
  const int m0 = mt * BM + wave * 32;          // first chunk-local row of this wavefront

  const int kv_len = p.q_start + p.C;
  const int qpos = p.q_start + m0 + l16;       // global position of this lane's first row; the second is 16 on
  bf16x8 qr[8];
  load_rows32(qr, static_cast<const __bf16*>(p.q) + b * p.qs[0] + h * p.qs[1], p.qs[2], m0, p.C - 1, lane);

  const __bf16* kbase = static_cast<const __bf16*>(p.k) + b * p.kvs[0] + kvh * p.kvs[1];
  const __bf16* vbase = static_cast<const __bf16*>(p.v) + b * p.kvs[0] + kvh * p.kvs[1];

  const int wg_kv_end = p.q_start + min((mt + 1) * BM, p.C);   // columns any row of the workgroup sees
  const int n_tiles = (wg_kv_end + BN - 1) / BN;
  const int wave_kv_end = m0 < p.C ? p.q_start + min(m0 + 32, p.C) : 0;  // columns this wavefront sees

  // K tiles stream through a ring of three LDS slots, V tiles through a ring of two: while the matrix pipe works on
  // S of tile n+1 (from K slot n+1) the vector ALU turns S of tile n into probabilities, and the product with V
  // of tile n follows; K of tile n+2 and V of tile n+1 are landing meanwhile.
  // Asynchronous global -> LDS copy of one tile: each wavefront copies 4 groups of 4 rows.  The per-lane byte
  // offsets inside a tile never change; a tile that lies entirely inside the cache is copied from a scalar base
  // address with no vector arithmetic, the last (ragged) one with clamped per-lane addresses.
  // (the four copies of a wavefront are 16 rows apart: the swizzle of a lane's chunk is the same in all four,
  // so one per-lane offset serves them and the row distance goes into the scalar base)
  const uint32_t lane_off = dma_lane_offset(4 * wave, p.kvs[2] * 2, lane);
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + wave * 4 * kRowBytes);
  lds_char* vring = smem + kKSlots * kTileBytes;
  auto copy_ring = [&](const __bf16* base, int n, int slot) {   // one tile of K (slots 0 ..) or V (kKSlots ..)
    if ((n + 1) * BN <= kv_len) {
      const __bf16* src = base + (int64_t)n * BN * p.kvs[2];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dma16_sbase(src + (int64_t)i * 16 * p.kvs[2], lane_off, lds_wave + slot * kTileBytes + i * (16 * kRowBytes));
    } else {
      lds_char* t = smem + slot * kTileBytes;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * (wave + 4 * i);
        const int64_t off = (int64_t)min(n * BN + r + (lane >> 4), kv_len - 1) * p.kvs[2];
        dma4rows(t, r, base + off, lane);
      }
    }
  };

  bf16x8 qf[8];                                // [row block][contraction step] (filled below, while the first tiles are on their way)
  f32x4 o[8][2];
#pragma unroll
  for (int db = 0; db < 8; ++db)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) o[db][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
  const float c = p.scale * kLog2e;

  // S^T of this wavefront's 64 cache rows of the K tile in slot ks, four blocks of 16 rows by two of 16 queries
  auto scores = [&](int ks, f32x4 (&sc)[4][2]) {
    lds_char* kt = smem + ks * kTileBytes;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      sc[rb][0] = sc[rb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bf16x8 a = lds_row16(kt, 16 * rb, t, lane);
        sc[rb][0] = mfma16(a, qf[t], sc[rb][0]);
        sc[rb][1] = mfma16(a, qf[4 + t], sc[rb][1]);
      }
    }
  };
  auto causal_mask = [&](int col0, f32x4 (&sc)[4][2]) {
    if (col0 + BN - 1 > p.q_start + m0) {  // reaches past this wavefront's first row
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (col0 + 16 * rb + 4 * pg + i > qpos + 16 * qb) sc[rb][qb][i] = -INFINITY;
    }
  };

  // One tile: `cur` holds S of tile n (slot ks of the K ring) on entry, `nxt` S of tile n+1 on exit.
  auto tile_body = [&](int n, int ks, int vs, f32x4 (&cur)[4][2], f32x4 (&nxt)[4][2]) {
    const int ks1 = ks + 1 == kKSlots ? 0 : ks + 1;
    if (n + 2 < n_tiles) copy_ring(kbase, n + 2, ks1 + 1 == kKSlots ? 0 : ks1 + 1);
    if (n + 1 < n_tiles) copy_ring(vbase, n + 1, kKSlots + (vs ^ 1));
    const int col0 = n * BN;                   // first cache row of the tile
    if (col0 < wave_kv_end) {
      lds_char* vt = vring + vs * kTileBytes;
      causal_mask(col0, cur);
      // Reference value of the row's exponentials.  A max subtraction only guards against overflow, so the
      // reference m_run is kept as it is as long as the exponentials stay representable: the (costly) row maximum
      // is computed only on a row's first visible tile and when the tile's sum of exponentials exceeds kBig = 2^40,
      // which for a whole kernel is a handful of times.  Exponentials may thus reach 2^40; bf16 and fp32 have
      // the exponent range for that, and O and the sum are rescaled together when the reference moves.
      auto tile_max = [&](int qb) {
        float mx = cur[0][qb][0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, cur[e >> 2][qb][e & 3]);
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        return fmaxf(mx, __shfl_xor(mx, 32)) * c;
      };
      auto move_reference = [&](int qb, float m_new) {  // m_new >= m_run; exp2(-inf - x) = 0 on the first tile
        const float alpha = fast_exp2(m_run[qb] - m_new);
        l_run[qb] *= alpha;
#pragma unroll
        for (int db = 0; db < 8; ++db) o[db][qb] *= alpha;
        m_run[qb] = m_new;
      };
      if (__builtin_amdgcn_ballot_w64(fminf(m_run[0], m_run[1]) == -INFINITY) != 0) {      // some row has seen nothing yet
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          const float m_blk = tile_max(qb);
          if (m_run[qb] == -INFINITY && m_blk != -INFINITY) m_run[qb] = m_blk;    // (o and l_run are still zero)
        }
      }
      // a part of a tile can be fully masked for a row (only when q_start is unaligned): such a row
      // has seen nothing yet and keeps m_run = -inf; use 0 so that exp2(-inf - (-inf)) never appears
      float m_use[2] = {m_run[0] == -INFINITY ? 0.f : m_run[0], m_run[1] == -INFINITY ? 0.f : m_run[1]};
      // S of the next tile is issued here, in the same straight-line code as the exponentials below, which do not
      // depend on it: the matrix pipe runs while the vector ALU works.  (On the last tile this computes on
      // whatever the slot holds; the result is never used.)
      float sum[2] = {0.f, 0.f};
      bf16x8 va[kAhead];
      if constexpr (TURNS) __builtin_amdgcn_s_setprio(1);
      {
        lds_char* kt1 = smem + ks1 * kTileBytes;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) nxt[rb][0] = nxt[rb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        // written interleaved: a pair of MFMAs of the next tile's chains, then two exponentials of this tile; operands are
        // read kAhead pairs ahead
        bf16x8 ka[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) ka[i] = lds_row16(kt1, 16 * (i & 3), i >> 2, lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int rb = i & 3, t = i >> 2;
          const bf16x8 a = ka[i % kAhead];
#pragma unroll
          for (int qb = 0; qb < 2; ++qb) {
            nxt[rb][qb] = mfma16(a, qf[4 * qb + t], nxt[rb][qb]);
            cur[i >> 2][qb][i & 3] = fast_exp2(__builtin_fmaf(cur[i >> 2][qb][i & 3], c, -m_use[qb]));
            sum[qb] += cur[i >> 2][qb][i & 3];
          }
          if (i + kAhead < 16) ka[i % kAhead] = lds_row16(kt1, 16 * ((i + kAhead) & 3), (i + kAhead) >> 2, lane);
          else va[i + kAhead - 16] = lds_tr16(vt, 0, i + kAhead - 16, lane);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (__builtin_amdgcn_ballot_w64(!(fmaxf(sum[0], sum[1]) <= kBig)) != 0) {           // reference too low for this tile (rare)
        scores(ks, cur);                                                // the scores again: K of this tile is still in its slot
        causal_mask(col0, cur);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          const float m_blk = tile_max(qb);
          if (m_blk > m_run[qb]) move_reference(qb, m_blk);
          m_use[qb] = m_run[qb] == -INFINITY ? 0.f : m_run[qb];
          sum[qb] = 0.f;
#pragma unroll
          for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              cur[rb][qb][i] = fast_exp2(__builtin_fmaf(cur[rb][qb][i], c, -m_use[qb]));
              sum[qb] += cur[rb][qb][i];
            }
        }
      }
      l_run[0] += sum[0];
      l_run[1] += sum[1];
      if constexpr (TURNS) __builtin_amdgcn_s_setprio(0);
      bf16x8 pb[2];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int kb = i >> 3, db = i & 7;
        if (db == 0) {
          pb[0] = pack44(cur[2 * kb][0], cur[2 * kb + 1][0]);
          pb[1] = pack44(cur[2 * kb][1], cur[2 * kb + 1][1]);
        }
        const bf16x8 a = va[i % kAhead];
        o[db][0] = mfma16(a, pb[0], o[db][0]);
        o[db][1] = mfma16(a, pb[1], o[db][1]);
        const int j = i + kAhead;
        if (j < 16) va[i % kAhead] = lds_tr16(vt, 32 * (j >> 3), j & 7, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    dma_wait_all();
    __syncthreads();
  };

  copy_ring(kbase, 0, 0);
  copy_ring(vbase, 0, kKSlots);
  if (1 < n_tiles) copy_ring(kbase, 1, 1);
  // (through the third K slot and the second V slot, which are empty until the loop)
  rows16_to_frags(qf, qr, smem + (wave < 2 ? 2 : 4) * kTileBytes + (wave & 1) * 8192, lane);
  settle8(qf);
  dma_wait_all();
  __syncthreads();

  f32x4 sa[4][2], sb[4][2];
  scores(0, sa);
  int ks = 0;
  for (int n = 0; n < n_tiles; n += 2) {       // two tiles per trip: the score registers swap roles
    tile_body(n, ks, 0, sa, sb);
    ks = ks + 1 == kKSlots ? 0 : ks + 1;
    if (n + 1 < n_tiles) {
      tile_body(n + 1, ks, 1, sb, sa);
      ks = ks + 1 == kKSlots ? 0 : ks + 1;
    }
  }

  float inv[2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    float l_tot = l_run[qb] + __shfl_xor(l_run[qb], 16);
    l_tot += __shfl_xor(l_tot, 32);
    inv[qb] = 1.f / l_tot;
    const int row = m0 + 16 * qb + l16;
    if (row < p.C && g == 0) p.lse[((int64_t)b * p.Hq + h) * p.C + row] = (m_run[qb] + __log2f(l_tot)) * kLn2;
  }
  store_rows16([&](int db, int qb, int i) { return o[db][qb][i] * inv[qb]; },
               static_cast<__bf16*>(p.o_out) + b * p.os[0] + h * p.os[1], p.os[2], m0, p.C, smem + wave * 8192);
}

template <bool TURNS>
int launch(const AttnParams& p, int n_mtiles, int total, hipStream_t s) {
  constexpr int smem = 5 * kTileBytes;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(fwd4_bf16_kernel<TURNS>), smem)) return SECO_ERR_LAUNCH;
  ProfScope prof(kKernelFwd, s);
  hipLaunchKernelGGL(fwd4_bf16_kernel<TURNS>, dim3(xcd_grid(total, p.B * p.Hkv)), dim3(256), smem, s, for_launch(p, n_mtiles), n_mtiles, total);
  return launch_status();
}

}  // namespace

int launch_fwd4_bf16(const AttnParams& p, int n_mtiles, int total, hipStream_t s) {
  return turns_pay(p, total) ? launch<true>(p, n_mtiles, total, s) : launch<false>(p, n_mtiles, total, s);
}

}  // namespace seco
