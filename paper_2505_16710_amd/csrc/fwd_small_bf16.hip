// Forward of a chunk with few query rows per KV head (C rows times the G query heads that share it) against a cache that is
// short for the workgroups there are: a few tokens at the end of a cache, short chunks at up to some thousand rows.
//
// What bounds it is reading the cache once, or, where that is short, the latency of one pass through memory: the row tiles
// of the other kernels would be mostly padding (a wavefront per head, four heads per workgroup, all on the same tile of
// the cache, one tile after the other).  Here the rows of a KV head, packed, are row tiles of 32, a workgroup holds one in
// every wavefront, and the wavefronts divide the cache: each takes blocks of 32 cache rows on its own, K and V copied into
// its own 16 KiB of LDS, no barrier in the loop.  Eight wavefronts keep 128 KiB in flight per CU.  Their sums meet in LDS; a
// long cache is divided among n_splits workgroups whose partial results fwd_merge_kernel combines: a quarter of what the
// 8-wavefront kernel's tiles of 128 packed rows write.
// Kernel times with the merge: 2 rows x 8 heads against 1101 cache rows 14.9 -> 10.0 us, 1 row x 32 heads (8 KV heads)
// against 600 / 8828 15.8 -> 8.9 / 16.7 -> 13.8 us; 8 rows x 32 heads against 32008 rows 30.7 -> 28.1 us (4.7 TB/s).
// Several row tiles, against the 8-wavefront kernel: 32 rows x 32 heads (8 KV heads) against 1032 / 4032 rows
// 12.8 -> 11.3 / 17.7 -> 13.9; 16 rows against 16368 20.9 -> 19.0; 64 against 2064 18.2 -> 14.7; 2 x 96 against 1096
// 18.9 -> 13.0.
#include <algorithm>

#include "mfma_tiles.h"
#include "seco_internal.h"

namespace seco {
namespace {

constexpr int kWaves = 8, kBlock = 32;
constexpr int kTurnStep = 1040;                          // bytes between the 64-lane groups of a turned tile (16 of padding)
constexpr int kOwn = 16 * kTurnStep;                     // a wavefront's LDS: K and V blocks, then its partial O
constexpr int kQTile = kWaves * kOwn, kMl = kQTile + 8192, kSmem = kMl + kWaves * 32 * 2 * 4;
static_assert(kOwn >= 2 * kBlock * kRowBytes && kOwn % 256 == 0, "a K and a V block");

__global__ __launch_bounds__(kWaves * 64, 2) void fwd_small_bf16_kernel(AttnParams p, int n_mtiles, int total_items) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds_char* smem = (lds_char*)smem_raw;
  const int item = xcd_item(blockIdx.x, total_items);
  if (item < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  // item -> (batch, kv head), share of the cache, row tile: the tiles that read the same rows run side by side on one XCD
  const int shared = over(item, p.by_tiles), r0 = (item - shared * n_mtiles) * 32;
  const int unit = over(shared, p.by_splits), sp = shared - unit * p.n_splits, b = over(unit, p.by_Hkv), kvh = unit - b * p.Hkv;
  const int n_rows = p.G * p.C, kv_len = p.q_start + p.C;
  const __bf16* kbase = static_cast<const __bf16*>(p.k) + b * p.kvs[0] + kvh * p.kvs[1];
  const __bf16* vbase = static_cast<const __bf16*>(p.v) + b * p.kvs[0] + kvh * p.kvs[1];
  // blocks of this workgroup: [first, last), dealt to the wavefronts in turn
  const int n_blocks = (kv_len + kBlock - 1) / kBlock, per = over(n_blocks + p.n_splits - 1, p.by_splits);
  const int first = sp * per, last = min(n_blocks, first + per);
  lds_char* kt = smem + wave * kOwn;
  lds_char* vt = kt + kBlock * kRowBytes;
  uint32_t lane_off[4];                                  // of rows 4 i .. 4 i + 3, by i % 4 (the chunk's XOR), without 4 i rows
#pragma unroll
  for (int i = 0; i < 4; ++i)
    lane_off[i] = (uint32_t)((lane >> 4) * (p.kvs[2] * 2)) + (uint32_t)(((lane & 15) ^ swz(4 * i + (lane >> 4))) << 4);
  // eight copies of four rows each: one block of K (dst kt) or V (dst vt)
  auto copy_block = [&](const __bf16* base, lds_char* dst, int blk) {
    const uint32_t d = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
    if ((blk + 1) * kBlock <= kv_len) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        dma16_sbase(base + (int64_t)(blk * kBlock + 4 * i) * p.kvs[2], lane_off[i & 3], d + i * 4 * kRowBytes);
    } else {                                   // rows past the cache's end repeat its last one
      const __bf16* first_row = base + (int64_t)(blk * kBlock) * p.kvs[2];
#pragma unroll
      for (int i = 0; i < 8; ++i) {            // (4 i rows on less those past the end: not negative, lane_off being that of lane / 16 rows)
        const int back = max(4 * i + (lane >> 4) + blk * kBlock - (kv_len - 1), 0);
        dma16_sbase(first_row, lane_off[i & 3] + __umul24(4 * i, (uint32_t)p.kvs[2] * 2u) - __umul24(back, (uint32_t)p.kvs[2] * 2u), d + i * 4 * kRowBytes);
      }
    }
  };
  // packed row r: head r / C of the group, chunk row r % C; rows past the last repeat it and are not stored
  {
    const int r = min(r0 + 4 * wave + (lane >> 4), n_rows - 1), hg = over(r, p.by_C);
    dma4rows(smem + kQTile, 4 * wave, static_cast<const __bf16*>(p.q) + b * p.qs[0] + (kvh * p.G + hg) * p.qs[1] +
                                          (int64_t)(r - hg * p.C) * p.qs[2], lane);
  }
  int blk = first + wave;
  if (blk < last) {
    copy_block(kbase, kt, blk);
    copy_block(vbase, vt, blk);
  }
  const int my_row = min(r0 + l32, n_rows - 1), qpos = p.q_start + my_row - over(my_row, p.by_C) * p.C;
  const float c = p.scale * kLog2e;
  f32x16 o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m = -INFINITY, l = 0.f;
  dma_wait_all();
  __syncthreads();
  bf16x8 qf[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) qf[t] = lds_row8(smem + kQTile, l32, 2 * t + g);

  for (; blk < last; blk += kWaves) {
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) s = mfma(lds_row8(kt, l32, 2 * t + g), qf[t], s);
    // The next block's K goes into the place of this one's as soon as its rows have been read, its V behind the second
    // product: copies land in order, so "at most 8 outstanding" means that the older of the two has arrived.
    const bool more = blk + kWaves < last;
    if (more) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      copy_block(kbase, kt, blk + kWaves);
    }
    const int col0 = blk * kBlock;
    if (col0 + kBlock - 1 > p.q_start) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (col0 + 8 * (r >> 2) + 4 * g + (r & 3) > qpos) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32)) * c);
    const float ref = mx == -INFINITY ? 0.f : mx;                   // a row that has seen nothing yet
    if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
      const float alpha = fast_exp2(m - ref);
      l *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      m = mx;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = fast_exp2(__builtin_fmaf(s[r], c, -ref));
      l += s[r];
    }
    if (more)
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");              // V of this block
    else
      dma_wait_all();
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const bf16x8 pb = pack8(s, t);
#pragma unroll
      for (int db = 0; db < 4; ++db) o[db] = mfma(lds_tr8(vt, 16 * t, db, lane), pb, o[db]);
    }
    if (more) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      copy_block(vbase, vt, blk + kWaves);
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");              // K of the next block
    }
  }
  l += __shfl_xor(l, 32);

  // the wavefronts' sums, relative to their common reference
  SECO_LDS float* ml = reinterpret_cast<SECO_LDS float*>(smem + kMl);
  if (g == 0) {
    ml[2 * (wave * 32 + l32)] = m;
    ml[2 * (wave * 32 + l32) + 1] = l;
  }
  __syncthreads();
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) M = fmaxf(M, ml[2 * (w * 32 + l32)]);
  const float a = M == -INFINITY ? 0.f : fast_exp2(m - M);
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const f32x4 v = {o[db][4 * r4] * a, o[db][4 * r4 + 1] * a, o[db][4 * r4 + 2] * a, o[db][4 * r4 + 3] * a};
      *reinterpret_cast<SECO_LDS f32x4*>(kt + (4 * db + r4) * kTurnStep + lane * 16) = v;
    }
  __syncthreads();
  // thread: four consecutive head_dim elements of rows tid / 32 and tid / 32 + 16
  const int q = tid & 31;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int r = (tid >> 5) + 16 * k;
    if (r0 + r >= n_rows) break;
    float rm = -INFINITY, rl = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) rm = fmaxf(rm, ml[2 * (w * 32 + r)]);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float mw = ml[2 * (w * 32 + r)];
      rl += mw == -INFINITY ? 0.f : ml[2 * (w * 32 + r) + 1] * fast_exp2(mw - rm);
    }
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
      sum += *reinterpret_cast<SECO_LDS f32x4*>(smem + w * kOwn + (q >> 1) * kTurnStep + ((q & 1) * 32 + r) * 16);
    const int hg = over(r0 + r, p.by_C), row = r0 + r - hg * p.C, h = kvh * p.G + hg;
    const int64_t rowid = ((int64_t)b * p.Hq + h) * p.C + row;
    if (p.n_splits > 1) {
      const int64_t part_row = (int64_t)sp * p.B * p.Hq * p.C + rowid;
      *reinterpret_cast<f32x4*>(p.part + part_row * kHeadDim + 4 * q) = sum;
      if (q == 0) {
        p.part_ml[2 * part_row] = rm;
        p.part_ml[2 * part_row + 1] = rl;
      }
    } else {
      const float inv = 1.f / rl;
      const bf16x4 v = {(__bf16)(sum[0] * inv), (__bf16)(sum[1] * inv), (__bf16)(sum[2] * inv), (__bf16)(sum[3] * inv)};
      *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.o_out) + b * p.os[0] + h * p.os[1] + (int64_t)row * p.os[2] + 4 * q) = v;
      if (q == 0) p.lse[rowid] = (rm + __log2f(rl)) * kLn2;
    }
  }
}

}  // namespace

namespace {
// Rounds of eight blocks, one per wavefront; divided where that pays (small_divides).  At most one workgroup per CU.
struct SmallPlan { int n_mtiles, n_splits, rounds; };      // rounds: of a workgroup
SmallPlan small_plan(const AttnParams& p, int max_splits) {
  SmallPlan sp;
  sp.n_mtiles = (p.G * p.C + 31) / 32;
  const int units = p.B * p.Hkv * sp.n_mtiles, all = ((p.q_start + p.C + kBlock - 1) / kBlock + kWaves - 1) / kWaves;
  int n = std::min(std::max(device_cus() / units, 1), max_splits);
  const int each = (all + n - 1) / n;
  n = (all + each - 1) / each;
  sp.n_splits = small_divides(p.B * p.Hkv, all - each) ? n : 1;
  sp.rounds = sp.n_splits > 1 ? each : all;
  return sp;
}
}  // namespace

// The rounds tell the two kernels apart where the rows are more than one tile: here a workgroup's wavefronts share nothing
// and a round is 256 cache rows for 32 query rows; the 8-wavefront kernel does 128 x 128 in the same time but starts, ends
// and merges slower.  204 shapes of 48 - 800 packed rows at 300 - 30000, times there over times here: 1 - 6 rounds 1.01 - 1.55
// (but for 0.98 and 0.99), 7 rounds 0.98 - 1.11, 8 0.89 - 1.03, 12 and more 0.71 - 1.03; with at most 64 rows, where both read the
// cache at the memory's rate, 0.99 - 1.03 at 8.
bool fwd_small_pays(const AttnParams& p, int max_splits) {
  const int rows = p.G * p.C;
  if (rows <= 32) return true;
  if ((int64_t)p.B * p.Hkv * ((rows + 31) / 32) > device_cus()) return false;
  return small_plan(p, max_splits).rounds <= (rows <= 64 ? 8 : 6);
}

int launch_fwd_small_bf16(AttnParams p, int max_splits, hipStream_t s) {
  const SmallPlan sp = small_plan(p, max_splits);
  const int n_mtiles = sp.n_mtiles, total = p.B * p.Hkv * n_mtiles * sp.n_splits;
  p.n_splits = sp.n_splits;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(fwd_small_bf16_kernel), kSmem)) return SECO_ERR_LAUNCH;
  {
    ProfScope prof(kKernelFwd, s);
    hipLaunchKernelGGL(fwd_small_bf16_kernel, dim3(xcd_grid(total)), dim3(kWaves * 64), kSmem, s, for_launch(p, n_mtiles), n_mtiles, total);
  }
  const int rc = launch_status();
  return rc || p.n_splits == 1 ? rc : launch_fwd_merge(p, s);
}

}  // namespace seco
