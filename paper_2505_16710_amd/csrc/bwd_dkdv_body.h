// dK/dV of one chunk, bf16 matrix cores, accumulated into the persistent fp32 KV-gradient
// buffers (Alg. 1 second loop; Alg. 2 with per-chunk weights):
//   gV[c] += w * sum_{heads of the group} P^T dO      gK[c] += w * s * sum_{heads} dS^T Q
//
// Column-parallel: one workgroup is the only writer of 128 cache rows of one (batch, KV head),
// so the read-modify-write of gK/gV needs no atomics and the result is deterministic.
//
// The workgroup has 8 wavefronts: 4 column blocks of 32 cache rows x 2 roles.
//   role A ("probabilities"): keeps K^T fragments and the dV accumulator; computes
//          S = Q K^T, P = exp(s S - LSE) (causal mask applied), hands P (bf16) to its partner
//          through LDS and accumulates dV += P^T dO;
//   role B ("score gradient"): keeps V^T fragments and the dK accumulator; computes
//          dP = dO V^T, dS = P * (dP - delta) and accumulates dK += dS^T Q.
// Each of the four products is computed exactly once, and a wavefront holds one 32x128 fp32
// accumulator plus one operand fragment set instead of two of each, which is what lets two
// wavefronts share a SIMD.  Role A runs one row tile ahead of role B, so the P hand-over
// costs no extra barrier: one barrier per 64-row stage.
//
// The two roles are two instantiations of one body (template parameter ROLE) behind a wavefront-uniform branch at
// the top of the kernel, not two arms of a branch inside a common loop: each role then has a loop, accumulators and
// a register allocation of its own (224 instead of 256 registers, no execution-mask juggling; 7 % faster).
//
// Q, dO, -LSE / s and -delta of one stage of query rows stream through a three-deep ring of swizzled LDS
// slots, laid out region by region (Q tiles, dO tiles, row statistics, P buffers; one of each per slot)
// (A reads Q of stage i+1 while B reads Q and dO of stage i and stage i+2 is landing);
// Q and dO are copied global -> LDS directly (no staging registers), issued two stages ahead (after the first
// MFMA chain of an iteration, so that the matrix pipe starts right behind the barrier).
// S and dP are computed in the "row = query" orientation, so P and dS sit in the C layout
// with lane = cache row and feed the second products as A operands; dO and Q for those
// products come through the LDS transpose read.  P is written to LDS once (bf16, in operand
// order) for role B; role A keeps its own copy in registers for the dV product of the next iteration.
// Inside an iteration every wavefront runs four MFMA chains; the LDS operands of a chain are requested while
// the chain before it runs (across the barrier too), and the exponentials / dS products of a row block are
// written between the MFMAs of a later chain.
//
// Column tiles are enumerated from a by-value segment table (runs of cache rows that share
// one non-zero weight); SpaCO's unselected chunks simply have no tiles.
//
// A workgroup occupies a whole CU, so a launch runs in rounds of 256 column tiles and a last round with few
// tiles costs as much as a full one.  The last column tiles of every (batch, KV head) are therefore shared out
// where that is expected to pay (share_plan in seco_internal.h): a share is a run of the tile's iterations (64 query rows
// of one head each, or of several heads: kJoined; cut through heads where the number of shares asks for it), its fp32 sums go to the workspace, and
// a merge adds them to gK/gV in the order of the shares (still one writer per element and a fixed summation order, so
// results stay reproducible).
//
// The same kernel serves the transposed order of the backward pass (seco_chunk_attn_bwd_gather): there the column
// run is one chunk and the query rows are that chunk's and every later one's, p.C of them from p.q_start on, with
// -delta and -LSE read from arrays kept for the whole sequence (stat_stride, stat_off).  With ROWS the rows come as
// runs with one weight each (Alg. 2 in that order): rows outside the runs are never read, and a run's weight
// enters as log2 w added to -LSE, i.e. as a factor on P and through it on dV and dS alike.
#pragma once
#include "mfma_tiles.h"
#include "seco_internal.h"

#ifndef SECO_DKDV_RB
#define SECO_DKDV_RB 2
#endif

namespace seco {
namespace {

constexpr int kPBytes = 2048;   // one 32x32 bf16 P tile
constexpr int kStages = 3;

// NCB: 32-row column blocks per workgroup (2 wavefronts each); RB: 32-row query blocks per stage
template <int NCB, int RB>
struct DkdvCfg {
  static constexpr int kThreads = NCB * 128;
  static constexpr int kBQ = 32 * RB;                                   // query rows per stage
  static constexpr int kTileBytes = kBQ * kRowBytes;
  // LDS layout, region by region: the Q tiles of the kStages slots, their dO tiles, their row statistics (-LSE / s
  // and -delta, kBQ floats each), and one P buffer per slot, column block and row block.  A per-lane operand
  // offset carries the region it is used with (role A reads rows of Q and transposed blocks of dO, role B the
  // reverse), so that a slot's tile base is one scalar for both tiles.
  static constexpr int kDoRegion = kStages * kTileBytes;
  static constexpr int kStatRegion = 2 * kStages * kTileBytes;
  static constexpr int kStatBytes = 2 * kBQ * 4;
  static constexpr int kPRegion = kStatRegion + kStages * kStatBytes;
  static constexpr int kSmemBytes = kPRegion + kStages * NCB * RB * kPBytes;
  static constexpr int kCols = NCB * 32;                                // cache rows per workgroup
};

// The products of a wavefront, in either shape of the matrix instructions: a chain is eight steps, each with one 16-byte
// operand from LDS, and gives a row block's 32 x 32 scores (or dP); a sum is eight steps too and adds a row block to the
// 32 x 128 accumulator.  Element e of a lane's sixteen scores is element e % 8 of operand half e / 8 of the second product,
// and belongs to query row row_of(e) + lane_row and cache row col_of(e) + lane_col of the block.
//
// 16x16x32, for whole launches of this pass: they are bound by power, and these take half the accumulator traffic per
// operation (2048 rows at 30720 of 32/8 heads 1949 -> 1841 us, 1024 at 15360 503 -> 477; the order of each step is fixed by a
// scheduling barrier, without which 1868 and 485).
struct Products16 {
  using Tile = f32x4[2][2];              // [16 query rows][16 cache rows]
  using Init = f32x4[2];
  using Acc = f32x4[8][2];
  int r_off[4], t_off[8], lane_row, lane_col;
  __device__ __forceinline__ Products16(int lane, int r_region, int t_region) {
    lane_col = lane & 15;
    lane_row = 4 * pi4(lane >> 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) r_off[t] = row16_lane_off(t, lane) + r_region;
#pragma unroll
    for (int db = 0; db < 8; ++db) t_off[db] = tr16_lane_off(db, lane) + t_region;
  }
  static __device__ __forceinline__ int row_of(int e) { return 16 * ((e >> 2) & 1) + (e & 3); }
  static __device__ __forceinline__ int col_of(int e) { return 16 * (e >> 3); }
  static __device__ __forceinline__ void frags(bf16x8 (&f)[8], const bf16x8 (&x)[8], lds_char* own, int lane) { rows16_to_frags(f, x, own, lane); }
  // operand i of a row block's chain (row0: the block's first row), and of its sum
  __device__ __forceinline__ bf16x8 row_op(lds_char* tile, int row0, int i) const { return lds_at(tile + r_off[i >> 1], row0 + 16 * (i & 1)); }
  __device__ __forceinline__ bf16x8 col_op(lds_char* tile, int row0, int i) const { return lds_tr16_at(tile + t_off[i], row0); }
  // what a chain starts from: the statistic of the lane's query rows
  __device__ __forceinline__ void chain_init(Init& x, SECO_LDS float* stat) const {
#pragma unroll
    for (int r = 0; r < 2; ++r) x[r] = *reinterpret_cast<SECO_LDS f32x4*>(stat + 16 * r + lane_row);
  }
  static __device__ __forceinline__ void add(Init& x, float v) {
    x[0] += v;
    x[1] += v;
  }
  static __device__ __forceinline__ void chain(Tile& x, int i, bf16x8 a, const bf16x8 (&frag)[8], const Init& init) {
#pragma unroll
    for (int c = 0; c < 2; ++c) x[i & 1][c] = mfma16(a, frag[4 * c + (i >> 1)], i < 2 ? init[i & 1] : x[i & 1][c]);
  }
  static __device__ __forceinline__ void sum(Acc& acc, int i, const bf16x8 (&pr)[2], bf16x8 b) {
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[i][c] = mfma16(pr[c], b, acc[i][c]);
  }
  template <typename F>
  static __device__ __forceinline__ void map(Tile& x, int e, const F& f) { x[(e >> 2) & 1][e >> 3][e & 3] = f(x[(e >> 2) & 1][e >> 3][e & 3]); }
  static __device__ __forceinline__ bf16x8 pack(const Tile& x, int half) { return pack44(x[0][half], x[1][half]); }
  static __device__ __forceinline__ void step_end() { __builtin_amdgcn_sched_barrier(0); }
  // (lgkmcnt(0): or the compiler waits for the operands that come with the loop in every iteration)
  static __device__ __forceinline__ void loop_begins() { __builtin_amdgcn_s_waitcnt(0xc07f); }
  static __device__ __forceinline__ void clear(Acc& acc) {
#pragma unroll
    for (int db = 0; db < 8; ++db) acc[db][0] = acc[db][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // put(row of the wavefront's 32, column, value)
  template <typename F>
  static __device__ __forceinline__ void each(const Acc& acc, int lane, const F& put) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int db = 0; db < 8; ++db) put(16 * c + 4 * (lane >> 4) + i, 16 * db + (lane & 15), acc[db][c][i]);
  }
};
// 32x32x16, for the short launches that hold dQ as well: a workgroup's few iterations wait for latencies, not for power, and
// vector instructions cost less beside these (probe, cycles per 32 of the matrix pipe with 4 multiply-adds and an
// exponential: 39 against 47): 512 rows at 3584 of 8/2 heads 47.5 us against 50.2, 512 at 0 of 32/8 30.0 against 31.0.  A
// call whose passes could share a launch but for what its outputs lie over takes them too: the same bits of gK and gV.
struct Products32 {
  using Tile = f32x16;
  using Init = f32x16;
  using Acc = f32x16[4];
  int r_off[8], lane_row, lane_col;
  TrOff t_off[4];
  __device__ __forceinline__ Products32(int lane, int r_region, int t_region) {
    lane_col = lane & 31;
    lane_row = 4 * (lane >> 5);
#pragma unroll
    for (int t = 0; t < 8; ++t) r_off[t] = row8_lane_off(lane & 31, 2 * t + (lane >> 5)) + r_region;
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      t_off[db] = tr8_lane_off(db, lane);
      t_off[db].lo += t_region;
      t_off[db].hi += t_region;
    }
  }
  static __device__ __forceinline__ int row_of(int e) { return 8 * (e >> 2) + (e & 3); }
  static __device__ __forceinline__ int col_of(int) { return 0; }
  static __device__ __forceinline__ void frags(bf16x8 (&f)[8], const bf16x8 (&x)[8], lds_char* own, int lane) { rows32_to_frags(f, x, own, lane); }
  __device__ __forceinline__ bf16x8 row_op(lds_char* tile, int row0, int i) const { return lds_at(tile + r_off[i], row0); }
  __device__ __forceinline__ bf16x8 col_op(lds_char* tile, int row0, int i) const { return lds_tr8_at(tile, t_off[i & 3], row0 + 16 * (i >> 2)); }
  __device__ __forceinline__ void chain_init(Init& x, SECO_LDS float* stat) const {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = stat[row_of(r) + lane_row];
  }
  static __device__ __forceinline__ void add(Init& x, float v) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] += v;
  }
  static __device__ __forceinline__ void chain(Tile& x, int i, bf16x8 a, const bf16x8 (&frag)[8], const Init& init) { x = mfma(a, frag[i], i == 0 ? init : x); }
  static __device__ __forceinline__ void sum(Acc& acc, int i, const bf16x8 (&pr)[2], bf16x8 b) { acc[i & 3] = mfma(pr[i >> 2], b, acc[i & 3]); }
  template <typename F>
  static __device__ __forceinline__ void map(Tile& x, int e, const F& f) { x[e] = f(x[e]); }
  static __device__ __forceinline__ bf16x8 pack(const Tile& x, int half) { return pack8(x, half); }
  static __device__ __forceinline__ void step_end() {}
  static __device__ __forceinline__ void loop_begins() {}
  static __device__ __forceinline__ void clear(Acc& acc) {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
  }
  template <typename F>
  static __device__ __forceinline__ void each(const Acc& acc, int lane, const F& put) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int db = 0; db < 4; ++db) put(row_of(r) + 4 * (lane >> 5), 32 * db + (lane & 31), acc[db][r]);
  }
};

// (RB is fixed to 2 by the hand-pipelined main loop.)
// MODE: kAll: the query rows are all p.C rows of each head with weight 1, a head's in stages of its own.
// kRuns: they are taken from a table of runs (rows relative to p.q_start, each run with one weight whose
// log2 is added to -LSE, i.e. its probabilities are scaled by the weight).
// kJoined: as kAll, but the stages cut the rows of all heads of the group one behind the other, so that only the last stage of all
// has rows that do not exist: 32 rows of 4 heads are two iterations instead of four half empty ones, 70 are five instead of eight.
// A stage with rows of several heads takes its addresses per lane and, on the diagonal, a position per row (joined_pays).
// ROLE: 0 = role A, 1 = role B.  The body of a wavefront is instantiated once per role, so that a role's accumulators
// and working set are the variables of a loop of its own: with both roles as the two arms of a branch inside one
// loop, unrolled over the ring slots, the register allocator could not keep the working set in registers.
// OWN: the row statistics (-LSE / s and -delta) are computed here, from the O and dO rows of each stage, instead of being
// taken from the arrays the dQ kernel leaves: for the launch that runs both passes at once.
template <int NCB, int RB, Rows MODE, int ROLE, class Products, bool OWN = false>
__device__ __forceinline__ void dkdv_bf16_body(const AttnParams& p, const SegTable& seg, const TailSplit& ts,
                                               const RowRuns& rr, int item, lds_char* smem) {
  using Cfg = DkdvCfg<NCB, RB>;
  constexpr bool ROWS = MODE == kRuns, JOINED = MODE == kJoined;
  constexpr int BQ = Cfg::kBQ, kTileBytes = Cfg::kTileBytes;
  constexpr int kDoRegion = Cfg::kDoRegion, kStatRegion = Cfg::kStatRegion, kStatBytes = Cfg::kStatBytes;
  constexpr int NW = 2 * NCB;                 // wavefronts
  constexpr int kCopies = (BQ / 4) / NW;      // 4-row direct copies of Q (and of dO) per wavefront and stage
  static_assert((BQ / 4) % NW == 0, "stage rows must split evenly over the wavefronts");
  lds_char* pbuf = smem + Cfg::kPRegion;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int role = ROLE;
  const int cb = wave % NCB;
  // item -> (batch, kv head, column tile, share of the tile's iterations); the listed tiles come last in a unit
  const int n_whole = p.n_ctiles - ts.plan.n_tiles;
  // (in long launches of its own the kernel is 0.5 - 1 % faster behind plain divisions: it is bound by power, and with another
  // prologue the loop's registers come out otherwise)
  const int per_unit = n_whole + ts.plan.n_entries;
  const int unit = OWN ? over(item, p.by_unit) : item / per_unit, in_unit = item - unit * per_unit;
  int tile = in_unit, share = 0, n_shares = 1;
  if (in_unit >= n_whole) {
    // (whole words of the tables: there are no scalar loads of less, and through vector loads, one behind the other, this takes 0.5 us)
    typedef uint32_t __attribute__((may_alias)) word;
    const int entry = in_unit - n_whole;
    const int pos = *reinterpret_cast<const word*>(ts.plan.tile_of + (entry & ~3)) >> (8 * (entry & 3)) & 0xff;
    const word* first = reinterpret_cast<const word*>(ts.plan.first + (pos & ~1));
    uint32_t lo = first[0], hi = first[1];
    asm("" : "+s"(lo), "+s"(hi));                  // (or the compiler makes loads of half a word of them)
    const int begin = pos & 1 ? lo >> 16 : lo & 0xffff;
    tile = n_whole + pos;
    share = entry - begin;
    n_shares = (int)(pos & 1 ? hi & 0xffff : lo >> 16) - begin;
  }
  const bool divided = n_shares > 1;
  const int b = over(unit, p.by_Hkv), kvh = unit - b * p.Hkv;
  int si = 0;
  while (si + 1 < seg.n && tile >= seg.tile_begin[si + 1]) ++si;
  const int c0 = seg.col_begin[si] + (tile - seg.tile_begin[si]) * Cfg::kCols;
  const int c_end = min(c0 + Cfg::kCols, seg.col_end[si]);
  const float weight = seg.weight[si];

  const int kv_len = p.q_start + p.C;
  const int n0 = c0 + cb * 32;     // first cache row of this wavefront
  // role A holds K^T fragments, role B holds V^T fragments
  bf16x8 frag[8], fr[8];
  load_rows32(fr, static_cast<const __bf16*>(role == 0 ? p.k : p.v) + b * p.kvs[0] + kvh * p.kvs[1], p.kvs[2], n0, kv_len - 1, lane);
  // Role A starts its MFMA chains from -LSE / s instead of zero, so that a chain delivers q.k - LSE / s and
  // P = exp2(c * that) with c = s * log2(e): one multiply per score, in fp32.  (Folding c into the K^T fragments
  // would save that multiply but round K a second time, to bf16: with scores far from zero, as with the outlier
  // components of trained models, P = exp(S - LSE) hangs on the low-order bits of S, and the extra rounding showed
  // as errors of several per cent in gV and gK.)  Role B starts its chains from -delta.
  const float c2 = p.scale * kLog2e;

  // query-row stages that see at least one cache row of this workgroup; iteration = (head of the group, stage)
  const int rt0 = max(0, c0 - p.q_start) / BQ;
  struct Pos { int hg, r0, ri; };   // head within the group, first chunk-local row of the stage, run of rows
  // first stage of a head, and the number of stages per head
  int first_ri = 0, first_r0 = rt0 * BQ, n_rt = 0;
  // (joined) rows of a head; r0 of a stage counts from first_r0 on.  One stage on: heads and rows, and another head where its rows end
  const int len = p.C - first_r0;
  int adv_h = 0, adv_r = BQ;
  float inv_len = 0.f;
  if constexpr (ROWS) {
    while (first_ri + 1 < rr.n && rr.end[first_ri] <= first_r0) ++first_ri;
    first_r0 = max(first_r0, rr.begin[first_ri]);
    n_rt = (rr.end[first_ri] - first_r0 + BQ - 1) / BQ;
    for (int i = first_ri + 1; i < rr.n; ++i) n_rt += (rr.end[i] - rr.begin[i] + BQ - 1) / BQ;
    n_rt = max(n_rt, 0);
  } else if constexpr (JOINED) {
    if (len < BQ) {                           // (quotients below 128 by the reciprocal, half added to the dividend: exact)
      inv_len = __builtin_amdgcn_rcpf((float)len);
      adv_h = (int)((BQ + 0.5f) * inv_len);
      adv_r = BQ - adv_h * len;
    }
  } else {
    n_rt = (p.C + BQ - 1) / BQ - rt0;
  }
  // this workgroup's share of the tile's iterations: [it0, it0 + n_iter)
  const int n_all = JOINED ? (len * p.G + BQ - 1) / BQ : n_rt * p.G;
  int it0 = 0, n_iter = n_all;
  if (divided) {
    // share i begins at floor(i n_all / n_shares) = i each + floor(i rest / n_shares), i and rest less than 2^9: a product with the
    // reciprocal is exact, half added (two 64-bit divisions are 300 instructions)
    const int each = n_all / n_shares, rest = n_all - each * n_shares;
    const float inv = __builtin_amdgcn_rcpf((float)n_shares);
    auto begin = [&](int i) { return i * each + (int)(((float)(i * rest) + 0.5f) * inv); };
    it0 = begin(share);
    n_iter = begin(share + 1) - it0;
  }
  // rows [x.r0, row_limit(x)) of a stage exist; the others are masked
  auto row_limit = [&](Pos x) { return ROWS ? rr.end[x.ri] : JOINED ? len : p.C; };
  auto inside = [&](Pos x) { return x.r0 + BQ <= row_limit(x); };        // (joined: of one head)
  // (joined) how many rows there are from the stage's first on, and where its row lr is: `rows` further and `heads` times from the end
  // of one head's rows to the start of the next one's; rows that do not exist repeat the last one
  auto rows_left = [&](Pos x) { return (p.G - x.hg) * len - x.r0; };
  auto heads_in = [&](int local) { return len < BQ ? (int)(((float)local + 0.5f) * inv_len) : (local >= len ? 1 : 0); };
  struct At { int rows, heads; };
  auto row_at = [&](Pos x, int lr) {
    if (inside(x)) return At{lr, 0};
    const int rows = min(lr, rows_left(x) - 1);
    return At{rows, heads_in(x.r0 + rows)};
  };
  auto advance = [&](Pos x) {
    x.r0 += JOINED ? adv_r : BQ;
    if constexpr (ROWS) {
      if (x.r0 >= rr.end[x.ri]) {
        if (++x.ri == rr.n) { x.ri = first_ri; x.r0 = first_r0; x.hg += 1; }
        else x.r0 = rr.begin[x.ri];
      }
    } else if constexpr (JOINED) {
      x.hg += adv_h;
      if (x.r0 >= len) { x.r0 -= len; x.hg += 1; }
    } else {
      if (x.r0 >= p.C) { x.r0 = first_r0; x.hg += 1; }
    }
    return x;
  };

  const __bf16* qbase = static_cast<const __bf16*>(p.q) + b * p.qs[0] + (int64_t)kvh * p.G * p.qs[1];
  const __bf16* dobase = static_cast<const __bf16*>(p.d_o) + b * p.os[0] + (int64_t)kvh * p.G * p.os[1];
  const int64_t stat_base = ((int64_t)b * p.Hq + (int64_t)kvh * p.G) * p.stat_stride + p.stat_off;
  // asynchronous global -> LDS copy of the Q and dO tiles of one stage (4 rows per wavefront and copy).  A stage
  // that lies entirely inside the chunk is copied from scalar base addresses with constant per-lane offsets (no
  // vector arithmetic); the last, ragged one uses clamped per-lane addresses.
  uint32_t q_lane_off[kCopies], do_lane_off[kCopies];
#pragma unroll
  for (int i = 0; i < kCopies; ++i) {
    q_lane_off[i] = dma_lane_offset(4 * (wave + NW * i), p.qs[2] * 2, lane);
    do_lane_off[i] = dma_lane_offset(4 * (wave + NW * i), p.os[2] * 2, lane);
  }
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + wave * 4 * kRowBytes);
  // Global addresses of a stage's first row (Q, dO, and the row statistic this wavefront copies).  They are carried
  // along with the stage two ahead and advanced by one stage's worth per iteration: computing them from (head, row)
  // costs a dozen 64-bit scalar multiplies per iteration and wavefront.
  struct Src { const __bf16* q; const __bf16* d_o; const float* stat; };
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto src_of = [&](Pos x) {
    Src r;
    const int row = JOINED ? x.r0 + first_r0 : x.r0;
    r.q = qbase + x.hg * p.qs[1] + (int64_t)row * p.qs[2];
    r.d_o = dobase + x.hg * p.os[1] + (int64_t)row * p.os[2];
    r.stat = OWN ? p.lse + ((int64_t)b * p.Hq + (int64_t)kvh * p.G + x.hg) * p.C + row
                 : (wave_u == 0 ? p.nlse2 : p.delta) + stat_base + (int64_t)x.hg * p.stat_stride + row;
    return r;
  };
  // (all rows, no runs) one stage on: BQ rows further, or, behind a head's last stage, back to the first stage's row
  // of the next head
  const int64_t q_step = (int64_t)BQ * p.qs[2], do_step = (int64_t)BQ * p.os[2];
  const int64_t back_rows = (int64_t)(n_rt - 1) * BQ;
  const int64_t q_wrap = p.qs[1] - back_rows * p.qs[2], do_wrap = p.os[1] - back_rows * p.os[2];
  const int64_t stat_wrap = (OWN ? p.C : p.stat_stride) - back_rows;
  auto stat_step = [&](Pos from, Pos to) {
    if constexpr (JOINED) return (int64_t)((to.hg - from.hg) * p.C + to.r0 - from.r0);          // (asked with OWN only)
    return to.hg != from.hg ? stat_wrap : (int64_t)BQ;
  };
  auto next_src = [&](Src x, Pos from, Pos to) {
    if constexpr (ROWS || JOINED) {
      x = src_of(to);
    } else {
      const bool wrap = to.hg != from.hg;
      x.q += wrap ? q_wrap : q_step;
      x.d_o += wrap ? do_wrap : do_step;
      x.stat += stat_step(from, to);
    }
    return x;
  };
  // (joined) bytes from the group's first row on, less than 2^32 (joined_pays); from: elements to the stage's first row
  auto group_offset = [&](int64_t from, At at, const int64_t (&stride)[3]) {
    return 2u * ((uint32_t)from + __umul24(at.rows, (uint32_t)stride[2]) + (uint32_t)at.heads * ((uint32_t)stride[1] - (uint32_t)len * (uint32_t)stride[2]));
  };
  const int stat_turn = (OWN ? p.C : p.stat_stride) - len;
  auto copy_stage = [&](Pos x, int slot, const Src& src) {
    if (inside(x)) {
      const __bf16* q_src = src.q;
      const __bf16* do_src = src.d_o;
      const uint32_t lds = OWN ? opaque(lds_wave) : lds_wave;
#pragma unroll
      for (int i = 0; i < kCopies; ++i) {
        const uint32_t dst = lds + slot * kTileBytes + i * (4 * NW * kRowBytes);
        dma16_sbase(q_src, q_lane_off[i], dst);
        dma16_sbase(do_src, do_lane_off[i], dst + kDoRegion);
      }
    } else if constexpr (JOINED) {
#pragma unroll
      for (int i = 0; i < kCopies; ++i) {
        const uint32_t dst = lds_wave + slot * kTileBytes + i * (4 * NW * kRowBytes);
        const int lr = 4 * (wave + NW * i) + (lane >> 4);
        const At at = row_at(x, lr);
        const uint32_t chunk = (uint32_t)((lane & 15) ^ swz(lr)) << 4;
        dma16_sbase(qbase, group_offset(src.q - qbase, at, p.qs) + chunk, dst);
        dma16_sbase(dobase, group_offset(src.d_o - dobase, at, p.os) + chunk, dst + kDoRegion);
      }
    } else {                                   // rows past the chunk repeat its last one
      const __bf16* q_src = src.q;
      const __bf16* do_src = src.d_o;
#pragma unroll
      for (int i = 0; i < kCopies; ++i) {
        const uint32_t dst = lds_wave + slot * kTileBytes + i * (4 * NW * kRowBytes);
        const uint32_t past = max(4 * (wave + NW * i) + (lane >> 4) + x.r0 - (p.C - 1), 0);
        dma16_sbase(q_src, q_lane_off[i] - __umul24(past, (uint32_t)p.qs[2] * 2u), dst);
        dma16_sbase(do_src, do_lane_off[i] - __umul24(past, (uint32_t)p.os[2] * 2u), dst + kDoRegion);
      }
    }
  };
  // -LSE / s and -delta of the stage's rows, as the dQ kernel left them in the workspace: one
  // asynchronous 64-lane copy each (wavefronts 0 and 1), straight into the stage's slot.  The last, ragged stage
  // of a head goes through registers instead: rows past the chunk get -LSE = -inf so that their probabilities vanish.
  static_assert(BQ == 64, "one 64-lane copy per row statistic");
  const uint32_t lds_stat = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + kStatRegion + (wave & 1) * BQ * 4);
  auto copy_stat = [&](Pos x, int slot, const Src& src) {
    if (inside(x)) {
      if (wave_u < 2) {
        const uint64_t a = (uint64_t)(uintptr_t)src.stat;
        // (wavefront-uniform by construction; the halves go through readfirstlane so that the compiler keeps them
        // in scalar registers; each half is widened from an unsigned 32-bit value)
        const uint64_t src = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32) |
                             (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a);
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1"
                     :
                     : "v"(lane * 4), "s"(src), "s"(lds_stat + slot * kStatBytes)
                     : "memory", "m0");
      }
    } else if (JOINED) {
      if (wave_u < 2) {
        const At at = row_at(x, lane);
        const float* from = src.stat + at.rows + at.heads * stat_turn;
        if (rows_left(x) >= BQ)
          asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dword %0, off" : : "v"(from), "s"(lds_stat + slot * kStatBytes) : "memory", "m0");
        else
          *reinterpret_cast<SECO_LDS float*>(smem + kStatRegion + slot * kStatBytes + (wave_u * BQ + lane) * 4) =
              wave_u == 0 && lane >= rows_left(x) ? -INFINITY : *from;
      }
    } else if (wave_u < 2) {             // (wavefront-uniform control flow only: the copies above need scalar addresses)
      const int row = x.r0 + lane;
      const float v = (wave_u == 0 ? p.nlse2 : p.delta)[stat_base + (int64_t)x.hg * p.stat_stride + min(row, p.C - 1)];
      const float stat = wave_u == 0 && row >= row_limit(x) ? -INFINITY : v;
      *reinterpret_cast<SECO_LDS float*>(smem + kStatRegion + slot * kStatBytes + (wave_u * BQ + lane) * 4) = stat;
    }
  };

  // OWN: each wavefront of role B (the other one has the exponentials) takes 16 of the stage's rows: their LSE, requested an iteration
  // before the stage's copies and left for role A with them, and the O rows, requested with the copies; delta, which role B needs an
  // iteration after that, comes from those and the dO tile that has landed by then.
  const int own_lr = 16 * cb + 4 * pi4((lane >> 2) & 3) + (lane & 3);      // this lane's row of a stage (pi4: no bank conflicts)
  auto own_row = [&](Pos x) { return (uint32_t)min(own_lr, p.C - 1 - x.r0); };
  auto load_lse = [&](Pos x, const float* stat) {                              // stat: of the stage's first row
    if constexpr (JOINED) {
      const At at = row_at(x, own_lr);
      return stat[at.rows + at.heads * stat_turn];
    } else {
      return stat[own_row(x)];
    }
  };
  auto put_lse = [&](Pos x, int slot, float lse) {
    SECO_LDS float* stat = reinterpret_cast<SECO_LDS float*>(smem + kStatRegion + slot * kStatBytes);
    const float v = (JOINED ? own_lr < rows_left(x) : x.r0 + own_lr < p.C) ? -lse / p.scale : -INFINITY;
    if (lane < 16) stat[own_lr] = v;
  };
  struct OwnRows { bf16x8 o[4]; };
  const int64_t o_from_do = static_cast<const char*>(p.o) - static_cast<const char*>(p.d_o);   // (their strides are the same)
  auto load_own = [&](Pos x, const Src& src) {
    OwnRows w;
    if constexpr (JOINED) {
      global_bytes group = scalar_address(reinterpret_cast<const char*>(dobase) + o_from_do);
      const uint32_t off = group_offset(src.d_o - dobase, row_at(x, own_lr), p.os) + (uint32_t)(lane >> 4) * 16u;
#pragma unroll
      for (int t = 0; t < 4; ++t) w.o[t] = global_load16(group, off + 64u * t);
      return w;
    }
    global_bytes from = scalar_address(reinterpret_cast<const char*>(src.d_o) + o_from_do);
    const uint32_t off = __umul24(own_row(x), (uint32_t)p.os[2] * 2u) + (uint32_t)(lane >> 4) * 16u;
#pragma unroll
    for (int t = 0; t < 4; ++t) w.o[t] = global_load16(from, off + 64u * t);
    return w;
  };
  auto put_delta = [&](int slot, const OwnRows& w) {
    bf16x8 d[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) d[t] = lds_row8(smem + kDoRegion + slot * kTileBytes, own_lr, 4 * t + (lane >> 4));
    const float x = row16_dot(w.o, d, lane);
    if (lane < 16) reinterpret_cast<SECO_LDS float*>(smem + kStatRegion + slot * kStatBytes)[BQ + own_lr] = -x;
  };

  // lane-dependent parts of the LDS operand addresses (constant for the whole kernel)
  // role A reads rows of Q and transposed blocks of dO, role B rows of dO and transposed blocks of Q: the region of
  // the tile an offset is used with is part of the offset
  const Products op(lane, role == 0 ? 0 : kDoRegion, role == 0 ? kDoRegion : 0);
  typename Products::Acc acc;   // role A: dV, role B: dK  (32 cache rows x 128)
  Products::clear(acc);

  // P of the stage held in slot `slot`, row block rb, this wavefront's column block: p_lane is the lane-dependent
  // part of the address (the lane's 16 bytes of the wavefront's block), the rest a constant per slot and row block
  int p_lane = cb * RB * kPBytes + lane * 16;
  auto pslot = [&](int slot, int rb) { return pbuf + (slot * NCB * RB + rb) * kPBytes + p_lane; };

  // zero the probabilities of a 32x32 block (first query position qpos0) that lie above the diagonal
  // (the lane-dependent part of the comparison is one value, the rest compile-time constants, so that nothing per-lane has
  // to be kept for it)
  using Tile = typename Products::Tile;
  using Init = typename Products::Init;
  auto mask_above_diagonal = [&](Tile& s, Pos x, int rb) {
    if (JOINED && !inside(x)) {                // each row from its own head's first one on
      const int first = p.q_start + first_r0;
      if (n0 + 31 > first) {
        const int at = x.r0 + 32 * rb, ahead = n0 + op.lane_col - first;
        if (len >= 32) {                       // (at most one head's end in 32 rows)
          const int local0 = at - heads_in(at) * len + op.lane_row, over0 = ahead - local0, over1 = over0 + len, to_end = len - local0;
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if ((Products::row_of(e) < to_end ? over0 : over1) + Products::col_of(e) > Products::row_of(e))
              Products::map(s, e, [](float) { return 0.f; });
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int local = at + op.lane_row + Products::row_of(e);
            if (ahead + Products::col_of(e) > local - heads_in(local) * len) Products::map(s, e, [](float) { return 0.f; });
          }
        }
      }
      return;
    }
    const int qpos0 = p.q_start + (JOINED ? first_r0 : 0) + x.r0 + 32 * rb;
    if (n0 + 31 > qpos0) {
      const int ahead = n0 + op.lane_col - qpos0 - op.lane_row;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (ahead + Products::col_of(e) > Products::row_of(e)) Products::map(s, e, [](float) { return 0.f; });
    }
  };
  auto prob = [&](Tile& s, int e) { Products::map(s, e, [&](float x) { return fast_exp2(x * c2); }); };

  // role A: S = Q K^T for row block rb of the stage in `slot`, P = exp2(c2 * (S - LSE / s)) with the causal mask;
  // P goes to pbuf as two operand halves (lane-contiguous 16-byte words)
  auto scores = [&](int slot, Pos x, int rb, float lw) {   // lw: log2 of the rows' weight, divided by c2
    lds_char* qt = smem + slot * kTileBytes;
    Init init;
    op.chain_init(init, reinterpret_cast<SECO_LDS float*>(smem + kStatRegion + slot * kStatBytes) + 32 * rb);
    if constexpr (ROWS) Products::add(init, lw);
    Tile s;
#pragma unroll
    for (int i = 0; i < 8; ++i) Products::chain(s, i, op.row_op(qt, 32 * rb, i), frag, init);
#pragma unroll
    for (int e = 0; e < 16; ++e) prob(s, e);
    mask_above_diagonal(s, x, rb);
    lds_char* pb = pslot(slot, rb);
    *reinterpret_cast<SECO_LDS bf16x8*>(pb) = Products::pack(s, 0);
    *reinterpret_cast<SECO_LDS bf16x8*>(pb + 1024) = Products::pack(s, 1);
  };

  Pos cur{0, JOINED ? 0 : first_r0, first_ri};
  if (JOINED && it0 > 0) {
    cur.hg = it0 * BQ / len;
    cur.r0 = it0 * BQ - cur.hg * len;
  } else if (it0 > 0) {
    cur.hg = it0 / n_rt;
    int skip = it0 - cur.hg * n_rt;
    if constexpr (ROWS) {
      for (int len; skip >= (len = (rr.end[cur.ri] - cur.r0 + BQ - 1) / BQ); skip -= len) cur.r0 = rr.begin[++cur.ri];
    }
    cur.r0 += skip * BQ;
  }
  Pos nxt = advance(cur);
  OwnRows own_rows;        // of the next stage
  float own_lse = 0.f;     // of the stage two ahead
  Pos nxt2 = advance(nxt);
  const Src s0 = src_of(cur), s1 = next_src(s0, cur, nxt);
  Src src2 = next_src(s1, nxt, nxt2);
  {
    copy_stage(cur, 0, s0);
    if constexpr (!OWN) copy_stat(cur, 0, s0);
    if (n_iter > 1) {
      copy_stage(nxt, 1, s1);
      if constexpr (!OWN) copy_stat(nxt, 1, s1);
    }
    if constexpr (OWN && role == 1) {
      const float lse0 = load_lse(cur, s0.stat);
      const float lse1 = n_iter > 1 ? load_lse(nxt, s1.stat) : 0.f;
      if (n_iter > 2) own_lse = load_lse(nxt2, src2.stat);
      own_rows = load_own(cur, s0);
      put_lse(cur, 0, lse0);
      if (n_iter > 1) put_lse(nxt, 1, lse1);
    }
  }
  // (through the third slot's Q and dO tiles and the P buffers, which are empty until the barriers below)
  Products::frags(frag, fr, wave < 4 ? smem + (wave < 2 ? 0 : kDoRegion) + 2 * kTileBytes + (wave & 1) * 8192
                                     : pbuf + (wave - 4) * 8192, lane);
  settle8(frag);
  dma_wait_all();
  __syncthreads();
  if constexpr (role == 0) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) scores(0, cur, rb, ROWS ? rr.log2w[cur.ri] / c2 : 0.f);
  } else if constexpr (OWN) {
    put_delta(0, own_rows);
    if (n_iter > 1) own_rows = load_own(nxt, s1);
  }
  __syncthreads();

  // One operand buffer x[8] rotates through the four MFMA chains of an iteration: while a chain consumes x[t], the
  // operand of the next chain is requested into the same register ("comes in behind").  The last chain of an
  // iteration requests the operands of the first chain of the next one, which read a stage that has already
  // landed, so that no wavefront starts an iteration by waiting for LDS.  Role A also carries the probabilities of
  // the stage it is about to use for dV (pa0, pa1: its own P blocks, as operands) in registers.
  bf16x8 x[8];
  bf16x8 pa0[2], pa1[2];
  auto p_half = [&](lds_char* pb, int t) { return *reinterpret_cast<SECO_LDS bf16x8*>(pb + 1024 * t); };
  if constexpr (role == 0) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      pa0[t] = p_half(pslot(0, 0), t);
      pa1[t] = p_half(pslot(0, 1), t);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = op.col_op(smem, 0, i);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = op.row_op(smem, 0, i);
  }

  int slot = 0;   // it % kStages
  Products::loop_begins();
  // (role A's last iteration follows the loop)
  for (int it = 0; it < n_iter - (role == 0 ? 1 : 0); ++it) {
    const int slot1 = slot + 1 == kStages ? 0 : slot + 1;
    const int slot2 = slot1 + 1 == kStages ? 0 : slot1 + 1;
    // The copies of stage it + 2 are issued after the first MFMA chain of the iteration, not at its top: right
    // after the barrier every wavefront has the operands of its first chain in registers, and the matrix pipe
    // should start on them at once instead of waiting behind sixteen copy instructions and their address
    // arithmetic (3 % on the kernel; issued later still, the copy has too little time to land before the
    // wait at the end of the iteration).
    auto issue_copies = [&]() {
      if (it + 2 < n_iter) {
        copy_stage(nxt2, slot2, src2);
        if constexpr (!OWN) copy_stat(nxt2, slot2, src2);
      }
      if constexpr (OWN && role == 1) {
        if (it + 1 < n_iter) put_delta(slot1, own_rows);
        if (it + 2 < n_iter) {
          own_rows = load_own(nxt2, src2);
          put_lse(nxt2, slot2, own_lse);
          if (const Pos nxt3 = advance(nxt2); it + 3 < n_iter) own_lse = load_lse(nxt3, src2.stat + stat_step(nxt2, nxt3));
        }
      }
    };
    // tiles of the stage in `slot` and of the next stage; whether an access goes to the Q or to the dO tile of the
    // slot is decided by the region that its per-lane offset (r_off, t_off) carries
    lds_char* t0 = smem + slot * kTileBytes;
    lds_char* t1 = smem + slot1 * kTileBytes;
    // Row blocks above the diagonal are not skipped: their probabilities are masked to zero and contribute nothing
    // (only the first stages of a diagonal column tile are affected).  In both roles the vector work on a row block
    // (exponentials; dS = P * (dP - delta)) is written between the MFMAs of a later chain, two values per MFMA, so
    // that a wavefront keeps the matrix pipe fed while its own vector instructions issue.
    if constexpr (role == 0) {
      // stage `it`: dV += P^T dO (P from the previous iteration); stage `it + 1`: P = exp2(Q K^T c - LSE)
      SECO_LDS float* lse_s = reinterpret_cast<SECO_LDS float*>(smem + kStatRegion + slot1 * kStatBytes);
      // dV of row block 0; Q rows of row block 0 of the next stage come in behind
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::sum(acc, i, pa0, x[i]);
        x[i] = op.row_op(t1, 0, i);
        Products::step_end();
      }
      issue_copies();
      Init init0, init1;
      op.chain_init(init0, lse_s);
      op.chain_init(init1, lse_s + 32);
      if constexpr (ROWS) {                   // probabilities of the next stage's rows carry their run's weight
        const float lw = rr.log2w[nxt.ri] / c2;
        Products::add(init0, lw);
        Products::add(init1, lw);
      }
      Tile s0, s1;
      // log2 P of row block 0 (chain started from -LSE); Q rows of row block 1 come in behind
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::chain(s0, i, x[i], frag, init0);
        x[i] = op.row_op(t1, 32, i);
        Products::step_end();
      }
      // log2 P of row block 1, with the exponentials of row block 0; dO^T of row block 1 (stage `it`) comes in behind
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::chain(s1, i, x[i], frag, init1);
        x[i] = op.col_op(t0, 32, i);
        prob(s0, 2 * i);
        prob(s0, 2 * i + 1);
        Products::step_end();
      }
      mask_above_diagonal(s0, nxt, 0);
      const bf16x8 pn0[2] = {Products::pack(s0, 0), Products::pack(s0, 1)};
      lds_char* pw0 = pslot(slot1, 0);
      *reinterpret_cast<SECO_LDS bf16x8*>(pw0) = pn0[0];
      *reinterpret_cast<SECO_LDS bf16x8*>(pw0 + 1024) = pn0[1];
      // dV of row block 1, with the exponentials of row block 1 of the next stage; dO^T of row block 0 of the next
      // stage comes in behind (for the first chain of the next iteration)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::sum(acc, i, pa1, x[i]);
        x[i] = op.col_op(t1, 0, i);
        prob(s1, 2 * i);
        prob(s1, 2 * i + 1);
        Products::step_end();
      }
      mask_above_diagonal(s1, nxt, 1);
      pa0[0] = pn0[0];
      pa0[1] = pn0[1];
      pa1[0] = Products::pack(s1, 0);
      pa1[1] = Products::pack(s1, 1);
      lds_char* pw1 = pslot(slot1, 1);
      *reinterpret_cast<SECO_LDS bf16x8*>(pw1) = pa1[0];
      *reinterpret_cast<SECO_LDS bf16x8*>(pw1 + 1024) = pa1[1];
    } else {
      // stage `it`: dS = P * (dO V^T - delta), dK += dS^T Q
      SECO_LDS float* delta_s = reinterpret_cast<SECO_LDS float*>(smem + kStatRegion + slot * kStatBytes) + BQ;
      lds_char* pb0 = pslot(slot, 0);
      const bf16x8 ph0[2] = {p_half(pb0, 0), p_half(pb0, 1)};
      lds_char* pb1 = pslot(slot, 1);
      const bf16x8 ph1[2] = {p_half(pb1, 0), p_half(pb1, 1)};
      Init init0, init1;
      op.chain_init(init0, delta_s);
      op.chain_init(init1, delta_s + 32);
      Tile d0, d1;
      auto times = [&](Tile& d, const bf16x8 (&ph)[2], int e) { Products::map(d, e, [&](float x) { return x * (float)ph[e >> 3][e & 7]; }); };
      // dP - delta of row block 0 (chain started from -delta); dO rows of row block 1 come in behind
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::chain(d0, i, x[i], frag, init0);
        x[i] = op.row_op(t0, 32, i);
        Products::step_end();
      }
      issue_copies();
      // dP - delta of row block 1, with dS of row block 0; Q^T of row block 0 comes in behind
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::chain(d1, i, x[i], frag, init1);
        x[i] = op.col_op(t0, 0, i);
        times(d0, ph0, 2 * i);
        times(d0, ph0, 2 * i + 1);
        Products::step_end();
      }
      const bf16x8 ds0[2] = {Products::pack(d0, 0), Products::pack(d0, 1)};
      // dK of row block 0, with dS of row block 1; Q^T of row block 1 comes in behind
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::sum(acc, i, ds0, x[i]);
        x[i] = op.col_op(t0, 32, i);
        times(d1, ph1, 2 * i);
        times(d1, ph1, 2 * i + 1);
        Products::step_end();
      }
      const bf16x8 ds1[2] = {Products::pack(d1, 0), Products::pack(d1, 1)};
      // dK of row block 1; dO rows of row block 0 of the next stage come in behind (for the next iteration)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::sum(acc, i, ds1, x[i]);
        x[i] = op.row_op(t1, 0, i);
        Products::step_end();
      }
    }
    dma_wait_all();
    __syncthreads();
    cur = nxt;
    nxt = nxt2;
    {
      const Pos adv = advance(nxt2);
      src2 = next_src(src2, nxt2, adv);
      nxt2 = adv;
    }
    slot = slot1;
  }

  // The sums leave through LDS (each wavefront turns its 32 x 128 tile in 16.5 KiB of its own), so that gK/gV and the
  // partial sums are accessed in whole 512-byte rows, 1 KiB per instruction: in the accumulators' layout an
  // instruction covers 128 bytes of two rows, and a workgroup's 1024 such accesses keep the address unit busy for
  // longer than the data takes.
  // (The lane-dependent indices are derived again from the thread index, through an empty asm, so that the compiler
  // does not keep the ones computed before the loop alive across it: the loop uses every register.)
  int tid_e = threadIdx.x;
  asm volatile("" : "+v"(tid_e));
  const int lane_e = tid_e & 63, l32_e = tid_e & 31, wave_e = tid_e >> 6;
  const int n0_e = c0 + (wave_e % NCB) * 32;
  float* gbase = (role == 0 ? p.gv : p.gk) + b * p.gs[0] + kvh * p.gs[1] + l32_e * 4;
  f32x4 old[16];
  auto request_old = [&]() {
#pragma unroll
    for (int j = 0; j < 16; ++j)
      old[j] = *reinterpret_cast<const f32x4*>(gbase + (int64_t)min(n0_e + 2 * j + (lane_e >> 5), c_end - 1) * p.gs[2]);
  };
  // Role A's last iteration: dV of the last stage, without the probabilities of a stage that does not exist, and with the old
  // values of gV on their way in the registers those would take, under its products and role B's.  With few iterations to a
  // tile that memory round trip is a good part of it: 32 rows at 16352 of 32/8 heads 94.4 -> 89.6 us for dQ and dK/dV, 128 at 4000 of
  // 8/8 31.7 -> 29.5, 128 at 16256 of 32/8 150.3 -> 147.5, 512 at 15872 419 -> 417; 1024 rows or more the same.  (Role B's last
  // iteration likewise: 128 at 16256 148.3, 128 at 4000 30.1, 2048 at 30720 0.3 % slower.)
  if constexpr (role == 0) {
    if (n_iter > 0) {
      lds_char* t0 = smem + slot * kTileBytes;
      if (!divided) request_old();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        Products::sum(acc, i, pa0, x[i]);
        x[i] = op.col_op(t0, 32, i);
        Products::step_end();
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) Products::sum(acc, i, pa1, x[i]);
      // (nothing is being copied any more; the old values need not have come)
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
    } else if (!divided) {
      request_old();
    }
  }
  constexpr int kTurnRow = 528;                                          // bytes; 16 of padding
  static_assert(2 * NCB * 32 * kTurnRow <= Cfg::kSmemBytes, "the turned tiles fit the ring's LDS");
  lds_char* own = smem + wave_e * (32 * kTurnRow);
  auto turn_in = [&]() {
    Products::each(acc, lane_e, [&](int row, int col, float x) { *reinterpret_cast<SECO_LDS float*>(own + row * kTurnRow + col * 4) = x; });
  };
  auto turned = [&](int j) {                                             // row 2 j + lane / 32, columns 4 (lane % 32) ..
    return *reinterpret_cast<SECO_LDS f32x4*>(own + (2 * j + (lane_e >> 5)) * kTurnRow + l32_e * 16);
  };
  if (divided) {
    // a share of the tile: plain stores of the unweighted sums, all 32 rows (the merge drops rows past the tile's end)
    const int n_slots = ts.plan.first[ts.plan.n_shared];
    float* pb = ts.part + (((int64_t)unit * n_slots + (in_unit - n_whole)) * 2 + role) * (int64_t)(Cfg::kCols * 128) +
                (wave_e % NCB) * 32 * 128 + lane_e * 4;
    turn_in();
#pragma unroll
    for (int j = 0; j < 16; ++j) *reinterpret_cast<f32x4*>(pb + j * 256) = turned(j);
    return;
  }
  // exclusive read-modify-write of this workgroup's gK/gV rows: role A adds dV, role B adds s * dK.  All old values
  // are requested before the tile is turned (rows past the tile's end read a clamped address and are not written
  // back): one memory round trip, under the LDS work and, for role A, the last products.
  const float wf = role == 0 ? weight : weight * p.scale;
  if constexpr (role != 0) request_old();
  turn_in();
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int row = n0_e + 2 * j + (lane_e >> 5);
    const f32x4 x = turned(j);
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = old[j][i] + wf * x[i];
    if (row < c_end) *reinterpret_cast<f32x4*>(gbase + (int64_t)row * p.gs[2]) = v;
  }
}

}  // namespace
}  // namespace seco
