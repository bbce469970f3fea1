// Internal declarations shared by the host entry points and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fast_div.h"
#include "seco.h"

namespace seco {

struct PendingDq;

// Everything a kernel needs to know about one chunk call (validated by the host side): what all of them need, and all that the
// fp32 kernels are launched with (with the divisors a backward call of 10 us takes 0.1 more), and ...
struct AttnArgs {
  const void* q;
  const void* k;
  const void* v;
  const void* o;
  const void* d_o;
  void* o_out;
  void* d_q;
  float* lse;        // [B, Hq, C] contiguous
  float* delta;      // bf16 backward: -rowsum(dO * O), [B, Hq, stat_stride], written by the dQ kernel for the dK/dV kernel
  float* nlse2;      // bf16 backward: -LSE / scale, likewise
  int stat_stride;   // rows per (batch, head) of delta / nlse2: C (workspace of one call), or the length of
  int stat_off;      // arrays kept for the whole sequence, in which this call's first query row sits at stat_off
  float* gk;
  float* gv;
  float* part;       // split path: partial O (forward) or partial dQ (backward), fp32 [n_splits, B, Hq, C, D]
  float* part_ml;    // split path, forward: (reference max in log2 units, sum) per partial row, [n_splits, B, Hq, C, 2]
  float* tail_part;  // workspace, or NULL: dQ pass: sums of the row tiles beyond the first round (row_shares); dK/dV pass,
                     // after it: of the column tiles shared out among several workgroups
  uint32_t tail_bytes; // room there (under 64 MiB); a function of the descriptor, not of the workspace that was passed
  int rows_whole;    // row tiles beyond the first round divided: how many of a (batch, KV head)'s are not
  int n_splits;      // > 1 selects the split path
  int Cpad;          // C rounded up to 32: rows per head in the packed row space of the split path
  int B, Hq, Hkv, D, C, q_start, G;
  float scale;
  int64_t qs[3], os[3], kvs[3], gs[3];
};
// ... the rest.
struct AttnParams : AttnArgs {
  Div by_C, by_Cpad, by_Hq, by_Hkv, by_G;
  Div by_tiles, by_splits;   // row tiles and n_splits of a launch (for_launch)
  int n_ctiles;              // dK/dV: column tiles of a (batch, KV head), and its workgroups
  Div by_unit;
  PendingDq* pending;   // backward, host side: a dQ pass that is announced but not launched yet
};

// What a kernel of row tiles is launched with
inline AttnParams for_launch(const AttnParams& p, int n_mtiles) {
  AttnParams x = p;
  x.by_tiles = make_div(n_mtiles);
  x.by_splits = make_div(p.n_splits);
  return x;
}

// Memory that a [B, H, rows, D] tensor lies in, first byte to last (strides in elements, none negative).
struct Span { uintptr_t begin, end; };
inline Span span_of(const void* t, const int64_t st[3], int B, int H, int rows, int D, int elem_bytes) {
  const uintptr_t last = (uintptr_t)(B - 1) * st[0] + (uintptr_t)(H - 1) * st[1] + (uintptr_t)(rows - 1) * st[2] + D;
  return Span{reinterpret_cast<uintptr_t>(t), reinterpret_cast<uintptr_t>(t) + last * elem_bytes};
}
inline bool overlap(Span a, Span b) { return a.begin < b.end && b.begin < a.end; }
// O may be written over Q: a workgroup that owns its rows reads Q before it writes O.  Several workgroups for the same rows
// would read what another has written, so a forward that has such a form asks here first (spans, not elements: interleaved
// tensors count as overlapping and only lose that form).
inline bool o_over_inputs(const AttnParams& p, int elem_bytes) {
  const Span o = span_of(p.o_out, p.os, p.B, p.Hq, p.C, p.D, elem_bytes);
  return overlap(o, span_of(p.q, p.qs, p.B, p.Hq, p.C, p.D, elem_bytes)) ||
         overlap(o, span_of(p.k, p.kvs, p.B, p.Hkv, p.q_start + p.C, p.D, elem_bytes)) ||
         overlap(o, span_of(p.v, p.kvs, p.B, p.Hkv, p.q_start + p.C, p.D, elem_bytes));
}
// Likewise dQ, which may be written over O: the dK/dV workgroups that run beside it in one launch read O too (as do several
// workgroups for the same rows).
inline bool dq_over_inputs(const AttnParams& p, int elem_bytes) {
  const Span dq = span_of(p.d_q, p.qs, p.B, p.Hq, p.C, p.D, elem_bytes);
  return overlap(dq, span_of(p.q, p.qs, p.B, p.Hq, p.C, p.D, elem_bytes)) ||
         overlap(dq, span_of(p.o, p.os, p.B, p.Hq, p.C, p.D, elem_bytes)) ||
         overlap(dq, span_of(p.d_o, p.os, p.B, p.Hq, p.C, p.D, elem_bytes)) ||
         overlap(dq, span_of(p.k, p.kvs, p.B, p.Hkv, p.q_start + p.C, p.D, elem_bytes)) ||
         overlap(dq, span_of(p.v, p.kvs, p.B, p.Hkv, p.q_start + p.C, p.D, elem_bytes));
}

// Column segments of the dK/dV pass: a run of cache rows that share one weight.
// The table travels by value in the kernel arguments, so no device memory or
// host-to-device copy is needed for SpaCO's selection.
constexpr int kMaxSegments = 48;
struct SegTable {
  int n;
  int col_begin[kMaxSegments];
  int col_end[kMaxSegments];
  float weight[kMaxSegments];
  int tile_begin[kMaxSegments + 1];  // prefix sum of column tiles, in units of the launcher's tile width
};

// What launch_dq_f32 / launch_dq_bf16 leave for the dK/dV launcher that follows
struct PendingDq {
  bool dq = false;
  bool sparse = false;   // bf16: dQ visits `runs` only (fp32 always has them)
  SegTable runs;
};

// Runs of query rows of the dK/dV pass in the transposed order: rows [begin, end) relative to the call's first
// query row, begin a multiple of 64, ascending and disjoint; the probabilities of a run's rows are scaled by its
// weight (log2w = log2 of the weight).  By value in the kernel arguments, like the column segments.
constexpr int kMaxRowRuns = 24;
// How the stages of the dK/dV pass take the query rows (bwd_dkdv_body.h)
enum Rows { kAll, kRuns, kJoined };
struct RowRuns {
  int n;
  int begin[kMaxRowRuns];
  int end[kMaxRowRuns];
  float log2w[kMaxRowRuns];
};

// Split path of the bf16 forward and dQ kernels (short chunks): the rows of the G heads of a KV head are packed
// into row tiles of 128, and the visible cache rows of a tile are divided among several workgroups.
struct SplitPlan {
  int n_mtiles;     // row tiles per (batch, KV head)
  int items;        // B * Hkv * n_mtiles
  int max_splits;   // 1: the split path is never used for this shape
};
// Compute units of the current device, asked of the device once per process (kDefaultCUs, an MI355X's 256, when
// there is no device to ask, as in host-only use of the planning calls).  Every launch-shape decision below and in the launchers counts
// workgroups against this one number; seco_device_info reports the same attribute.
constexpr int kDefaultCUs = 256;
int device_cus();

// Times that the rules below and in bwd_plan.h weigh against each other, in microseconds: a workgroup takes `wg` around its loop
// and `step` per step of it (forward, dQ: 128 cache rows; dK/dV: an iteration, 64 query rows of one head).  What a
// workgroup takes depends on what runs beside it (the clock falls as the chip fills, dK/dV workgroups that end together wait for each
// other's gK / gV), so a kernel has a line for each situation, and a rule uses the line of its own.  After a change to a kernel
// its lines are measured anew: calls of the named kind at several numbers of steps, one workgroup per CU, kernel times from
// seco_profile_read, a straight line through them; those called "fit": least squares over the calls that their rule
// names, whole backward calls timed, with the offsets beside them.  (Measured with 32x32x16 products throughout.  With dQ and dK/dV in
// 16x16x32 ones, 3 - 7 % faster in launches of their own, 36 calls on both sides of the rules' lines were timed in one launch
// and in two: what the rules take is the faster or within 1.7 % of it.)
struct WgTime {
  float wg, step;
  float of(float steps) const { return wg + step * steps; }
};
constexpr WgTime kFwdTime{6.f, 1.8f};           // forward, dense calls of one round
constexpr WgTime kDqTime{7.5f, 2.7f};           // dQ, likewise
constexpr WgTime kDqBesideTime{7.5f, 2.5f};     // dQ while dK/dV workgroups have the other CUs
constexpr WgTime kDkdvTime{8.f, 1.6f};          // dK/dV alone, at most a round
constexpr WgTime kDkdvOwnTime{8.5f, 1.8f};      // dK/dV that computes its row statistics, dQ beside it
constexpr WgTime kDkdvRoundTime{14.f, 2.f};     // the same over several rounds, dQ in front of it: fit (rounds_in_one_launch)
constexpr WgTime kDqFrontTime{8.f, 2.7f};       // that dQ
constexpr float kMergeLaunch = 4.f;             // a merge, without what it reads and writes

inline SplitPlan split_plan(int B, int Hkv, int G, int C) {
  SplitPlan pl;
  const int cus = device_cus();
  const int cpad = (C + 31) / 32 * 32;
  pl.n_mtiles = (G * cpad + 127) / 128;
  pl.items = B * Hkv * pl.n_mtiles;
  pl.max_splits = pl.items >= cus ? 1 : (2 * cus + pl.items - 1) / pl.items;
  if (pl.max_splits > 64) pl.max_splits = 64;
  return pl;
}
// Number of splits for a call that sees kv_len cache rows: the one with the least estimated time, in units of 0.1 us as
// measured: a round of one workgroup per CU takes 60 plus 17 per 128-row tile of its share, a merge 40 plus 0.3 per share.
inline int split_count(const SplitPlan& pl, int kv_len) {
  const int tiles = (kv_len + 127) / 128, cus = device_cus();
  const int most = pl.max_splits < tiles ? pl.max_splits : tiles;
  int best = 1, best_t = 0;
  for (int n = 1; n <= most; ++n) {
    const int wgs = pl.items * n, rounds = (wgs + cus - 1) / cus;
    const int t = rounds * (60 + 17 * ((tiles + n - 1) / n)) + (n > 1 ? 40 + 3 * wgs / 10 : 0);
    if (n == 1 || t < best_t) {
      best = n;
      best_t = t;
    }
  }
  return best;
}
// Row tiles between one and two rounds of workgroups, one per CU: the second round, which would be as long as the first
// however few tiles it has, is divided.  Of every (batch, KV head)'s packed row tiles the first `whole` (together one round)
// stay whole, the others have their cache rows divided among `shares` workgroups each, which run in short rounds of their
// own; shares 1: nothing is divided.  slots: partial tiles that the workspace holds; n_plain: workgroups without packing,
// the alternative.  wg: kFwdTime or kDqTime; a merge 5 us + 0.03 per share.  Chosen where that comes out 5 % below the undivided call, and only where the
// tiles are about equally long (a chunk of at most half of what precedes it: the rounds' lengths are those of the mean).
// Microseconds before -> after, 32 heads on 8, batch 1:
//   rows @ preceding    1100 @ 9000   1500 @ 9000   1300 @ 3000   1060 @ 30000   1900 @ 9000 (undivided by the rule)
//   forward              268 -> 196    281 -> 265    106 -> 100    878 -> 597     328 -> 327
//   backward, both passes 684 -> 577   803 -> 764    291 -> 278   2097 -> 1691    977 -> 977
// and 16 heads on 2, 2500 @ 9000: 308 -> 234, 844 -> 737; 8 on 8, 4500 @ 12000: 372 -> 290.  Least where dK/dV outweighs dQ and
// the clock falls as idle CUs get work: two sequences of 777 @ 9324 844 -> 835 (dQ 404 -> 374 and a merge of 7, 2.07 -> 1.96 GHz).
constexpr int kMaxRowShares = 8;
struct RowShares { int whole, shares; };
inline RowShares row_shares(int n_units, int n_mtiles, int n_plain, int q_start, int C, size_t slots, WgTime wg) {
  const int cus = device_cus(), whole = cus / n_units, n_cut = n_mtiles - whole, tiles = (q_start + C / 2 + 127) / 128;
  RowShares best{0, 1};
  if (whole < 1 || n_cut < 1 || n_plain >= 2 * cus || q_start < 2 * C) return best;
  const float one = wg.of(tiles);
  float best_t = 0.95f * ((n_plain + cus - 1) / cus) * one;
  for (int k = 2; k <= kMaxRowShares && k <= q_start / 128; ++k) {
    const int64_t n = (int64_t)n_units * n_cut * k;
    if ((size_t)n > slots) break;
    const float t = one + (n + cus - 1) / cus * wg.of((tiles + k - 1) / k) + 5.f + 0.03f * n;
    if (t < best_t) {
      best_t = t;
      best = RowShares{whole, k};
    }
  }
  return best;
}
// Partial tiles that a forward's workspace holds for that (0: the shape never divides them); by the shape alone
inline int fwd_share_slots(int B, int Hq, int Hkv, int C) {
  const int cus = device_cus(), units = B * Hkv, n_mtiles = split_plan(B, Hkv, Hq / Hkv, C).n_mtiles;
  if (units > cus || (int64_t)units * n_mtiles <= cus || (int64_t)B * Hq * ((C + 127) / 128) >= 2 * cus) return 0;
  const int n = units * (n_mtiles - cus / units) * kMaxRowShares;
  return n < 2 * cus ? n : 2 * cus;
}
// Tiles of 128 cache rows that dQ over a table of runs visits (the chunk's last rows; no run starts behind them)
inline int visited_tiles(const AttnParams& p, const SegTable& runs) {
  int n = 0;
  for (int i = 0; i < runs.n; ++i) {
    const int end = runs.col_end[i] < p.q_start + p.C ? runs.col_end[i] : p.q_start + p.C;
    n += (end - runs.col_begin[i] + 127) / 128;
  }
  return n;
}
int launch_fwd_merge(const AttnParams& p, hipStream_t s);   // O, LSE from the partials
int launch_dq_merge(const AttnParams& p, hipStream_t s);    // dQ = scale * sum of the partials, in split order

// Last round of the bf16 dK/dV pass.  One workgroup fills a CU, so n_units * n_ctiles column tiles run in rounds of
// one workgroup per CU; when the last round would hold at most half of that, the last n_tiles column tiles of every
// (batch, KV head) are shared out among at least hs workgroups (hs = 1: by this rule none are).  hs divides the group's
// heads, a share keeps at least 512 query rows, and all shares together fit one round (device_cus() shares at most,
// which is also what the workspace for their partial sums is sized for).  share_plan below starts from this.
struct TailPlan {
  int n_tiles;
  int hs;
};
inline TailPlan tail_plan(int n_units, int n_ctiles, int G, int C) {
  TailPlan tp{0, 1};
  const int round = device_cus();
  const int64_t items = (int64_t)n_units * n_ctiles;
  const int tail = (int)(items % round);
  if (tail == 0 || tail > round / 2) return tp;
  const int n_tiles = (tail + n_units - 1) / n_units;
  for (int hs = 4; hs >= 2; hs >>= 1) {
    if (G % hs != 0 || (int64_t)n_units * n_tiles * hs > round) continue;
    if ((int64_t)C * (G / hs) < 512) continue;
    tp.n_tiles = n_tiles;
    tp.hs = hs;
    break;
  }
  return tp;
}

// What the dK/dV launcher makes of that: the list of column tiles that end a (batch, KV head)'s work, each with the
// number of workgroups that share its iterations (an iteration: 64 query rows of one head).  The last round's tiles as
// above, or, when all tiles fit one round, all of them; an iteration range may cut through heads, so that any number
// of shares is possible, and tiles on the diagonal, which have fewer iterations, get fewer shares.
constexpr int kMaxEntries = 256;
struct SharePlan {
  int n_tiles;                        // column tiles in the list, the last ones of every (batch, KV head)
  int n_shared;                       // of these, how many are shared out: the first ones (they see the most rows)
  int n_entries;                      // workgroups per (batch, KV head) for the list
  uint8_t tile_of[kMaxEntries];       // list position of a workgroup's tile (the kernel reads words: 4-byte boundaries)
  uint16_t first[kMaxEntries + 2];    // first workgroup of a list position; shared tiles come first, so for them it is
};                                    // also the first slot of partial sums

// Iterations of the last n_tiles (at most kMaxEntries) column tiles of a (batch, KV head), as runs of equal numbers; they do
// not increase (a tile behind the chunk's first row sees fewer rows), so there are few runs.
struct IterRuns {
  int n_tiles, n;
  int iters[kMaxEntries], count[kMaxEntries];
};
template <typename F>
inline IterRuns iter_runs(int n_ctiles, const F& iters) {
  IterRuns r;
  r.n_tiles = n_ctiles < kMaxEntries ? n_ctiles : kMaxEntries;
  r.n = 0;
  for (int i = 0; i < r.n_tiles; ++i) {
    const int it = iters(n_ctiles - r.n_tiles + i);
    if (r.n > 0 && r.iters[r.n - 1] == it) {
      ++r.count[r.n - 1];
    } else {
      r.iters[r.n] = it;
      r.count[r.n++] = 1;
    }
  }
  return r;
}
// f(iterations, tiles with that many) over the last n tiles
template <typename F>
inline void for_last(const IterRuns& r, int n, const F& f) {
  int skip = r.n_tiles - n;
  for (int i = 0; i < r.n; ++i) {
    const int c = r.count[i] - (skip < r.count[i] ? skip : r.count[i]);
    skip -= r.count[i] - c;
    if (c > 0) f(r.iters[i], c);
  }
}

// How to share out the last n tiles of every unit: the most iterations a workgroup gets (0: nothing is shared out), the
// time that is expected to take and how much of it the longest workgroup takes.  wg: of a workgroup; partial sums take
// 4 us + 0.03 per share (written and read again) + 0.02 per tile.
// fit: all workgroups of the list must run at once, on `cus` compute units.
struct ShareChoice { int per; float time, longest, even, span; };   // even, span: without the merge, if all CUs worked alike and as it is
template <int N>
inline void choose_shares(const IterRuns& r, int n, int n_units, const int (&cus)[N], int slots, int min_ways, bool fit, WgTime wg,
                          ShareChoice (&best)[N]) {      // for each of N numbers of compute units
  static const int ways[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32};
  int most = 0;
  for_last(r, n, [&](int it, int) { most = it > most ? it : most; });
  for (ShareChoice& c : best) c = ShareChoice{0, -1.f, 0.f, 0.f, 0.f};
  for (int w : ways) {
    if (w < min_ways) continue;
    const int per = (most + w - 1) / w;
    if (per < 2 && w > 1) break;
    int entries = 0, shared = 0, tiles = 0;
    float sum = 0.f, longest = 0.f;
    for_last(r, n, [&](int it, int count) {
      const int k = it > per ? (it + per - 1) / per : 1;
      if (k > 1) shared += k * count, tiles += count;
      entries += k * count;
      sum += count * (k * wg.wg + it * wg.step);
      const float t = wg.of((it + k - 1) / k);
      if (t > longest) longest = t;
    });
    if (entries > kMaxEntries || shared * n_units > slots) break;
    bool any = false;                                    // (more ways are more workgroups still)
    for (int i = 0; i < N; ++i) {
      if (fit && entries * n_units > cus[i]) continue;
      any = true;
      const float even = sum * n_units / cus[i];
      float t = entries * n_units <= cus[i] ? longest : even + 0.5f * longest > longest + wg.wg ? even + 0.5f * longest : longest + wg.wg;
      const float span = t;
      if (shared > 0) t += kMergeLaunch + (0.03f * shared + 0.02f * tiles) * n_units;
      if (best[i].time < 0.f || t < best[i].time) best[i] = ShareChoice{w > 1 ? per : 0, t, longest, even, span};
    }
    if (!any) break;
  }
}
inline ShareChoice choose_shares(const IterRuns& r, int n, int n_units, int cus, int slots, int min_ways, bool fit, WgTime wg) {
  const int one[1] = {cus};
  ShareChoice best[1];
  choose_shares(r, n, n_units, one, slots, min_ways, fit, wg, best);
  return best[0];
}
inline SharePlan make_shares(const IterRuns& r, int n, int per) {
  SharePlan sp;
  sp.n_tiles = sp.n_shared = sp.n_entries = 0;
  if (per == 0) return sp;
  for_last(r, n, [&](int it, int count) {
    const int k = it > per ? (it + per - 1) / per : 1;
    for (int c = 0; c < count; ++c) {
      const int i = sp.n_tiles++;
      if (k > 1) sp.n_shared = i + 1;
      sp.first[i] = (uint16_t)sp.n_entries;
      for (int j = 0; j < k; ++j) sp.tile_of[sp.n_entries++] = (uint8_t)i;
    }
  });
  sp.first[n] = (uint16_t)sp.n_entries;
  return sp;
}
// The column tiles at the end of every (batch, KV head) that are shared out among several workgroups: a share's sums go
// to part[unit][workgroup of the list][dV, dK][cache row of the tile][128] instead of gK/gV.
struct TailSplit {
  float* part;
  SharePlan plan;
};
// What a launch of column tiles is told of them; returns the workgroups of a (batch, KV head)
inline int for_column_tiles(AttnParams& p, const SegTable& seg, const TailSplit& ts) {
  p.n_ctiles = seg.tile_begin[seg.n];
  const int per_unit = p.n_ctiles - ts.plan.n_tiles + ts.plan.n_entries;
  p.by_unit = make_div(per_unit);
  return per_unit;
}
// For a dK/dV pass that has the chip to itself; time: what it is expected to take from its last full round on; busy: the part of its
// workgroups' time in that of all CUs
inline SharePlan share_plan(const IterRuns& r, int n_units, int n_ctiles, int G, int n_rows, int slots, float& time, float* busy = nullptr) {
  const int cus = device_cus();
  const int64_t items = (int64_t)n_units * n_ctiles;
  const int tail = (int)(items % cus);
  const TailPlan tp = tail_plan(n_units, n_ctiles, G, n_rows);
  const int n = tp.hs > 1 ? tp.n_tiles : items < cus ? n_ctiles : (tail + n_units - 1) / n_units;
  time = kDkdvTime.of(r.iters[0]);
  const float full = (float)(items / cus);
  if (busy) *busy = tail == 0 ? 1.f : (full + (float)tail / cus) / (full + 1.f);
  // One full round, whose tiles on the diagonal end early (of further rounds the next tiles would follow).  us, dK/dV taken for busy
  // throughout -> so (kBusy): 4096 rows at 0 of 32/8 heads 370 -> 353, two of 1933 at 0 of 8/8 55.4 -> 53.3, 3300 at 700 of 16/8 157 ->
  // 152.  With two pairs for the eight XCDs half of these idle and the others work as in a full launch (16384 at 0 of 16/2 3125 -> 3174).
  if (busy && items == cus && n_units >= 4) {
    float sum = 0.f;
    for_last(r, r.n_tiles, [&](int it, int count) { sum += count * kDkdvTime.of(it); });
    *busy = sum / (r.n_tiles * time);
  }
  if (tail == 0 || slots < 2 * n_units || n > r.n_tiles) return make_shares(r, 0, 0);
  const ShareChoice c = choose_shares(r, n, n_units, cus, slots, tp.hs > 1 ? tp.hs : 1, false, kDkdvTime);
  if (c.time >= 0.f) {
    if (busy) *busy = (full * time + c.even) / (full * time + c.span);
    time = c.time;
  }
  return make_shares(r, n, c.per);
}

// fp32 kernels (any head_dim that is a multiple of 4, up to 256)
int launch_fwd_f32(const AttnParams& p, hipStream_t s);
int launch_dq_f32(const AttnParams& p, const SegTable* dq_runs, hipStream_t s);   // dq_runs as in launch_dq_bf16
int launch_dkdv_f32(const AttnParams& p, const SegTable& seg, hipStream_t s);
constexpr int kColTileF32 = 16;    // columns per workgroup in launch_dkdv_f32

// bf16 matrix-core kernels (head_dim 128)
int launch_fwd_bf16(const AttnParams& p, hipStream_t s);
// the 4-wavefront forward kernel (its own translation unit)
int launch_fwd4_bf16(const AttnParams& p, int n_mtiles, int total, hipStream_t s);
// Whether the workgroups of a CU take turns.  If not, the older one ends first, which is what a launch wants only where its next
// tile then starts at a better time; else its last tiles start late or run alone.  600 calls of 1 - 8 rounds (two workgroups per CU) measured;
// 1.03 times as fast by this rule, us without -> with turns:
//   5125 rows at 5125 of 16/8 heads 359 -> 315    2372 at 1221 of 32/8 112 -> 98     7428 at 0 of 16/8 220 -> 202
//   two of 4126 at 0 of 8/8 107 -> 98             15863 at 0 of 32/8 1671 -> 1641
// Without where long and short tiles meet, up to 1.6 rounds and around three: a causal chunk with little before it (2556 at 0 of 32/8 61 ->
// 63, 12412 at 0 of 8/8 291 -> 305, 2476 at 281 69 -> 71, 5229 at 0 201 -> 206; but 2842 at 848 118 -> 107), unless an XCD has two KV
// heads one behind the other; and with tiles alike, a little over two rounds (4551 at 11084 948 -> 990, two of 8215 at 6682 of 8/8 654 ->
// 694; at 2.56 rounds, 5159 at 6104, 695 -> 667).
// Nor where an XCD has three or four KV heads and the tiles of the last begin as those of the first end: four heads with two full rounds
// or a little more (4096 at 0 of 32/32 157 -> 162, 3994 at 300 166 -> 174, at 1800 249 -> 253; but 3964 at 0, a tile of each
// head less, 156 -> 148), three with 1.7 to 2.95 and little before the chunk (5400 at 0 of 24/24 197 -> 205, 5917 226 -> 233, 7900 363 -> 377;
// 200 calls).  With two or eight heads to an XCD turns are 1.04 - 1.1 times as fast there.
inline bool turns_pay(const AttnParams& p, int total) {
  const float rounds = total / (2.f * device_cus()), before = (float)p.q_start / p.C;
  if (p.B * p.Hkv <= 8 && before < 0.8f * (1.6f - rounds)) return false;
  if (p.B * p.Hkv <= 8 && before < 0.1f && rounds >= 2.4f && rounds < 3.25f) return false;
  if (p.B * p.Hkv == 24 && rounds >= 1.7f && (rounds < 2.02f ? before < 0.6f : rounds < 2.95f - 2.f * before)) return false;
  if (p.B * p.Hkv == 32 && before < 0.5f && rounds >= 2.f && rounds < 2.2f) return false;
  return !(before >= 0.15f && rounds >= 2.02f && rounds < 2.55f);
}
// the 8-wavefront forward kernel's short-chunk variant, which writes partials (likewise)
int launch_fwd8_split_bf16(const AttnParams& p, int n_mtiles, int total, hipStream_t s);
// ... and its variant that divides the row tiles beyond the first round, with the merge behind it
int launch_fwd8_shares_bf16(const AttnParams& p, int n_mtiles, hipStream_t s);
// few query rows per KV head (fwd_small_pays); max_splits: how many partial results the workspace holds (1: there is none)
int launch_fwd_small_bf16(AttnParams p, int max_splits, hipStream_t s);
bool fwd_small_pays(const AttnParams& p, int max_splits);   // whether that kernel is the faster one (rows, cache, divisions at hand)
// Whether it divides the cache of `pairs` (batch, KV head) pairs, which saves a workgroup `saved` rounds of eight blocks.  A round takes
// about 1.8 us and the merge 4.3 (2, 4 and 5 rounds of one row tile 8.4, 12.1 and 14.0 us; a round each and a merge 10.6).  From about 7
// pairs for 16 CUs on undivided workgroups already read at nearly the memory's rate, and three rounds saved are less than the merge: us,
// whole -> divided, buffers in no cache, 128 pairs at 1336 / 1592 rows 21.3 -> 22.5 / 24.4 -> 24.8 (in one: 17.4 -> 20.2); 64 at 1080 16.5 -> 14.3, 96
// at 1592 22.9 -> 20.7.
inline bool small_divides(int pairs, int saved) { return 18 * saved > (16 * pairs > 7 * device_cus() ? 60 : 43); }
// dq_runs: NULL for all visible cache rows with weight 1; else runs of cache rows (ascending, disjoint), each with
// a positive weight (tile_begin is not used)
int launch_dq_bf16(const AttnParams& p, const SegTable* dq_runs, hipStream_t s);
int launch_dkdv_bf16(const AttnParams& p, const SegTable& seg, hipStream_t s);
// dQ (p.n_splits workgroups per row tile; runs as for launch_dq_bf16) and dK/dV in one launch
int launch_bwd_fused_bf16(const AttnParams& p, const SegTable& seg, const TailSplit& ts, bool kv_first, bool joined, const SegTable* runs, hipStream_t s);
// alone: not a call whose passes could share a launch but for what its outputs lie over (which takes that launch's products)
int launch_dq_bf16_now(const AttnParams& p, const SegTable* dq_runs, bool alone, hipStream_t s);
// its kernel in whole row tiles with 32x32x16 products (a translation unit of its own), for launches of so few rows that these are the
// faster ones: up to 0.72 of what a row tile on every CU holds (n_rows: over all heads and batches).  us, 16x16x32 -> 32x32x16
// products, of 160 calls of 100 - 256 whole tiles: 0.51 1041 rows at 4430 of 16/8 heads 100 -> 96; 0.52 two of 530 at 1322 of 16/2 42.0 ->
// 40.3; 0.63 643 at 4396 of 32/8 95 -> 92; 0.70 two of 719 at 10360 of 16/8 209 -> 202; but 0.74 two of 380 at 9644 of 32/8 186 ->
// 190; 0.83 1693 at 4482 of 16/8 117 -> 121; 0.88 899 at 6342 of 32/8 142 -> 149 (short causal ones up to 3 % either way).
inline bool dq_leaves_cus(int total, int64_t n_rows) { return total <= device_cus() && 25 * n_rows <= 18 * 128 * (int64_t)device_cus(); }
int launch_dq32_bf16(const AttnParams& p, const SegTable* dq_runs, int n_mtiles, int total, hipStream_t s);
// the same with the query rows taken from runs (p.C: number of rows that may be addressed from p.q / p.d_o)
int launch_dkdv_rows_bf16(const AttnParams& p, const SegTable& seg, const RowRuns& rr, hipStream_t s);
// the kernel of either with 32x32x16 products (its own translation unit)
int launch_dkdv32_bf16(const AttnParams& p, const SegTable& seg, const TailSplit& ts, const RowRuns& rr, Rows mode, hipStream_t s);
#ifndef SECO_DKDV_COLS
#define SECO_DKDV_COLS 128
#endif
constexpr int kColTileBf16 = SECO_DKDV_COLS;  // columns per workgroup in launch_dkdv_bf16

// Both gradients of a product in one launch (gemm_bf16.hip): whether the 32 x 64 tiles (`low`) of a data gradient whose contraction
// wavefronts divide become 64 x 64 ones (`tall`) beside `other` tiles of a weight gradient.  By itself the taller tile only leaves CUs
// idle; here those work on the other product, and an operand comes from the L2s, which bound both, a third less often (512 rows,
// 1024 x 4096: 134 for 201 MB).  They go in front, half of the chip for long, the weight gradient's tiles on the other half (behind those:
// 22.3 for 17.3 us).  us, 32 rows -> 64:
//   512 rows  1024 x 4096 19.1 -> 17.3   1024 x 2048 12.3 -> 10.6   1024 x 1536 10.4 -> 9.7   1024 x 512 7.0 -> 5.5
//   384 rows  1024 x 4096 16.8 -> 16.3   1024 x 1536  9.5 ->  8.6   1024 x 1024  7.9 -> 7.3
// What it gains first is a round: a workgroup has a CU to itself, and with fewer of them an XCD's 32 CUs are done in one round where they
// took two (530 random calls: time over that with low tiles 0.69 - 1.05, 0.84 on average).  With as many rounds as before it gains what the
// L2s deliver less, where the data gradient reads more than the weight gradient (a contraction of twice the rows), from 320 rows and an eighth of
// a round behind the first on, while the long workgroups are half of the CUs or fewer and the second round does not take a second half for
// a few more (207 calls 0.77 - 1.06, 0.91; the others 0.81 - 1.28, 1.01: 97 rows, 3520 x 1280 12.0 / 13.3; 1015, 448 x 1344 11.8 / 12.7; 331,
// 1408 x 2880 16.9 / 19.0).  Not with fewer tall tiles than three eighths of the CUs (320 rows, 1024 x 4096 15.3 / 15.9; 64 rows 11.6 / 15.5).
// (Each call timed behind large products: in short bursts everything is faster.)
inline bool taller_pays(int64_t rows, int64_t contraction, int64_t low, int64_t tall, int64_t other) {
  const int64_t cus = device_cus();
  auto per_xcd = [&](int64_t n) { return (n + 7) / 8 + (other + 7) / 8; };
  auto rounds = [&](int64_t n) { return (8 * per_xcd(n) + cus - 1) / cus; };
  if (8 * tall < 3 * cus) return false;
  const int64_t all = 64 * per_xcd(tall);
  return rounds(tall) < rounds(low) || (rows >= 320 && contraction >= 2 * rows && 2 * tall <= cus && all >= 9 * cus && all <= 12 * cus);
}

// Bandwidth-bound helpers; each takes a pair of tensors (gK and gV, keys and values) handled by one launch,
// a NULL member of the pair is skipped.
int launch_kvgrad_zero(float* ga, float* gb, int B, int H, int D, const int64_t gs[3], int64_t r0, int64_t r1,
                       hipStream_t s);
int launch_kvgrad_axpy(float* da, float* db, const float* sa, const float* sb, float scale, int B, int H, int D,
                       const int64_t gs[3], int64_t r0, int64_t r1, hipStream_t s);

// rows [r0, r0 + C) of a [B, H, *, D] array <- a [B, H, C, D] array (same element type, eb bytes per element)
int launch_rows_copy(void* da, void* db, const void* sa, const void* sb, int eb, int B, int H, int C, int D,
                     const int64_t dst_s[3], const int64_t src_s[3], int64_t r0, hipStream_t s);
// out[B, H, C, D] (bf16 or fp32) = scaler * g[rows r0 .. r0 + C) (fp32)
int launch_readout(void* oa, void* ob, const float* ga, const float* gb, float scaler, bool bf16, int B, int H, int C,
                   int D, const int64_t out_s[3], const int64_t gs[3], int64_t r0, hipStream_t s);

// out rows [out_r0, out_r0 + C) <- rotary embedding (or its inverse) of scale * in rows [in_r0, in_r0 + C), row r at
// position pos0 + r; in_kind / out_kind: SECO_F32 or SECO_BF16 (bf16 -> f32 is not needed and not provided).
// plain_out / plain_in: a second pair with the same strides and row ranges that is scaled and converted but not
// rotated, in the same launch; either pair may be NULL (skipped).
int launch_rope_rows(void* out, const void* in, void* plain_out, const void* plain_in, int in_kind, int out_kind, int B,
                     int H, int C, int D, const int64_t out_s[3], const int64_t in_s[3], int64_t out_r0, int64_t in_r0,
                     int64_t pos0, float base, bool inverse, float scale, hipStream_t s);

// Optional per-kernel timing (seco_profile_enable): a scope brackets one launch with HIP events
// on the launch stream.  Disabled by default; then a scope costs one branch.
enum KernelKind { kKernelFwd = 0, kKernelBwd, kKernelDq, kKernelDkdv, kKernelKvgrad, kKernelMerge, kKernelKinds };
struct ProfScope {
  ProfScope(KernelKind kind, hipStream_t s);
  ~ProfScope();
  hipStream_t stream;
  int slot;
};

inline int launch_status() { return hipGetLastError() == hipSuccess ? SECO_OK : SECO_ERR_LAUNCH; }

}  // namespace seco
