// How a bf16 backward call is laid out (host arithmetic only): whether dQ and dK/dV run in one launch, in how many shares a row
// tile of dQ goes, and which column tiles of dK/dV are shared out.
#pragma once
#include <algorithm>

#include "seco_internal.h"

namespace seco {
namespace {

constexpr size_t kSlotBytes = (size_t)2 * kColTileBf16 * 128 * sizeof(float);
int slots_in(size_t bytes) { return (int)std::min(bytes / kSlotBytes, (size_t)device_cus()); }

// Iterations of the last column tiles
template <typename Cfg, bool ROWS>
IterRuns tile_iterations(const AttnParams& p, const SegTable& seg, const RowRuns& rr, bool joined = false) {
  // iterations of a column tile (as the kernel counts them)
  auto iters = [&](int tile) {
    int si = 0;
    while (si + 1 < seg.n && tile >= seg.tile_begin[si + 1]) ++si;
    const int c0 = seg.col_begin[si] + (tile - seg.tile_begin[si]) * Cfg::kCols;
    const int r0 = (c0 > p.q_start ? c0 - p.q_start : 0) / Cfg::kBQ * Cfg::kBQ;
    if (!ROWS) return joined ? ((p.C - r0) * p.G + Cfg::kBQ - 1) / Cfg::kBQ : ((p.C - r0 + Cfg::kBQ - 1) / Cfg::kBQ) * p.G;
    int n = 0;
    for (int i = 0; i < rr.n; ++i)
      if (rr.end[i] > r0) n += (rr.end[i] - (rr.begin[i] > r0 ? rr.begin[i] : r0) + Cfg::kBQ - 1) / Cfg::kBQ;
    return n * p.G;
  };
  return iter_runs(seg.tile_begin[seg.n], iters);
}

// Whether the stages of dK/dV cut the rows of a group's heads one behind the other (kJoined): by the part of the iterations that
// saves.  From a quarter of a round of column tiles on, three in ten; with fewer tiles, whose iterations workgroups share out so that
// less is gained from fewer of them than addresses and positions per row cost, two thirds, or half of four or less, which are not
// shared out.  15700 random calls of 1 - 1000 rows, time joined over time apart, by the part saved: more than 70 % 0.47 - 1.11, 0.74 on
// average; 35 - 70 % 0.60 - 1.08, 0.90; 30 - 35 % 0.77 - 1.17, 0.96; of those not taken 0.59 - 1.43, 0.99.  us, apart -> joined:
//   32/8 heads  32 at 16352: 87.4 -> 75.4   16 at 8000: 48.0 -> 36.8   16/8 x 2  14 at 6000: 51.9 -> 47.6
//   16/2  9 at 900: 17.0 -> 13.9   70 at 20000: 94.2 -> 64.4
// A dK/dV pass of its own, with its row statistics at hand and one and a half rounds of tiles or more: a tenth (330 of the calls: 0.88 -
// 1.10, 0.96 on average).  150 at 16000 of 32/8 178.3 -> 172.0.
inline bool joined_pays(const AttnParams& p, const SegTable& seg, bool apart_from_dq = false) {
  const int64_t rows = (int64_t)p.C * p.G, apart = (int64_t)(p.C + 63) / 64 * p.G, saved = apart - (rows + 63) / 64;
  // (a group's rows are addressed by 32-bit offsets)
  if (rows > 1 << 24) return false;
  for (const int64_t* s : {p.qs, p.os})
    if (p.G * s[1] + p.C * s[2] >= (int64_t)1 << 31) return false;
  if (3 * saved >= 2 * apart || (apart <= 4 && 2 * saved >= apart)) return true;
  const int64_t tiles = (int64_t)p.B * p.Hkv * seg.tile_begin[seg.n];
  if (apart_from_dq && 10 * saved >= apart && 2 * tiles >= 3 * device_cus()) return true;
  return 10 * saved >= 3 * apart && 4 * tiles >= device_cus();
}

// Both passes of a dense call: in one launch with dq_splits workgroups per row tile for dQ (0: one after the other), and
// the column tiles that are shared out.
struct BwdPlan {
  int dq_splits;
  bool kv_first, joined;
  TailSplit ts;
  float busy;        // of the CUs, in dK/dV by itself (share_plan)
};
// Column tiles for a round or more (n_kv of them, iters iterations each): in how many shares a row tile of dQ joins them
// in one launch, dQ first; 0: not.  The column tiles of a round all start together and reach the read-modify-write of
// gK / gV together, and the last round is seldom full; dQ's workgroups, of another length, fill it and put them out of step.
// Against it stand the row statistics, computed anew in every iteration.  So: up to 4 iterations; up to 8 behind more than a round, but
// for four full rounds or more and nothing behind them; up to 12 where a last round leaves a tenth of all rounds' time or more, or where
// dQ's row tiles are half of the CUs or more, so that its own round leaves CUs without work.  Beyond 4 iterations those tiles, whole in one
// launch, may hold padding that they do not hold packed and divided: with two fifths more of them, from 9 iterations on three in ten,
// only where the last round leaves three tenths or more.  5200 calls of 4 - 2400 rows on 256 - 3700 tiles and 2100 with padding, time of one launch
// over that of two: up to 4 iterations 0.55 - 0.99; 5 - 8 0.62 - 1.10, 0.90 on average, with that padding 0.98 - 1.30, 1.14 (three tenths
// left or more 0.73 - 1.01, 0.88); 9 - 12 0.74 - 1.18, 0.93, with padding 0.84 - 1.22, 1.05 (0.75 - 1.03, 0.95), others 0.87 - 1.17, 1.00; 13 - 16 0.82 - 1.22, 1.03.
// Shares: the fewest that end within 0.9 of the time the column tiles take (few workgroups, few partial sums).  Of 1 to 1.25 rounds the last
// leaves most CUs to dQ: an empirical 1.55 rounds, as long as the CUs without dQ's workgroups hold all column tiles in two (time over that
// with the rounds there are, 5 - 8 iterations: 0.86 - 1.18, 0.97 on average; where they do not 0.87 - 1.16, 1.06), and with 7 or 8 iterations
// only up to a sixteenth of the second round if its tiles are shared out (beyond it 0.86 - 1.18, 1.00, but some calls longer than in two
// launches); more shares than that leave few CUs to the first column tiles (66 rows at 4663 of 48/8 heads, 240 workgroups for 160: 55 -> 69 us).
// Two launches -> one, us:
//   32/8 heads  32 at 16256: 103 -> 75   64 at 8128: 64 -> 52   128 at 8064: 83 -> 75   128 at 14000: 139 -> 124
//   8/8  128 at 4000: 43 -> 32           16/8  256 at 8000: 92 -> 79                    16/2  64 at 32000: 105 -> 82
// row_tiles, whole: those of dQ packed, and whole in one launch; shared: whether column tiles are shared out
inline int rounds_in_one_launch(int n_kv, int iters, int tiles, int max_splits, int row_tiles, int whole, bool shared) {
  const int cus = device_cus(), full = n_kv / cus, rest = n_kv % cus;
  auto left_over = [&](int tenths) { return rest > 0 && 10 * (cus - rest) >= tenths * cus * (full + 1); };
  const bool pays = iters <= 4 || (n_kv > cus && (iters <= 8 ? rest > 0 || full < 4 : iters <= 12 && (left_over(1) || 2 * row_tiles > cus)));
  if (!pays) return 0;
  auto shares = [&](float rounds) {
    int n = 1;
    while (n < max_splits && kDqFrontTime.of((tiles + n - 1) / n) > 0.9f * rounds * kDkdvRoundTime.of(iters)) ++n;
    return n;
  };
  const bool few_behind = 4 * n_kv < 5 * cus;
  int n = shares(few_behind ? 1.55f : (float)n_kv / cus);
  if (few_behind && iters <= 8 && (2 * (cus - (n > 1 ? n * row_tiles : whole)) < n_kv || (iters > 6 && shared && 16 * n_kv > 17 * cus)))
    if (const int more = shares((float)n_kv / cus); 16 * more * row_tiles < 15 * cus) n = more;
  const bool padded = n == 1 && 10 * whole > (iters <= 8 ? 14 : 13) * row_tiles;
  return padded && iters > 4 && !left_over(3) ? 0 : n;
}

// When the last of a row of workgroups ends on `places` that take them in order: the places by the time they are free at, those
// within a quarter of a microsecond as one.
class Schedule {
 public:
  static constexpr int kMost = 64;
  explicit Schedule(int places) : first_(0), end_(1) { at_[0] = 0.f, of_[0] = places; }
  void run(float time, int count) {
    while (count > 0) {
      const int k = std::min(of_[first_], count);
      const float t = at_[first_] + time;
      count -= k;
      if ((of_[first_] -= k) == 0) ++first_;
      int i = end_;
      while (i > first_ && at_[i - 1] > t + 0.25f) --i;
      if (i > first_ && at_[i - 1] >= t - 0.25f) {
        of_[i - 1] += k;
        continue;
      }
      if (end_ == kRoom) {                     // (there are at most kMost groups)
        std::copy(at_ + first_, at_ + end_, at_);
        std::copy(of_ + first_, of_ + end_, of_);
        i -= first_, end_ -= first_, first_ = 0;
      }
      for (int j = end_++; j > i; --j) at_[j] = at_[j - 1], of_[j] = of_[j - 1];   // (few: most end last)
      at_[i] = t, of_[i] = k;
    }
  }
  float end() const { return at_[end_ - 1]; }

 private:
  static constexpr int kRoom = 4 * kMost;
  float at_[kRoom];
  int of_[kRoom], first_, end_;                // groups [first_, end_)
};

// Fewer column tiles than a round, but more workgroups in all than fit at once: the plan of sharing out the column tiles with
// which both passes in one launch, dK/dV first, dQ in whole row tiles behind it, are expected to end before the two would
// one after the other; false: none.  Both are laid out workgroup by workgroup on the compute units of an XCD (whole units
// of a batch and KV head each, in the order of the items).  The times, in microseconds, are fitted to 74 shapes of 130 - 3200
// rows (3 - 4 % off); one launch where it comes out 5 % ahead, and below 200 us, from where gains and errors were both about 3 %.
// Of 400 other random shapes with less than a round of column tiles it takes 76, 1.13 times as fast, none more than 1 %
// slower; two -> one, us:
//   32/8  745 at 0: 50.9 -> 39.1   873 at 0: 55.9 -> 43.2   1482 at 445: 134.5 -> 131   16/8  1174 at 0: 58 -> 45
//   8/8  2156 at 5: 84.9 -> 63.9   x 2  1011 at 96: 58.6 -> 40.9
// The search itself takes 0.3 - 1.1 us of the host (745 rows 0.6, 1174 1.1; two sequences of 400 at 100, where it finds nothing,
// 0.3), beside 3 of a launch: three in four calls that reach it are taken, and a bound on the time from the work alone tells
// one in fifty of the others, so there is none.
bool one_launch_behind_column_tiles(const AttnParams& p, const IterRuns& runs, int n_ctiles, int slots, const SharePlan& apart_plan,
                                    SharePlan& one_plan) {
  const int n_units = p.B * p.Hkv, places = device_cus() / 8, mtiles = (p.C + 127) / 128, heads = p.B * p.Hq / 8;
  const int row_wgs = p.B * p.Hq * mtiles;
  if (n_units % 8 != 0 || places > Schedule::kMost || row_wgs >= 2 * device_cus()) return false;
  if (row_wgs > device_cus() && p.q_start >= 2 * p.C) return false;      // (row_shares divides dQ's second round)
  // fit: workgroups of both passes one after the other and in one launch, what overlaps between launches, a share in a merge
  constexpr WgTime kKv{14.9f, 1.7f}, kKvOne{15.7f, 1.8f}, kDq{7.1f, 1.7f}, kDqOne{8.2f, 2.4f};
  constexpr float kAroundApart = -1.6f, kAroundOne = -4.7f, kShareApart = 0.03f, kShareOne = 0.024f, kShareDq = 0.02f;
  auto column_tiles = [&](Schedule& sc, const SharePlan& plan, WgTime wg) {
    for (int u = 0; u < n_units / 8; ++u) {
      int listed = plan.n_tiles - n_ctiles;                              // position in the list of the next tile, once not negative
      for (int r = 0; r < runs.n; ++r) {
        const int whole = std::clamp(-listed, 0, runs.count[r]), shared = runs.count[r] - whole;
        sc.run(wg.of(runs.iters[r]), whole);
        listed += whole;
        if (shared > 0) {                                                // (tiles of equal length have equally many shares)
          const int k = plan.first[listed + 1] - plan.first[listed];
          sc.run(wg.wg + wg.step * runs.iters[r] / k, k * shared);
          listed += shared;
        }
      }
    }
  };
  auto row_tiles = [&](Schedule& sc, WgTime wg) {
    for (int mt = mtiles; mt > 0; --mt) sc.run(wg.of((p.q_start + std::min(mt * 128, p.C) + 127) / 128), heads);
  };
  auto merge = [&](const SharePlan& plan, float each) { return plan.n_shared > 0 ? kMergeLaunch + each * plan.first[plan.n_shared] * n_units : 0.f; };
  Schedule kv(places);
  column_tiles(kv, apart_plan, kKv);
  float apart = kv.end() + merge(apart_plan, kShareApart) + kAroundApart;
  if (p.n_splits > 1) {
    const int wgs = split_plan(p.B, p.Hkv, p.G, p.C).items * p.n_splits, tiles = (p.q_start + p.C + 127) / 128;
    apart += (wgs + device_cus() - 1) / device_cus() * kDq.of((tiles + p.n_splits - 1) / p.n_splits) + kMergeLaunch + kShareDq * wgs;
  } else {
    Schedule dq(places);
    row_tiles(dq, kDq);
    apart += dq.end();
  }
  if (apart > 200.f) return false;
  float best = apart / 1.05f;
  int last = -1;
  bool found = false;
  const int cus[3] = {96 * device_cus() / 256, 160 * device_cus() / 256, device_cus()};
  ShareChoice choices[3];
  choose_shares(runs, n_ctiles, n_units, cus, slots, 1, false, kDkdvOwnTime, choices);
  for (const ShareChoice& c : choices) {
    if (c.time < 0.f || c.per == last) continue;
    last = c.per;
    const SharePlan plan = make_shares(runs, n_ctiles, c.per);
    Schedule both(places);
    column_tiles(both, plan, kKvOne);
    row_tiles(both, kDqOne);
    const float t = both.end() + merge(plan, kShareOne) + kAroundOne;
    if (t < best) {
      best = t;
      one_plan = plan;
      found = true;
    }
  }
  return found;
}

// With column tiles for less than a round, one launch is taken when all workgroups of both passes fit the chip at one per
// CU and the longer pass, with the extra work, is expected to end before the two would one after the other: with more
// workgroups than CUs the two halves of the grid would queue behind each other on some CUs (16/2 heads, chunk 704 at 5632:
// 7% slower in one launch).  The passes divide the CUs: for every number of shares of a dQ row tile the column tiles are
// shared out over the rest (kDqBesideTime, kDkdvOwnTime).
// dq: the dQ pass is still to go out, so that it may share the launch (it goes with the first table of more runs than one holds)
template <typename Cfg>
BwdPlan plan_both(const AttnParams& p, const SegTable& seg, bool dq) {
  const int cus = device_cus(), n_units = p.B * p.Hkv, n_ctiles = seg.tile_begin[seg.n];
  RowRuns none;
  none.n = 0;
  BwdPlan best;
  best.joined = joined_pays(p, seg);
  const IterRuns runs = tile_iterations<Cfg, false>(p, seg, none, best.joined);
  best.dq_splits = 0;
  best.kv_first = true;
  best.ts.part = p.tail_part;
  float kv_alone = 0.f;
  best.ts.plan = share_plan(runs, n_units, n_ctiles, p.G, p.C, slots_in(p.tail_bytes), kv_alone, &best.busy);
  if (!dq) return best;
  const SplitPlan sp = split_plan(p.B, p.Hkv, p.G, p.C);
  const int tiles = (p.q_start + p.C + 127) / 128;
  const size_t dq_bytes = (size_t)p.B * p.Hq * p.C * 128 * sizeof(float);
  auto dq_wgs = [&](int n) { return n > 1 ? sp.items * n : p.B * p.Hq * ((p.C + 127) / 128); };
  auto dq_part = [&](int n) { return n > 1 ? (n * dq_bytes + 255) / 256 * 256 : (size_t)0; };
  if ((int64_t)n_units * n_ctiles >= cus) {
    if (sp.items >= cus) return best;
    const int n = rounds_in_one_launch(n_units * n_ctiles, runs.iters[0], tiles, p.n_splits, sp.items, dq_wgs(1), best.ts.plan.n_shared > 0);
    if (n > 0 && dq_part(n) <= p.tail_bytes) {
      best.dq_splits = n;
      best.kv_first = false;
      best.ts.part = p.tail_part + dq_part(n) / sizeof(float);
      best.ts.plan = share_plan(runs, n_units, n_ctiles, p.G, p.C, slots_in(p.tail_bytes - dq_part(n)), kv_alone, &best.busy);
    }
    return best;
  }
  auto dq_time = [&](int n) { return kDqBesideTime.of((tiles + n - 1) / n); };
  auto merge_time = [&](int n) { return n > 1 ? kMergeLaunch + 0.02f * dq_wgs(n) : 0.f; };
  float best_t = (dq_wgs(p.n_splits) + cus - 1) / cus * dq_time(p.n_splits) + merge_time(p.n_splits) + kv_alone + 2.f;   // (2: between the launches)
  int per = 0;
  for (int n = 1; n <= p.n_splits && dq_wgs(n) + n_units * n_ctiles <= cus; ++n) {
    const size_t used = dq_part(n);
    if (used > p.tail_bytes) break;
    const ShareChoice c = choose_shares(runs, n_ctiles, n_units, cus - dq_wgs(n), slots_in(p.tail_bytes - used), 1, true, kDkdvOwnTime);
    // (both merges are one launch)
    const float t = std::max(dq_time(n), c.longest) + (c.time - c.longest) + (n > 1 ? merge_time(n) - (c.per ? kMergeLaunch : 0.f) : 0.f);
    if (c.time >= 0.f && t < best_t) {
      best_t = t;
      best.dq_splits = n;
      best.kv_first = c.longest >= dq_time(n);
      best.ts.part = p.tail_part + used / sizeof(float);
      per = c.per;
    }
  }
  if (best.dq_splits > 0) {
    best.ts.plan = make_shares(runs, n_ctiles, per);
  } else if (SharePlan plan; n_ctiles <= runs.n_tiles && one_launch_behind_column_tiles(p, runs, n_ctiles, slots_in(p.tail_bytes), best.ts.plan, plan)) {
    best.dq_splits = 1;
    best.ts.plan = plan;
  }
  return best;
}

template <typename Cfg>
BwdPlan plan_bwd(const AttnParams& p, const SegTable& seg, bool dq) {
  BwdPlan plan = plan_both<Cfg>(p, seg, dq);
  if (plan.dq_splits == 0 && !plan.joined && joined_pays(p, seg, true)) {
    RowRuns none;
    none.n = 0;
    float time;
    plan.joined = true;
    plan.ts.plan = share_plan(tile_iterations<Cfg, false>(p, seg, none, true), p.B * p.Hkv, seg.tile_begin[seg.n], p.G, p.C,
                              slots_in(p.tail_bytes), time, &plan.busy);
  }
  return plan;
}

// dQ over selected columns takes the place of n shares per row tile of the dense pass: as many as keep a share's length,
// and whole row tiles only where those are no more workgroups
int sparse_shares(const AttnParams& p, const SegTable& runs, int n) {
  const int tiles = (p.q_start + p.C + 127) / 128, m = std::max(1, (visited_tiles(p, runs) * n + tiles - 1) / tiles);
  if (n == 1 || m > 1) return std::min(m, n);
  return p.B * p.Hq * ((p.C + 127) / 128) <= n * split_plan(p.B, p.Hkv, p.G, p.C).items ? 1 : 2;
}

}  // namespace
}  // namespace seco
