// dQ and dK/dV of a short call in one launch.
//
// A backward call with few rows and cache tiles is two passes of 10 - 25 us one after the other, each on a part of the chip
// and each with 6 - 9 us before its first product and behind its last.  The passes do not need each other's results: all
// that dK/dV takes from dQ are the row statistics, which are cheap enough to be computed twice for a short call (from the
// O and dO rows of a stage; OWN in bwd_dkdv_body.h).  So the workgroups of both are one grid, a third as many launches deep.
// A call among others with its merges, one pass after the other -> in one launch, in us (Hq/Hkv, chunk at position):
//   8/8  32 at 0     18.0 -> 10.1     32/8 128 at 1024   39.5 -> 26.9
//   8/8  32 at 1024  24.0 -> 14.9     32/8 256 at 0      31.6 -> 21.4
//   8/8 128 at 512   25.5 -> 16.1     32/8 256 at 2048   57.8 -> 47.0
//   16/2 184 at 736  40.1 -> 25.4     8/2  512 at 2048   48.5 -> 33.5
// What bounds it now: one workgroup's prologue, 1 - 10 iterations and epilogue, at one workgroup per CU.  With a round or more
// of column tiles one launch pays by what rounds_in_one_launch weighs (8/8 heads, 128 rows at 16256: 112 -> 95): bound then by
// the read-modify-write of gK and gV (with the reads of K and V 2.5 KiB per cache row and KV head, at 3.6 TB/s).
// dQ over selected columns (spaco_chunk_attn_bwd_sparse_dq) joins in wherever the dense pass would, in fewer shares; us, two launches
// of which dQ's was divided as for the whole cache -> one (Hq/Hkv, rows, chunks selected of all):
//   16/8 x 2  29, 2 of 64  24.5 -> 14.8     16/2 188, 8 of 35  51 -> 38
//   32/8  32, 2 of 64      28.1 -> 15.8     32/8 128, 4 of 32  41 -> 23
//   32/8 256, 4 of 16      51 -> 38         8/8   64, 8 of 64  25.4 -> 15.2
#include <cstddef>
#include <type_traits>

#include "bwd_dkdv_body.h"
#include "bwd_dq_body.h"
#include "merge_body.h"

namespace seco {
namespace {

using Cfg = DkdvCfg<kColTileBf16 / 32, SECO_DKDV_RB>;
constexpr int kNcb = kColTileBf16 / 32, kDqSmem = 4 * BNW * 2 * kRowBytes;
constexpr int kSmem = Cfg::kSmemBytes > kDqSmem ? Cfg::kSmemBytes : kDqSmem;
static_assert(offsetof(TailSplit, plan.tile_of) % 4 == 0 && offsetof(TailSplit, plan.first) % 4 == 0, "tables read in words");
static_assert(Cfg::kThreads == 512, "both passes in workgroups of 8 wavefronts");

// The first first_grid workgroups are those of dK/dV (kv_first: the pass with the longer workgroups) or of dQ; both numbers are rounded up to whole XCD rounds.
// RUNS: nothing, or the SegTable of dQ over selected columns
struct AllColumns {};
template <bool SPLIT, typename RUNS, Rows MODE>
__global__ __launch_bounds__(512, 2) void bwd_fused_bf16_kernel(AttnParams p, SegTable seg, TailSplit ts, int n_mtiles,
                                                                int kv_total, int dq_total, int first_grid, int kv_first, RUNS runs) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds_char* smem = (lds_char*)smem_raw;
  const bool first = (int)blockIdx.x < first_grid, kv = first == (kv_first != 0);
  const int item = xcd_item(first ? blockIdx.x : blockIdx.x - first_grid, kv ? kv_total : dq_total);
  if (item < 0) return;
  if (kv) {
    RowRuns none;
    none.n = 0;
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x / (64 * kNcb)) == 0)
      dkdv_bf16_body<kNcb, SECO_DKDV_RB, MODE, 0, Products32, true>(p, seg, ts, none, item, smem);
    else
      dkdv_bf16_body<kNcb, SECO_DKDV_RB, MODE, 1, Products32, true>(p, seg, ts, none, item, smem);
  } else {
    constexpr int kSplit = SPLIT ? kDivided : kWholeTiles;
    if constexpr (std::is_same_v<RUNS, SegTable>)
      dq_bf16_body<2, kSplit, true, DqProducts16, true>(p, runs, n_mtiles, item, smem);
    else
      dq_bf16_body<2, kSplit, false, DqProducts16, true>(p, seg, n_mtiles, item, smem);
  }
}

// Both merges: the first n_tail workgroups add up shared-out column tiles, the others rows of dQ.  (Two launches of 4 - 6 us
// each one behind the other otherwise.)
template <int GP, int K>
__global__ __launch_bounds__(256) void bwd_merge_kernel(AttnParams p, SegTable seg, TailSplit ts, int n_tail) {
  if ((int)blockIdx.x < n_tail)
    tail_merge_body<kColTileBf16>(p, seg, ts, blockIdx.x);
  else
    dq_merge_body<GP, K>(p, blockIdx.x - n_tail);
}

int launch_merges(const AttnParams& p, const SegTable& seg, const TailSplit& ts, hipStream_t s) {
  const int n_tail = ts.plan.n_shared > 0 ? (int)tail_merge_grid<kColTileBf16>(p, ts) : 0;
  if (n_tail == 0) return p.n_splits > 1 ? launch_dq_merge(p, s) : SECO_OK;
  const int64_t R = p.n_splits > 1 ? (int64_t)p.B * p.Hq * p.C : 0;
  ProfScope prof(kKernelMerge, s);
  auto go = [&](auto kern, int rows) {
    hipLaunchKernelGGL(kern, dim3((unsigned)(n_tail + (R + rows - 1) / rows)), dim3(256), 0, s, p, seg, ts, n_tail);
  };
  if (p.n_splits <= 2) go(bwd_merge_kernel<1, 2>, 8);       // (the forms of launch_dq_merge)
  else if (p.n_splits <= 4) go(bwd_merge_kernel<1, 4>, 8);
  else if (p.n_splits <= 8) go(bwd_merge_kernel<1, 8>, 8);
  else if (p.n_splits <= 16) go(bwd_merge_kernel<2, 8>, 4);
  else if (p.n_splits <= 32) go(bwd_merge_kernel<4, 8>, 2);
  else go(bwd_merge_kernel<8, 8>, 1);
  return launch_status();
}

template <bool SPLIT, typename RUNS, Rows MODE>
int launch(const AttnParams& p, const SegTable& seg, const TailSplit& ts, const RUNS& runs, int n_mtiles, int kv_total, int dq_total,
           bool kv_first, hipStream_t s) {
  auto kern = bwd_fused_bf16_kernel<SPLIT, RUNS, MODE>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), kSmem)) return SECO_ERR_LAUNCH;
  AttnParams pl = for_launch(p, n_mtiles);
  for_column_tiles(pl, seg, ts);
  const int first = xcd_grid(kv_first ? kv_total : dq_total), second = xcd_grid(kv_first ? dq_total : kv_total);
  {
    ProfScope prof(kKernelBwd, s);
    hipLaunchKernelGGL(kern, dim3(first + second), dim3(512), kSmem, s, pl, seg, ts, n_mtiles, kv_total, dq_total, first,
                       kv_first ? 1 : 0, runs);
  }
  return launch_status();
}

}  // namespace

int launch_bwd_fused_bf16(const AttnParams& p, const SegTable& seg, const TailSplit& ts, bool kv_first, bool joined, const SegTable* runs, hipStream_t s) {
  const int kv_total = p.B * p.Hkv * (seg.tile_begin[seg.n] - ts.plan.n_tiles + ts.plan.n_entries);
  const SplitPlan plan = split_plan(p.B, p.Hkv, p.G, p.C);
  const int mtiles = (p.C + BM - 1) / BM;
  const AllColumns all;
  const int whole = p.B * p.Hq * mtiles, divided = plan.items * p.n_splits;
  auto go = [&](auto mode) {
    constexpr Rows kMode = decltype(mode)::value;
    if (p.n_splits == 1)
      return runs ? launch<false, SegTable, kMode>(p, seg, ts, *runs, mtiles, kv_total, whole, kv_first, s)
                  : launch<false, AllColumns, kMode>(p, seg, ts, all, mtiles, kv_total, whole, kv_first, s);
    return runs ? launch<true, SegTable, kMode>(p, seg, ts, *runs, plan.n_mtiles, kv_total, divided, kv_first, s)
                : launch<true, AllColumns, kMode>(p, seg, ts, all, plan.n_mtiles, kv_total, divided, kv_first, s);
  };
  const int rc = joined ? go(std::integral_constant<Rows, kJoined>()) : go(std::integral_constant<Rows, kAll>());
  return rc ? rc : launch_merges(p, seg, ts, s);
}

}  // namespace seco
