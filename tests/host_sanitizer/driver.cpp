// Host side of the C ABI under AddressSanitizer + UndefinedBehaviorSanitizer (CPU only; built and run by
// tests/test_host_sanitizer.py).  The kernel launchers are recording stubs, so the device pointers below are fake
// and never dereferenced; what runs for real is everything the entry points do before a launch: validation, the
// column-segment tables of the dK/dV pass, the run tables of the column-weighted dQ and of the transposed order,
// the workspace layout, chunk selection and the weight vectors.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "bwd_plan.h"
#include "fast_div.h"
#include "seco.h"
#include "stub_launch.h"
#include "xcd_map.h"

#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      std::fprintf(stderr, "%s:%d: CHECK failed: %s\n", __FILE__, __LINE__, #cond); \
      std::exit(1);                                                        \
    }                                                                      \
  } while (0)

static seco_desc desc(int dtype = SECO_BF16, int C = 256, int q_start = 256, int Hq = 4, int Hkv = 2, int D = 128) {
  seco_desc d;
  std::memset(&d, 0, sizeof(d));
  d.batch = 1; d.n_q_heads = Hq; d.n_kv_heads = Hkv; d.head_dim = D;
  d.chunk_len = C; d.q_start = q_start; d.dtype = dtype; d.softmax_scale = 0.088f;
  int64_t* ss[4] = {d.q_stride, d.o_stride, d.kv_stride, d.g_stride};
  for (auto s : ss) { s[0] = (int64_t)Hq << 22; s[1] = (int64_t)1 << 22; s[2] = D; }
  return d;
}

struct Cfg { static constexpr int kCols = 128, kBQ = 64; };   // (of the dK/dV kernel)

static void* const FAKE = reinterpret_cast<void*>(0x10000);
static float* const FAKEF = reinterpret_cast<float*>(0x10000);

// Calls named on the command line (joined_shapes.py), which the rules are to plan with stages of several heads' rows (kJoined):
// d:B,Hq,Hkv,C,q_start dense; g:...,later rows the transposed order; s:B,Hq,Hkv,C,chunks,selected... dQ over those; w:...,chunks... dK/dV
// over those.  Between them they have to reach every form of the kernel.
struct Forms {
  bool divided, whole, apart16, apart32, shared_one, shared_apart, late_one, late_apart, late_gather, selected_divided, selected_whole;
};
static void check_joined(const char* arg, Forms& seen) {
  std::vector<int> v;
  for (const char* c = arg + 1; *c; c += std::strcspn(c, ",")) v.push_back(std::atoi(++c));
  const char kind = arg[0];
  const bool chunks = kind == 's' || kind == 'w';
  const int C = v[3], n = chunks ? v[4] : 1, q_start = chunks ? (n - 1) * C : v[4];
  seco_desc d = desc(SECO_BF16, C, q_start, v[1], v[2]);
  d.batch = v[0];
  const size_t bytes = seco_workspace_bytes(&d, SECO_OP_BWD);
  std::vector<float> w(n, kind == 'w' ? 0.f : 1.f), wq(n, 0.f);
  for (size_t i = 5; i < v.size() && chunks; ++i) (kind == 's' ? wq : w)[v[i]] = 1.f + i;
  w[n - 1] = wq[n - 1] = 1.f;
  const int rc =
      kind == 'g'   ? seco_chunk_attn_bwd_gather(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKEF, (q_start + C + v[5] + 3) / 4 * 4,
                                                 v[5], FAKE, bytes, nullptr)
      : kind == 'd' ? seco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKE, bytes, nullptr)
      : kind == 's' ? spaco_chunk_attn_bwd_sparse_dq(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, w.data(), wq.data(), n, C, FAKE,
                                                     bytes, nullptr)
                    : spaco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, w.data(), n, C, FAKE, bytes, nullptr);
  CHECK(rc == SECO_OK);
  const seco::AttnParams& p = g_stub.last;
  const seco::SegTable& seg = g_stub.dkdv_tables.back();
  const seco::BwdPlan plan = seco::plan_bwd<Cfg>(p, seg, kind != 'g');
  if (!plan.joined) std::fprintf(stderr, "%s: stages of one head each\n", arg);
  CHECK(plan.joined);
  // (late: the last column tile begins a stage or more behind the chunk's first row)
  const int begin = seg.col_begin[seg.n - 1], last = begin + (seg.col_end[seg.n - 1] - begin - 1) / Cfg::kCols * Cfg::kCols;
  const bool late = last >= p.q_start + Cfg::kBQ, one = plan.dq_splits > 0, shared = plan.ts.plan.n_shared > 0;
  if (kind == 'g') {
    seen.late_gather |= late;
  } else if (kind == 's') {
    CHECK(one);
    (seco::sparse_shares(p, g_stub.dq_tables.back(), plan.dq_splits) > 1 ? seen.selected_divided : seen.selected_whole) = true;
  } else if (kind == 'd') {
    (one ? (plan.dq_splits > 1 ? seen.divided : seen.whole) : plan.busy >= 0.74f ? seen.apart16 : seen.apart32) = true;   // (kBusy)
    if (shared) (one ? seen.shared_one : seen.shared_apart) = true;
    if (late) (one ? seen.late_one : seen.late_apart) = true;
  }
}

int main(int argc, char** argv) {
  Forms seen{};
  for (int i = 1; i < argc; ++i) check_joined(argv[i], seen);
  CHECK(argc == 1 || (seen.divided && seen.whole && seen.apart16 && seen.apart32 && seen.shared_one && seen.shared_apart && seen.late_one &&
                      seen.late_apart && seen.late_gather && seen.selected_divided && seen.selected_whole));
  // ---- division by multiplication: around every multiple that can go wrong, up to the largest dividend ----
  for (int d : {1, 2, 3, 5, 7, 31, 32, 33, 255, 640, 641, 4095, 65537, 16777213, 1 << 30, (1 << 30) + 1, 0x7fffffff}) {
    const seco::Div by = seco::make_div(d);
    for (int64_t k : {(int64_t)0, (int64_t)1, (int64_t)2, (int64_t)97, (int64_t)0x7fffffff / d / 2, (int64_t)0x7fffffff / d})
      for (int64_t n = k * d - 2; n <= k * d + 2; ++n)
        if (n >= 0 && n <= 0x7fffffff) CHECK(seco::over((int)n, by) == (int)(n / d));
    CHECK(seco::over(0x7fffffff, by) == 0x7fffffff / d);
  }
  // ---- validation codes (nothing may be launched) ----
  {
    seco_desc d = desc();
    g_stub.clear();
    seco_desc bad = d; bad.dtype = 7;
    CHECK(seco_chunk_attn_fwd(&bad, FAKE, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_ERR_DTYPE);
    bad = d; bad.n_q_heads = 3;
    CHECK(seco_chunk_attn_fwd(&bad, FAKE, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_ERR_SHAPE);
    bad = d; bad.head_dim = 96;
    CHECK(seco_chunk_attn_fwd(&bad, FAKE, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_ERR_HEAD_DIM);
    bad = d; bad.q_stride[2] = 132;
    CHECK(seco_chunk_attn_fwd(&bad, FAKE, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_ERR_ALIGN);
    bad = d; bad.q_start = 1 << 30;
    CHECK(seco_chunk_attn_fwd(&bad, FAKE, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_ERR_TOO_LARGE);
    bad = d; bad.softmax_scale = NAN;
    CHECK(seco_chunk_attn_fwd(&bad, FAKE, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_ERR_SHAPE);
    CHECK(seco_chunk_attn_fwd(&d, nullptr, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_ERR_NULL);
    CHECK(seco_chunk_attn_fwd(nullptr, FAKE, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_ERR_NULL);
    CHECK(seco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, nullptr, 0, nullptr) ==
          SECO_ERR_WORKSPACE);
    CHECK(seco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKE, 16, nullptr) ==
          SECO_ERR_WORKSPACE);
    CHECK(seco_workspace_bytes(&bad, SECO_OP_BWD) == (size_t)-1);
    CHECK(seco_workspace_bytes(&d, 99) == (size_t)-1);
    CHECK(kvgrad_zero(&d, FAKEF, FAKEF, 5, 4, nullptr) == SECO_ERR_RANGE);
    CHECK(kvgrad_accumulate(&d, FAKEF, nullptr, FAKEF, nullptr, 1.f, 0, 4, nullptr) == SECO_ERR_RANGE);   // aliasing
    CHECK(g_stub.fwd + g_stub.dq + g_stub.dkdv + g_stub.zero + g_stub.axpy == 0);
  }
  // ---- dense backward: one segment over all visible rows; forward with and without the split workspace ----
  {
    seco_desc d = desc(SECO_BF16, 256, 768);               // kv_len 1024 = 8 column tiles of 128
    const size_t ws = seco_workspace_bytes(&d, SECO_OP_BWD);
    CHECK(ws != (size_t)-1 && ws > 0);
    g_stub.clear();
    CHECK(seco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKE, ws, nullptr) == SECO_OK);
    CHECK(g_stub.dq == 1 && g_stub.dkdv == 1 && g_stub.dq_tables.empty());
    const seco::SegTable& t = g_stub.dkdv_tables[0];
    CHECK(t.n == 1 && t.col_begin[0] == 0 && t.col_end[0] == 1024 && t.weight[0] == 1.f && t.tile_begin[1] == 8);
    CHECK(g_stub.last.n_splits > 1);                        // a short chunk: the cache range is divided
    g_stub.clear();
    CHECK(seco_chunk_attn_fwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, nullptr, 0, nullptr) == SECO_OK);
    CHECK(g_stub.fwd == 1 && g_stub.last.n_splits == 1);    // no workspace: direct path
    const size_t wf = seco_workspace_bytes(&d, SECO_OP_FWD);
    CHECK(seco_chunk_attn_fwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, wf, nullptr) == SECO_OK);
    CHECK(g_stub.last.n_splits > 1);
    // row tiles between one and two rounds: divided only with all of an aligned workspace
    const seco_desc sh = desc(SECO_BF16, 700, 2900, 48, 16);
    const size_t wsh = seco_workspace_bytes(&sh, SECO_OP_FWD);
    CHECK(wsh > 0);
    for (const int off : {0, 16, -1}) {                     // whole, misaligned, one byte short
      CHECK(seco_chunk_attn_fwd(&sh, FAKE, FAKE, FAKE, FAKE, FAKEF, static_cast<char*>(FAKE) + std::max(off, 0), wsh + std::min(off, 0),
                                nullptr) == SECO_OK);
      CHECK((g_stub.last.tail_bytes > 0) == (off == 0) && (g_stub.last.part != nullptr) == (off == 0) && g_stub.last.n_splits == 1);
    }
    // the same call on the library's own scratch array
    g_stub.clear();
    CHECK(seco_chunk_attn_bwd_noalloc(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, nullptr) == SECO_OK);
    CHECK(g_stub.dq == 1 && g_stub.dkdv == 1 && g_stub.last.delta != nullptr);
    CHECK((reinterpret_cast<uintptr_t>(g_stub.last.delta) & 255u) == 0);
    seco_desc big = desc(SECO_BF16, 1 << 15, 0, 64, 8);
    CHECK(seco_workspace_bytes(&big, SECO_OP_BWD) > SECO_STATIC_SCRATCH_BYTES);
    CHECK(seco_chunk_attn_bwd_noalloc(&big, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, nullptr) ==
          SECO_ERR_TOO_LARGE);
    // the plan does not depend on how much workspace there is: with and without grouped heads, few rows and many
    for (int hkv : {2, 8})
      for (int c : {256, hkv == 2 ? 1000 : 3976}) {
        const seco_desc e = desc(SECO_BF16, c, 512, 8, hkv);
        const size_t need = seco_workspace_bytes(&e, SECO_OP_BWD);
        CHECK(seco_workspace_bytes_preferred(&e, SECO_OP_BWD) == need);
        size_t room[4];
        for (int i = 0; i < 3; ++i) {
          CHECK(seco_chunk_attn_bwd(&e, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKE, need + ((size_t)i << 24), nullptr) == SECO_OK);
          room[i] = g_stub.last.tail_bytes;
        }
        CHECK(seco_chunk_attn_bwd_noalloc(&e, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, nullptr) == SECO_OK);
        room[3] = g_stub.last.tail_bytes;
        for (int i = 1; i < 4; ++i) CHECK(room[i] == room[0] && room[0] <= need);
      }
    // fp32
    seco_desc f = desc(SECO_F32, 100, 200, 4, 4, 64);
    g_stub.clear();
    CHECK(seco_chunk_attn_bwd(&f, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKE,
                              seco_workspace_bytes(&f, SECO_OP_BWD), nullptr) == SECO_OK);
    CHECK(g_stub.dq == 1 && g_stub.dkdv == 1);
    CHECK(g_stub.dkdv_tables[0].tile_begin[1] == (300 + seco::kColTileF32 - 1) / seco::kColTileF32);
  }
  // ---- weights: merged runs, zero chunks skipped, ragged last chunk, more runs than one table holds ----
  {
    seco_desc d = desc(SECO_BF16, 160, 7 * 160);           // 8 chunks of 160 rows, kv_len 1280
    const size_t ws = seco_workspace_bytes(&d, SECO_OP_BWD);
    const float w[8] = {2.f, 2.f, 0.f, 0.5f, 0.f, 0.f, 2.f, 1.f};
    g_stub.clear();
    CHECK(spaco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, w, 8, 160, FAKE, ws, nullptr) ==
          SECO_OK);
    CHECK(g_stub.dkdv == 1);
    const seco::SegTable& t = g_stub.dkdv_tables[0];
    CHECK(t.n == 4);
    CHECK(t.col_begin[0] == 0 && t.col_end[0] == 320 && t.weight[0] == 2.f && t.tile_begin[1] == 3);
    CHECK(t.col_begin[1] == 480 && t.col_end[1] == 640 && t.weight[1] == 0.5f && t.tile_begin[2] == 5);
    CHECK(t.col_begin[2] == 960 && t.col_end[2] == 1120 && t.weight[2] == 2.f && t.tile_begin[3] == 7);
    CHECK(t.col_begin[3] == 1120 && t.col_end[3] == 1280 && t.weight[3] == 1.f && t.tile_begin[4] == 9);
    const float bad[8] = {2.f, INFINITY, 0.f, 0.5f, 0.f, 0.f, 2.f, 1.f};
    CHECK(spaco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, bad, 8, 160, FAKE, ws, nullptr) ==
          SECO_ERR_WEIGHTS);
    CHECK(spaco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, w, 7, 160, FAKE, ws, nullptr) ==
          SECO_ERR_WEIGHTS);
    CHECK(spaco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, w, 9, 160, FAKE, ws, nullptr) ==
          SECO_ERR_WEIGHTS);
    // all weights zero: the dQ pass runs, no dK/dV launch
    const float z[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    g_stub.clear();
    CHECK(spaco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, z, 8, 160, FAKE, ws, nullptr) ==
          SECO_OK);
    CHECK(g_stub.dq == 1 && g_stub.dkdv == 0);
    // 110 chunks of 32 rows, every second weight zero, the others all different: 55 runs = 48 + 7
    seco_desc m = desc(SECO_BF16, 32, 109 * 32, 2, 1);
    std::vector<float> wm(110);
    for (int i = 0; i < 110; ++i) wm[i] = i % 2 ? 0.f : 1.f + 0.05f * i;
    wm[109] = 1.f;
    g_stub.clear();
    CHECK(spaco_chunk_attn_bwd(&m, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, wm.data(), 110, 32, FAKE,
                               seco_workspace_bytes(&m, SECO_OP_BWD), nullptr) == SECO_OK);
    CHECK(g_stub.dkdv == 2 && g_stub.dkdv_tables[0].n == 48 && g_stub.dkdv_tables[1].n == 8);
    int rows = 0;
    for (const auto& tb : g_stub.dkdv_tables) {
      CHECK(tb.tile_begin[tb.n] == tb.n);                   // one 32-row chunk = one (partly filled) column tile per run
      for (int i = 0; i < tb.n; ++i) rows += tb.col_end[i] - tb.col_begin[i];
    }
    CHECK(rows == 56 * 32);
    // column-weighted dQ: runs table, 48 runs at most
    const float wq[8] = {0.f, 3.f, 3.f, 0.f, 0.f, 1.25f, 0.f, 1.f};
    g_stub.clear();
    CHECK(spaco_chunk_attn_bwd_sparse_dq(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, w, wq, 8, 160, FAKE, ws,
                                         nullptr) == SECO_OK);
    CHECK(g_stub.dq_tables.size() == 1 && g_stub.dq_tables[0].n == 3);
    CHECK(g_stub.dq_tables[0].col_begin[0] == 160 && g_stub.dq_tables[0].col_end[0] == 480);
    CHECK(g_stub.dq_tables[0].col_begin[2] == 1120 && g_stub.dq_tables[0].col_end[2] == 1280);
    const float ones[8] = {1, 1, 1, 1, 1, 1, 1, 1};
    g_stub.clear();
    CHECK(spaco_chunk_attn_bwd_sparse_dq(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, w, ones, 8, 160, FAKE,
                                         ws, nullptr) == SECO_OK);
    CHECK(g_stub.dq_tables.empty());                        // all ones: the dense kernel
    std::vector<float> many(128), wone(128, 1.f);
    for (int i = 0; i < 128; ++i) many[i] = (float)(i % 2);
    seco_desc s4 = desc(SECO_BF16, 4, 127 * 4);
    CHECK(spaco_chunk_attn_bwd_sparse_dq(&s4, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, wone.data(),
                                         many.data(), 128, 4, FAKE, seco_workspace_bytes(&s4, SECO_OP_BWD), nullptr) ==
          SECO_ERR_TOO_LARGE);
  }
  // ---- transposed order: row runs ----
  {
    seco_desc d = desc(SECO_BF16, 128, 256);
    const size_t ws = seco_workspace_bytes(&d, SECO_OP_BWD);
    const float rw[6] = {1.f, 0.f, 4.f, 4.f, 0.f, 4.f};     // own chunk + 5 later chunks of 128 rows
    g_stub.clear();
    CHECK(spaco_chunk_attn_bwd_gather(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKEF, 1024, 640, rw, 6,
                                      128, FAKE, ws, nullptr) == SECO_OK);
    CHECK(g_stub.row_runs.size() == 1 && g_stub.row_runs[0].n == 3);
    CHECK(g_stub.row_runs[0].begin[1] == 256 && g_stub.row_runs[0].end[1] == 512 && g_stub.row_runs[0].log2w[1] == 2.f);
    CHECK(g_stub.dkdv_tables[0].col_begin[0] == 256 && g_stub.dkdv_tables[0].col_end[0] == 384);
    CHECK(spaco_chunk_attn_bwd_gather(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKEF, 1000, 640, rw, 6,
                                      128, FAKE, ws, nullptr) == SECO_ERR_RANGE);          // too few statistic rows
    CHECK(spaco_chunk_attn_bwd_gather(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKEF, 1024, 640, rw, 6,
                                      100, FAKE, ws, nullptr) == SECO_ERR_WEIGHTS);        // not a multiple of 64
    std::vector<float> alt(50);
    for (int i = 0; i < 50; ++i) alt[i] = (float)(1 - i % 2);
    seco_desc d64 = desc(SECO_BF16, 64, 0);
    CHECK(spaco_chunk_attn_bwd_gather(&d64, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKEF, 3200, 49 * 64,
                                      alt.data(), 50, 64, FAKE, seco_workspace_bytes(&d64, SECO_OP_BWD), nullptr) ==
          SECO_ERR_TOO_LARGE);                                                              // 25 runs > 24
    g_stub.clear();
    CHECK(seco_chunk_attn_bwd_gather(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKEF, 1024, 640, FAKE, ws,
                                     nullptr) == SECO_OK);
    CHECK(g_stub.row_runs.empty() && g_stub.last.C == 768 && g_stub.last.stat_stride == 1024);
  }
  // ---- host policies: selection, weight vectors, launch plan ----
  {
    int32_t sel[16];
    for (uint64_t seed = 0; seed < 50; ++seed) {
      CHECK(spaco_select_chunks(seed, seed * 7, 16, 16, sel) == SECO_OK);
      for (int i = 0; i < 16; ++i) CHECK(sel[i] == 15 - i);
      CHECK(spaco_select_chunks(seed, 1, 13, 5, sel) == SECO_OK);
      for (int i = 0; i < 5; ++i) CHECK(sel[i] >= 0 && sel[i] < 13 && (i == 0 || sel[i] < sel[i - 1]));
    }
    CHECK(spaco_select_chunks(0, 0, 4, 5, sel) == SECO_ERR_RANGE);
    float w[16];
    int32_t s3[3] = {9, 4, 1};
    CHECK(spaco_chunk_weights(s3, 3, 9, 2.5f, w) == SECO_OK);
    CHECK(w[9] == 1.f && w[4] == 2.5f && w[1] == 2.5f && w[0] == 0.f && w[8] == 0.f);
    CHECK(spaco_gather_row_weights(s3, 3, 1, 12, 2.5f, w) == SECO_OK);
    CHECK(w[0] == 1.f && w[3] == 2.5f && w[8] == 2.5f && w[1] == 0.f && w[10] == 0.f);
    CHECK(spaco_percall_weights(3, 0, 15, 4, w) == SECO_OK);
    int nz = 0;
    for (int i = 0; i < 15; ++i) nz += w[i] != 0.f;
    CHECK(nz == 4 && w[15] == 1.f);
    int32_t out[64], n = -1;
    CHECK(spaco_select_bernoulli(5, 0, 64, 0.25, out, &n) == SECO_OK && n >= 0 && n <= 64);
    CHECK(spaco_select_bernoulli(5, 0, 64, 1.0, out, &n) == SECO_OK && n == 64);
    CHECK(spaco_compensation_factor(16, 4, 0.f) == 4.f && spaco_compensation_factor(16, 4, 2.f) == 2.f);
    CHECK(spaco_compensation_factor(4, 5, 0.f) < 0.f);
    int32_t plan[4];
    seco_desc c3 = desc(SECO_BF16, 2048, 14 * 2048, 32, 8);
    CHECK(seco_launch_plan(&c3, 15 * 16, plan) == SECO_OK && plan[0] == 1 && plan[1] == 512);
    seco_desc one = desc(SECO_BF16, 2048, 14 * 2048, 4, 1);
    CHECK(seco_launch_plan(&one, 15 * 16, plan) == SECO_OK && plan[0] > 1);
    CHECK(std::strcmp(seco_strerror(0), "ok") == 0 && std::strcmp(seco_strerror(-99), "unknown status") == 0);
    // appended rows, read-out, rotation: argument checks and dispatch
    seco_desc d = desc();
    g_stub.clear();
    CHECK(kv_append(&d, FAKE, FAKE, FAKE, FAKE, nullptr) == SECO_OK && g_stub.copy == 1);
    CHECK(kv_append_rope(&d, FAKE, FAKE, FAKE, FAKE, 500000.f, nullptr) == SECO_OK && g_stub.rope == 1 && g_stub.copy == 1);
    CHECK(kvgrad_readout_rope(&d, FAKEF, FAKEF, FAKE, FAKE, 2.f, 500000.f, nullptr) == SECO_OK && g_stub.rope == 2);
    CHECK(kv_append_rope(&d, FAKE, FAKE, FAKE, FAKE, 0.5f, nullptr) == SECO_ERR_RANGE);
    CHECK(kv_append(&d, FAKE, nullptr, nullptr, nullptr, nullptr) == SECO_ERR_NULL);
    CHECK(rope_rotate(&d, 0, FAKE, FAKE, 0, 10000.f, 0, nullptr) == SECO_ERR_RANGE);
    CHECK(kvgrad_readout(&d, FAKEF, FAKEF, FAKE, FAKE, INFINITY, nullptr) == SECO_ERR_RANGE);
  }
  // ---- work items and workgroups: every item once, those of a unit on its XCDs ----
  for (int units : {1, 2, 3, 4, 5, 8, 16})
    for (int run : {1, 7, 31, 64, 65, 128, 130, 256, 257, 519}) {
      const int total = run * units, first = total / 3;
      const bool dealt = seco::xcds_share_units(total, units);
      CHECK(dealt == (total > 256 && (units == 1 || units == 2 || units == 4)));
      std::vector<int> taken(total, 0), taken2(total, 0);
      for (int block = 0; block < seco::xcd_grid(total, units); ++block) {
        const int item = seco::xcd_item(block, total, units);
        CHECK(item < total);
        if (item >= 0) ++taken[item];
        if (item >= 0 && dealt) CHECK((block & 7) / (8 / units) == item / run);
      }
      for (int block = 0; block < seco::xcd_grid(first) + seco::xcd_grid(total - first); ++block)
        if (const int item = seco::shares_item(block, first, total); item >= 0) ++taken2[item];
      CHECK(std::count(taken.begin(), taken.end(), 1) == total && std::count(taken2.begin(), taken2.end(), 1) == total);
    }
  // one round of column tiles, alike or on the diagonal: how busy it keeps the compute units
  for (const int* s : {(const int[]){32, 8}, (const int[]){64, 4}, (const int[]){128, 2}}) {
    const seco::IterRuns alike = seco::iter_runs(s[0], [](int) { return 40; }), causal = seco::iter_runs(s[0], [&](int t) { return 2 * (s[0] - t); });
    float time, busy;
    seco::share_plan(alike, s[1], s[0], 1, 2560, 256, time, &busy);
    CHECK(busy == 1.f);
    CHECK(seco::share_plan(causal, s[1], s[0], 1, 128 * s[0], 256, time, &busy).n_tiles == 0);
    CHECK(s[1] >= 4 ? busy > 0.5f && busy < 0.7f : busy == 1.f);
  }
  CHECK(seco::dq_leaves_cus(256, 23592) && !seco::dq_leaves_cus(256, 23593) && !seco::dq_leaves_cus(257, 257));
  // taller tiles beside a weight gradient (rows, K, n, that gradient's tiles): a round of an XCD saved, or long contractions
  for (const int* s : {(const int[]){512, 1024, 4096, 256, 1}, (const int[]){512, 1024, 2048, 128, 1}, (const int[]){512, 1024, 1024, 256, 1}, (const int[]){384, 1024, 1536, 192, 1},
                       (const int[]){140, 2560, 192, 120, 1}, (const int[]){97, 3520, 1280, 280, 0}, (const int[]){1015, 448, 1344, 147, 0}, (const int[]){2701, 192, 5312, 249, 0}, (const int[]){331, 1408, 2880, 253, 0},
                       (const int[]){1139, 384, 128, 12, 0}, (const int[]){320, 1024, 4096, 256, 0}, (const int[]){87, 3008, 256, 188, 0}}) {
    const int n64 = (s[1] + 63) / 64;
    CHECK(seco::taller_pays(s[0], s[2], (s[0] + 31) / 32 * n64, (s[0] + 63) / 64 * n64, s[3]) == (s[4] != 0));
  }
  // the small forward's cache: three rounds saved are worth a merge until its workgroups read at the memory's rate
  CHECK(seco::small_divides(8, 3) && seco::small_divides(112, 3) && !seco::small_divides(113, 3) && seco::small_divides(128, 4) && !seco::small_divides(1, 2));
  // the 4-wavefront forward's turns: not with three or four KV heads to an XCD around two rounds
  for (const int* s : {(const int[]){32, 4096, 0, 1024, 0}, (const int[]){32, 3994, 300, 1024, 0}, (const int[]){32, 4471, 0, 1120, 0}, (const int[]){24, 5400, 0, 1032, 0}, (const int[]){24, 4900, 0, 936, 0}, (const int[]){24, 7000, 600, 1320, 0},
                       (const int[]){24, 7500, 0, 1416, 0}, (const int[]){24, 7900, 0, 1488, 0}, (const int[]){24, 8192, 0, 1536, 1}, (const int[]){24, 7900, 600, 1488, 1}, (const int[]){24, 4300, 0, 816, 1}, (const int[]){24, 4900, 4000, 936, 1},
                       (const int[]){32, 3964, 0, 992, 1}, (const int[]){32, 4600, 0, 1152, 1}, (const int[]){32, 4000, 4000, 1024, 1},
                       (const int[]){16, 4096, 0, 1024, 1}, (const int[]){64, 4096, 0, 1024, 1}}) {
    seco::AttnParams p{};
    p.B = 1;
    p.Hkv = s[0];
    p.C = s[1];
    p.q_start = s[2];
    CHECK(seco::turns_pay(p, s[3]) == (s[4] != 0));
  }
  // ---- where an output lies over an input ----
  {
    static char mem[1 << 20];
    seco::AttnParams p;
    std::memset(&p, 0, sizeof(p));
    p.B = 2; p.Hq = 4; p.Hkv = 2; p.D = 64; p.C = 20; p.q_start = 30;
    const int64_t packed[3] = {4 * 20 * 64, 20 * 64, 64}, kv[3] = {2 * 50 * 64, 50 * 64, 64};
    for (int i = 0; i < 3; ++i) p.qs[i] = p.os[i] = packed[i], p.kvs[i] = kv[i];
    const int q_bytes = 2 * 4 * 20 * 64 * 4, kv_bytes = 2 * 2 * 50 * 64 * 4;
    p.q = mem; p.k = mem + q_bytes; p.v = mem + q_bytes + kv_bytes;
    for (const int at : {q_bytes + 2 * kv_bytes, q_bytes + 2 * kv_bytes + 4096}) {      // behind all of them
      p.o_out = mem + at;
      CHECK(!seco::o_over_inputs(p, 4));
    }
    for (const int at : {0, 16, q_bytes - 16, q_bytes, q_bytes + kv_bytes, q_bytes + 2 * kv_bytes - 16}) {
      p.o_out = mem + at;
      CHECK(seco::o_over_inputs(p, 4));
    }
    p.o = mem + (1 << 18); p.d_o = mem + (1 << 19);
    for (const int at : {q_bytes + 2 * kv_bytes, (1 << 18) - q_bytes, (1 << 18) + q_bytes, (1 << 19) - q_bytes, (1 << 19) + q_bytes}) {
      p.d_q = mem + at;
      CHECK(!seco::dq_over_inputs(p, 4));
    }
    for (const int at : {0, q_bytes, q_bytes + kv_bytes, 1 << 18, (1 << 18) + q_bytes - 16, 1 << 19, (1 << 19) - q_bytes + 16}) {
      p.d_q = mem + at;
      CHECK(seco::dq_over_inputs(p, 4));
    }
    p.q = mem + (1 << 19); p.o_out = mem + (1 << 19) - q_bytes;                        // right before q
    CHECK(!seco::o_over_inputs(p, 4));
    p.os[1] += 4;                                                                       // heads 16 bytes further apart
    CHECK(seco::o_over_inputs(p, 4));
    p.C = 1; p.B = p.Hq = 1;                                                            // (strides that reach no row do not count)
    p.os[0] = p.os[1] = (int64_t)1 << 61;
    CHECK(!seco::o_over_inputs(p, 4));
  }
  // ---- the plan of a backward: both passes in one launch only while dQ is still to go out; by itself dK/dV shares out the iterations of
  // the stages that it walks (joined: of several heads' rows; the last two only then, {32, 8, 199, 8127} with shared tiles) ----
  {
    const int shapes[][6] = {{8, 8, 64, 6400, 1, 0}, {32, 8, 745, 0, 1, 0}, {8, 2, 32, 3488, 1, 1}, {32, 8, 32, 0, 1, 1},
                             {32, 4, 1200, 4000, 0, 0}, {32, 8, 150, 16000, 0, 1}, {32, 8, 199, 8127, 0, 1}};
    for (const auto& sh : shapes) {
      const seco_desc d = desc(SECO_BF16, sh[2], sh[3], sh[0], sh[1]);
      CHECK(seco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKE,
                                seco_workspace_bytes(&d, SECO_OP_BWD), nullptr) == SECO_OK);
      const seco::AttnParams p = g_stub.last;
      const seco::SegTable& seg = g_stub.dkdv_tables.back();
      const seco::BwdPlan with = seco::plan_bwd<Cfg>(p, seg, true), without = seco::plan_bwd<Cfg>(p, seg, false);
      CHECK((with.dq_splits > 0) == (sh[4] != 0) && without.dq_splits == 0 && without.ts.part == p.tail_part);
      CHECK(without.joined == (sh[5] != 0) && (sh[4] || with.joined == without.joined));
      seco::RowRuns none;
      none.n = 0;
      float time, busy;
      const seco::IterRuns runs = seco::tile_iterations<Cfg, false>(p, seg, none, without.joined);
      const seco::SharePlan alone = seco::share_plan(runs, p.B * p.Hkv, seg.tile_begin[seg.n], p.G, p.C, seco::slots_in(p.tail_bytes), time, &busy);
      const seco::BwdPlan& apart = sh[4] ? without : with;
      const seco::SharePlan& got = apart.ts.plan;
      CHECK(apart.busy == busy && got.n_tiles == alone.n_tiles && got.n_shared == alone.n_shared && got.n_entries == alone.n_entries);
      CHECK(std::equal(alone.tile_of, alone.tile_of + alone.n_entries, got.tile_of));
      CHECK(alone.n_tiles == 0 || std::equal(alone.first, alone.first + alone.n_tiles + 1, got.first));
      // no workgroup of a shared tile is left without an iteration
      for (int i = 0; i < got.n_shared; ++i) {
        int tile = i, it = 0;
        seco::for_last(runs, got.n_tiles, [&](int iters, int count) {
          if (tile >= 0 && tile < count) it = iters;
          tile -= count;
        });
        CHECK(got.first[i + 1] - got.first[i] <= it);
      }
    }
  }
  // a round or more of column tiles: one launch by their iterations, by what a last round leaves over, and by dQ's row tiles, which
  // in one launch of full workgroups are whole and hold padding.  (B, Hq, Hkv, C, q_start, shares of dQ; 0: two launches)
  for (const int* s : {(const int[]){4, 64, 8, 64, 11814, 0}, (const int[]){4, 64, 8, 41, 4359, 0}, (const int[]){4, 48, 8, 44, 12097, 0},   // half of them padding
                       (const int[]){4, 48, 8, 50, 1050, 1}, (const int[]){4, 32, 8, 145, 10190, 0}, (const int[]){4, 32, 8, 85, 1190, 1},
                       (const int[]){1, 16, 4, 175, 14784, 0}, (const int[]){1, 24, 8, 181, 7240, 0}, (const int[]){1, 32, 32, 617, 3916, 1},   // full rounds but for a tenth
                       (const int[]){1, 8, 8, 532, 6442, 4},
                       (const int[]){1, 16, 4, 88, 8779, 10}, (const int[]){1, 48, 8, 66, 4663, 4}, (const int[]){1, 32, 8, 64, 4032, 4}}) {   // a little over a round, one round
    seco_desc d = desc(SECO_BF16, s[3], s[4], s[1], s[2]);
    d.batch = s[0];
    CHECK(seco_chunk_attn_bwd(&d, FAKE, FAKE, FAKE, FAKE, FAKEF, FAKE, FAKE, FAKEF, FAKEF, FAKE,
                              seco_workspace_bytes(&d, SECO_OP_BWD), nullptr) == SECO_OK);
    CHECK(seco::plan_bwd<Cfg>(g_stub.last, g_stub.dkdv_tables.back(), true).dq_splits == s[5]);
  }
  // workgroups laid out in groups end when they do one by one (whole microseconds: no two groups are taken as one), also past the
  // room for groups; the choice of shares for several numbers of compute units is that for each
  {
    unsigned x = 12345;
    auto draw = [&](int n) { return (int)((x = x * 1664525u + 1013904223u) >> 16) % n; };
    for (int places : {1, 3, 32, 64}) {
      seco::Schedule sc(places);
      std::vector<int> at(places, 0);
      for (int i = 0; i < 600; ++i) {
        const int time = 1 + draw(i % 7 == 0 ? 500 : 40), count = 1 + draw(2 * places);
        sc.run((float)time, count);
        for (int c = 0; c < count; ++c) *std::min_element(at.begin(), at.end()) += time;
        CHECK(sc.end() == (float)*std::max_element(at.begin(), at.end()));
      }
    }
    for (int i = 0; i < 200; ++i) {
      const int rows = 64 * (1 + draw(60)), n = 1 + draw(40), units = 1 + draw(16), cus[3] = {96, 160, 256};
      const seco::IterRuns r = seco::iter_runs(n, [&](int t) { return std::max(1, rows / 64 - 2 * std::max(0, t - n / 2)); });
      for (bool fit : {false, true}) {
        seco::ShareChoice c[3];
        seco::choose_shares(r, n, units, cus, 256, 1, fit, seco::kDkdvOwnTime, c);
        for (int k = 0; k < 3; ++k) {
          const seco::ShareChoice one = seco::choose_shares(r, n, units, cus[k], 256, 1, fit, seco::kDkdvOwnTime);
          CHECK(c[k].per == one.per && c[k].time == one.time && c[k].longest == one.longest);
        }
      }
    }
  }
  std::puts("host sanitizer run: all checks passed");
  return 0;
}
