// Backward of one chunk, fp32: dQ and dK/dV (f32_tiles.h).
#include <algorithm>
#include <type_traits>

#include "f32_tiles.h"

namespace seco {
namespace {

// Rows that every wavefront of a backward's workgroup keeps: copied once, each wavefront a part, into an image that all read
// after a barrier.  (Copied by all of them they were half of a short call's loads: head_dim 128, 16.7 -> 15.7 us.)
template <int NT, int NW> struct Shared {
  static constexpr int kPer = (NT + NW - 1) / NW;
  f32x4 v[kPer];
  __device__ __forceinline__ void load(const float* base, int64_t stride, int n, int D, int w, int lane) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int piece = lane + 64 * (w + NW * k);
      if (w + NW * k < NT) v[k] = load4(base + min(piece / (4 * NT), n - 1) * stride + min(piece % (4 * NT) * 4, D - 4));
    }
  }
  __device__ __forceinline__ void put(float* image, int w, int lane) const {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int piece = lane + 64 * (w + NW * k);
      if (w + NW * k < NT) *reinterpret_cast<f32x4*>(image + piece / (4 * NT) * kPartRow<NT> + piece % (4 * NT) * 4) = v[k];
    }
  }
};
// sum over the wavefronts, in order, of row i's elements d .. d + 3
template <int NT, int NO, int NW>
__device__ __forceinline__ f32x4 sum_part(const float* part, int i, int d) {
  f32x4 s = zero4();
#pragma unroll
  for (int w = 0; w < NW; ++w) s += load4(part + w * kPart<NT> + i * kPartRow<NO> + d);
  return s;
}

// The backward of a chunk in one launch: the first n_dq workgroups own 16 query rows each (dQ), the others 16 cache rows
// (dK/dV); neither needs the other's results, since both take rowsum(dO * O) from the O and dO rows they hold anyway.
// (As three launches - rowsum, dQ, dK/dV - a call of cfg1 took 35 us, each launch 3 - 4 us before its first load returns
// and on a quarter of the CUs.)  A wavefront has two LDS images of its own for the rows it turns.

// One run of rows with weight, in place of a SegTable of one: the kernel then takes 0.4 KB of arguments instead of 1.9, which
// the host writes to device memory for every launch (3.1 against 4.2 us), and finds them in two cache lines.
struct OneRun {
  int begin, end;
  float weight;
};
__device__ __forceinline__ int runs_of(const SegTable& t) { return t.n; }
__device__ __forceinline__ int runs_of(const OneRun&) { return 1; }
__device__ __forceinline__ OneRun run_at(const SegTable& t, int si) { return {t.col_begin[si], t.col_end[si], t.weight[si]}; }
__device__ __forceinline__ OneRun run_at(const OneRun& t, int) { return t; }
// the rows of column tile `tile` (end: of its run)
__device__ __forceinline__ OneRun tile_at(const SegTable& t, int tile) {
  int si = 0;
  while (si + 1 < t.n && tile >= t.tile_begin[si + 1]) ++si;
  return {t.col_begin[si] + (tile - t.tile_begin[si]) * kRows, t.col_end[si], t.weight[si]};
}
__device__ __forceinline__ OneRun tile_at(const OneRun& t, int tile) { return {t.begin + tile * kRows, t.end, t.weight}; }

// dQ = s * sum over the runs of cache rows of w * dS K (one run with weight 1 over all visible rows: the exact dQ); of dQ the
// columns of NO of the NT blocks
template <int NT, int NO, int NW, typename Runs>
__device__ __forceinline__ void dq_f32(const AttnArgs& p, const Runs& runs, int item_part, float* part) {
  constexpr int kParts = (NT + NO - 1) / NO;
  const int item = item_part / kParts, o0 = item_part % kParts * (16 * NO), n_o = kParts == 1 ? p.D : min(p.D - o0, 16 * NO);
  if (kParts > 1 && n_o <= 0) return;
  constexpr bool kAhead = NT <= 5;                      // (longer rows do not leave the registers)
  constexpr bool kTable = std::is_same<Runs, SegTable>::value;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;
  const int n_rt = (p.C + kRows - 1) / kRows, rt = item / (p.Hq * p.B), bh = item - rt * p.Hq * p.B, b = bh / p.Hq, h = bh - b * p.Hq;
  const int r0 = (n_rt - 1 - rt) * kRows, D = p.D;      // the rows that see most first
  const float* K = static_cast<const float*>(p.k) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const float* V = static_cast<const float*>(p.v) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const int64_t row = p.kvs[2];
  const int qpos = p.q_start + r0 + i, kv_end = p.q_start + min(r0 + kRows, p.C);
  float *own = part + w * kPart<NT>, *own2 = own + NW * kPart<NT>;
  const Pieces<NT> pk(lane, row, D);
  Block<NT> kb, vb;
  auto load_kv = [&](int c0, int end) {
    pk.load(kb, K + c0 * row, row, end - c0);
    pk.load(vb, V + c0 * row, row, end - c0);
  };
  f32x4 qf[NT], dof[NT];
  float delta = 0.f;
  {
    Shared<NT, NW> sq, sd, so;
    const int64_t orow = b * p.os[0] + h * p.os[1] + r0 * p.os[2];
    sq.load(static_cast<const float*>(p.q) + b * p.qs[0] + h * p.qs[1] + r0 * p.qs[2], p.qs[2], p.C - r0, D, w, lane);
    sd.load(static_cast<const float*>(p.d_o) + orow, p.os[2], p.C - r0, D, w, lane);
    so.load(static_cast<const float*>(p.o) + orow, p.os[2], p.C - r0, D, w, lane);
    if (kAhead && runs_of(runs) > 0) {                  // (under the query rows' loads)
      const OneRun run = run_at(runs, 0);
      const int end = min(kv_end, run.end), c0 = run.begin + 16 * w;
      if (c0 < end) load_kv(c0, end);
    }
    sq.put(part, w, lane);
    sd.put(part + kPart<NT>, w, lane);
    so.put(part + 2 * kPart<NT>, w, lane);
    __syncthreads();
    f32x4 of[NT];
    rows_of<NT>(part, i, g, qf);
    rows_of<NT>(part + kPart<NT>, i, g, dof);
    rows_of<NT>(part + 2 * kPart<NT>, i, g, of);
    mask_kept<NT>(D, g, qf);
    mask_kept<NT>(D, g, dof);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) delta += of[t][j] * dof[t][j];
    delta += __shfl_xor(delta, 16);
    delta += __shfl_xor(delta, 32);
    __syncthreads();
  }
  const float lse = p.lse[((int64_t)b * p.Hq + h) * p.C + min(r0 + i, p.C - 1)] * kLog2e, c = p.scale * kLog2e;
  Acc<NO> dq;
  dq.clear();
  int next = w;                                         // blocks of all runs are dealt to the wavefronts in turn
  for (int si = 0; si < runs_of(runs); ++si) {
    const OneRun run = run_at(runs, si);
    const int end = min(kv_end, run.end);
    if (run.begin >= end) break;
    int c0 = run.begin + 16 * next;
    if (kAhead && si > 0 && c0 < end) load_kv(c0, end);
#pragma unroll 1
    for (; c0 < end; c0 += 16 * NW) {
      const bool more = kAhead && c0 + 16 * NW < end;
      if (!kAhead) load_kv(c0, end);
      f32x4 s, dp, ds;
      pk.put(own, kb, lane);
      pk.put(own2, vb, lane);
      if (more) load_kv(c0 + 16 * NW, end);
      {
        f32x4 x[NT];
        rows_of<NT>(own, i, g, x);
        s = score<NT>(x, qf);
      }
      {
        f32x4 x[NT];
        rows_of<NT>(own2, i, g, x);
        dp = score<NT>(x, dof);
      }
      Cols<NO> kc;
      kc.load([&](int r) { return own + (4 * g + r) * kPartRow<NT> + o0; }, min(16 * NO, 16 * NT - o0), i);
      asm volatile("" : : : "memory");
#pragma unroll
      for (int r = 0; r < 4; ++r) ds[r] = fast_exp2(__builtin_fmaf(s[r], c, -lse)) * (dp[r] - delta);
      if (kTable) ds *= run.weight;                     // (of a single run: with the scale, at the end)
      if (c0 + kRows > min(end, p.q_start + r0)) {      // a block on the diagonal or past the run's end
#pragma unroll
        for (int r = 0; r < 4; ++r) ds[r] = c0 + 4 * g + r <= qpos && c0 + 4 * g + r < end ? ds[r] : 0.f;
      }
      dq.add(kc, ds);
    }
    next = (c0 - run.begin) / 16 - (end - run.begin + 15) / 16;   // this wavefront's next block, counted from the run's end
  }
  dq.store(own, i, g);
  __syncthreads();
  for (int e = threadIdx.x; e < kRows * NO * 4; e += NW * 64) {
    const int rr = e / (NO * 4), d = 4 * (e % (NO * 4));
    if (r0 + rr >= p.C || d >= n_o) continue;
    float* out = static_cast<float*>(p.d_q) + b * p.qs[0] + h * p.qs[1] + (r0 + rr) * p.qs[2] + o0 + d;
    *reinterpret_cast<f32x4*>(out) = (kTable ? p.scale : p.scale * run_at(runs, 0).weight) * sum_part<NT, NO, NW>(part, rr, d);
  }
}

// gK[c] += w * s * sum_h dS^T Q, gV[c] += w * sum_h P^T dO for 16 cache rows (exclusive owner); the wavefronts divide
// the (query head, block of 16 query rows) pairs that see them.
template <int NT, int NW, typename Runs>
__device__ __forceinline__ void dkdv_f32(const AttnArgs& p, const Runs& runs, int item, float* part) {
  constexpr bool kAhead = NT <= 5;                      // (longer rows do not leave the registers)
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;
  const int tile = item / (p.Hkv * p.B), bh = item - tile * p.Hkv * p.B, b = bh / p.Hkv, kvh = bh - b * p.Hkv, D = p.D;
  const OneRun run = tile_at(runs, tile);
  const int c0 = run.begin, c_end = run.end;
  // the group's first head (per-head products of 64-bit strides in the loop would cost scalar registers that are not there)
  const int h0 = kvh * p.G;
  const float* q_group = static_cast<const float*>(p.q) + b * p.qs[0] + h0 * p.qs[1];
  const float* do_group = static_cast<const float*>(p.d_o) + b * p.os[0] + h0 * p.os[1];
  const float* o_group = static_cast<const float*>(p.o) + b * p.os[0] + h0 * p.os[1];
  const float* lse_group = p.lse + ((int64_t)b * p.Hq + h0) * p.C;
  const int rb0 = max(0, c0 - p.q_start) / kRows, n_rb = (p.C + kRows - 1) / kRows - rb0;   // row blocks that see the tile
  // (head of the group, row block) pairs of a wavefront: every NW-th
  struct Pos { int hg, rb; };
  auto advance = [&](Pos x, int by) {
    x.rb += by;
    while (x.rb >= n_rb) x.rb -= n_rb, ++x.hg;
    return x;
  };
  float *own = part + w * kPart<NT>, *own2 = own + NW * kPart<NT>;
  const Pieces<NT> pq(lane, p.qs[2], D), po(lane, p.os[2], D);
  Block<NT> qb, db, ob;
  auto load_q = [&](Pos x) {
    const int q0 = (rb0 + x.rb) * kRows;
    pq.load(qb, q_group + x.hg * p.qs[1] + q0 * p.qs[2], p.qs[2], p.C - q0);
  };
  auto load_o = [&](Pos x) {
    const int q0 = (rb0 + x.rb) * kRows;
    const int64_t at = x.hg * p.os[1] + q0 * p.os[2];
    po.load(db, do_group + at, p.os[2], p.C - q0);
    po.load(ob, o_group + at, p.os[2], p.C - q0);
  };
  Pos nx = advance(Pos{0, 0}, w);
  f32x4 kf[NT], vf[NT];
  {
    Shared<NT, NW> sk, sv;
    const int64_t at = b * p.kvs[0] + kvh * p.kvs[1] + c0 * p.kvs[2];
    sk.load(static_cast<const float*>(p.k) + at, p.kvs[2], c_end - c0, D, w, lane);
    sv.load(static_cast<const float*>(p.v) + at, p.kvs[2], c_end - c0, D, w, lane);
    if (kAhead && nx.hg < p.G) load_o(nx), load_q(nx);
    sk.put(part, w, lane);
    sv.put(part + kPart<NT>, w, lane);
    __syncthreads();
    rows_of<NT>(part, i, g, kf);
    rows_of<NT>(part + kPart<NT>, i, g, vf);
    mask_kept<NT>(D, g, kf);
    mask_kept<NT>(D, g, vf);
    __syncthreads();
  }
  const float c = p.scale * kLog2e;
  Acc<NT> dk, dv;
  dk.clear();
  dv.clear();
#pragma unroll 1
  while (nx.hg < p.G) {
    const Pos at = nx;
    const int q0 = (rb0 + at.rb) * kRows;
    nx = advance(nx, NW);
    const bool more = kAhead && nx.hg < p.G;
    const float lse = lse_group[(int64_t)at.hg * p.C + min(q0 + i, p.C - 1)] * kLog2e;
    if (!kAhead) load_o(at);
    float delta = 0.f;                                  // of row i
    f32x4 s, dp;
    pq.put(own, ob, lane);
    pq.put(own2, db, lane);
    if (more) load_o(nx);
    {
      f32x4 dox[NT], ox[NT];
      rows_of<NT>(own, i, g, ox);
      rows_of<NT>(own2, i, g, dox);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) delta += t < kWhole<NT> || 16 * t + 4 * g < D ? ox[t][j] * dox[t][j] : 0.f;
      if (!kAhead) load_q(at);
      dp = score<NT>(dox, vf);
    }
    delta += __shfl_xor(delta, 16);
    delta += __shfl_xor(delta, 32);
    pq.put(own, qb, lane);
    if (more) load_q(nx);
    {
      f32x4 qx[NT];
      rows_of<NT>(own, i, g, qx);
      s = score<NT>(qx, kf);
    }
    f32x4 pr, ds;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float row_lse = __shfl(lse, 4 * g + r), row_delta = __shfl(delta, 4 * g + r);   // (by all lanes)
      pr[r] = fast_exp2(__builtin_fmaf(s[r], c, -row_lse));
      ds[r] = dp[r] - row_delta;
    }
    if (c0 + kRows > p.q_start + q0 || q0 + kRows > p.C) {   // on the diagonal or past the last row
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qr = q0 + 4 * g + r;
        pr[r] = qr < p.C && c0 + i <= p.q_start + qr ? pr[r] : 0.f;
      }
    }
    ds *= pr;
    Cols<NT> x;
    x.of(own2, i, g);
    dv.add(x, pr);
    x.of(own, i, g);
    dk.add(x, ds);
  }
  // gV's elements, then gK's; their old values are requested before the partial sums are exchanged
  constexpr int kQuads = kRows * NT * 4, kPer = (2 * kQuads + NW * 64 - 1) / (NW * 64);
  auto target = [&](int e, float*& q, float& wt) {      // false: nothing there
    const int pass = e / kQuads, rr = (e % kQuads) / (NT * 4), d = 4 * (e % (NT * 4));
    q = (pass ? p.gk : p.gv) + b * p.gs[0] + kvh * p.gs[1] + min(c0 + rr, c_end - 1) * p.gs[2] + min(d, D - 4);
    wt = pass ? run.weight * p.scale : run.weight;
    return e < 2 * kQuads && c0 + rr < c_end && d < D;
  };
  f32x4 old[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    float *q, wt;
    target(min((int)threadIdx.x + k * NW * 64, 2 * kQuads - 1), q, wt);
    old[k] = load4(q);
  }
  dv.store(own, i, g);
  dk.store(own2, i, g);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = threadIdx.x + k * NW * 64;
    float *q, wt;
    if (!target(e, q, wt)) continue;
    *reinterpret_cast<f32x4*>(q) = old[k] + wt * sum_part<NT, NT, NW>(part + e / kQuads * (NW * kPart<NT>), (e % kQuads) / (NT * 4), 4 * (e % (NT * 4)));
  }
}

template <int NT, int NO, int NW, typename Runs>
__global__ __launch_bounds__(NW * 64) void bwd_f32_kernel(AttnArgs p, Runs dq_runs, Runs seg, int n_dq) {
  extern __shared__ float part[];                       // two images per wavefront
  if ((int)blockIdx.x < n_dq)
    dq_f32<NT, NO, NW>(p, dq_runs, blockIdx.x, part);
  else
    dkdv_f32<NT, NW>(p, seg, blockIdx.x - n_dq, part);
}

// Wavefronts per workgroup: as many as the register file holds of the kernel at that head_dim.
template <int NT> constexpr int kBwdWaves = NT <= 8 ? 8 : 4;

inline int64_t columns_of(const OneRun& t) { return t.end - t.begin; }
inline int64_t columns_of(const SegTable& t) {
  int64_t n = 0;
  for (int i = 0; i < t.n; ++i) n += t.col_end[i] - t.col_begin[i];
  return n;
}

// Few row tiles: as in the forward, two or four workgroups for each, which compute a part of dQ's columns apiece (a third of
// the work).  64 + 128 tiles of head_dim 64 10.9 -> 10.1 us; 15 + 120 of 128 23.3 -> 19.1 (four); 28 + 252 of 64 18.1 -> 16.5 (two: the
// others' CUs may be shared a little, 64 + 256 gain nothing); 120 + 120 of 128 by two 26.2 -> 28.1.
// Where the whole tiles have a CU each and the halves would not, `crowded` says whether sharing costs more than the halves save: the
// time of a dQ tile goes with its columns, that of the column tiles which share a CU (the last, launched last) with the rows they
// see.  Of 55 calls measured, of head_dim 32 .. 256, none below the line is slower whole: 64 + 192 of 64 over 768 columns 17.7 -> 14.8 us,
// 64 + 160 over 640 14.4 -> 12.8, 66 + 174 of 128 over 917 36.8 -> 33.1; beyond it 57 + 159 of 128 over 843 take 30.6 whole, 26.7 in halves.
template <int NT, int NO, typename Runs>
int bwd_launch(const AttnParams& p, const Runs& dq_runs, const Runs& seg, int64_t n_dq, int64_t n_kv, hipStream_t s) {
  constexpr int NW = kBwdWaves<NT>, smem = 2 * NW * kPart<NT> * 4;
  auto kern = bwd_f32_kernel<NT, NO, NW, Runs>;
  n_dq *= (NT + NO - 1) / NO;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  if (n_dq + n_kv > 0x7fffffff) return SECO_ERR_TOO_LARGE;
  ProfScope prof(n_dq == 0 ? kKernelDkdv : n_kv ? kKernelBwd : kKernelDq, s);
  hipLaunchKernelGGL(kern, dim3((unsigned)(n_dq + n_kv)), dim3(NW * 64), smem, s, p, dq_runs, seg, (int)n_dq);
  return launch_status();
}
inline bool crowded(const AttnParams& p, int64_t columns, int64_t n_dq, int64_t n_kv, int64_t cus) {
  const int64_t shared = n_dq * 2 + n_kv - cus, rows = std::min<int64_t>(p.C, kRows * shared / (p.Hkv * p.B));
  return n_dq + n_kv <= cus && shared > 0 && 4 * columns < 1200 + 11 * rows * p.G;
}
template <int NT, typename Runs>
int bwd_parts(const AttnParams& p, const Runs& dq_runs, const Runs& seg, int64_t n_dq, int64_t n_kv, hipStream_t s) {
  const int64_t cus = device_cus();
  if constexpr (NT < 16 || std::is_same<Runs, OneRun>::value) {    // (with the table scalar registers are short at the longest rows)
    if (dq_over_inputs(p, sizeof(float))) return bwd_launch<NT, NT>(p, dq_runs, seg, n_dq, n_kv, s);
    if (n_dq * 4 + n_kv <= cus) return bwd_launch<NT, (NT + 3) / 4>(p, dq_runs, seg, n_dq, n_kv, s);
    if (n_dq * 2 + n_kv <= cus + cus / 4 && !crowded(p, columns_of(dq_runs), n_dq, n_kv, cus))
      return bwd_launch<NT, (NT + 1) / 2>(p, dq_runs, seg, n_dq, n_kv, s);
  }
  return bwd_launch<NT, NT>(p, dq_runs, seg, n_dq, n_kv, s);
}
template <int NT>
int bwd_nt(const AttnParams& p, const SegTable& dq_runs, const SegTable& seg, bool dq, hipStream_t s) {
  const int64_t n_dq = dq ? (int64_t)((p.C + kRows - 1) / kRows) * p.Hq * p.B : 0;
  const int64_t n_kv = (int64_t)seg.tile_begin[seg.n] * p.Hkv * p.B;
  if (dq_runs.n == 1 && seg.n == 1) {
    const OneRun d{dq_runs.col_begin[0], dq_runs.col_end[0], dq_runs.weight[0]}, k{seg.col_begin[0], seg.col_end[0], seg.weight[0]};
    return bwd_parts<NT>(p, d, k, n_dq, n_kv, s);
  }
  return bwd_parts<NT>(p, dq_runs, seg, n_dq, n_kv, s);
}

}  // namespace

// Both passes of the fp32 backward are one launch: dQ is noted in p.pending and goes out with dK/dV (launch_dkdv_f32;
// with an empty table when there are no cache rows to cover).  rowsum(dO * O) is taken from O and dO where it is used, so a
// dQ that lies over one of them goes out behind the last dK/dV table, in a launch of its own.
int launch_dq_f32(const AttnParams& p, const SegTable* dq_runs, hipStream_t) {
  SegTable& runs = p.pending->runs;
  runs = SegTable{};
  runs.n = 1;
  runs.col_end[0] = p.q_start + p.C;
  runs.weight[0] = 1.f;
  if (dq_runs) runs = *dq_runs;
  p.pending->dq = true;
  return SECO_OK;
}

int launch_dkdv_f32(const AttnParams& p, const SegTable& seg, hipStream_t s) {
  static_assert(kColTileF32 == kRows, "one workgroup per column tile");
  const bool rows = seg.tile_begin[seg.n] > 0, dq = p.pending->dq && !(rows && dq_over_inputs(p, sizeof(float)));
  if (dq) p.pending->dq = false;
  if (!dq && !rows) return SECO_OK;
  SECO_F32_DISPATCH(bwd_nt, p, p.pending->runs, seg, dq, s)
}

}  // namespace seco
