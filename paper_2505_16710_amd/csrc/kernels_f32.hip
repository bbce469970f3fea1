// fp32 kernels for chunked causal attention: forward, dQ and dK/dV on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 products and sums, 157 TFLOP/s on this GPU), for any head_dim that is a multiple of 4
// up to 256.
//
// The fp32 configuration is small (cfg1: 4 heads, 256-row chunks, 1024 tokens), so what bounds it is how much of the
// GPU a call can occupy and the length of the dependent chains, not bandwidth: a workgroup owns only 16 query rows
// (forward, dQ) or 16 cache rows (dK/dV), its wavefronts divide the other dimension among themselves, and their partial
// results are combined through LDS in wavefront order (one writer per element, fixed order: reproducible).
//
// Operand forms (lane l, i = l % 16, g = l / 16; a contraction may visit its index in any order, so each lane takes
// four consecutive elements with one load and instruction j uses the j-th):
//   row form  X[r0 + i][16 t + 4 g + j]   contraction over head_dim, instruction (t, j)
//   col form  X[r0 + 4 g + r][64 n + 4 i + j]   contraction over rows, instruction r; output (n, j)
// A score tile computed as (rows of X) x (rows of Y) leaves lane l with Y row i and X rows 4 g + r, r = 0..3: exactly
// the second operand of the col form.  An output tile holds head_dim 64 n + 16 g + 4 r + j for the lane's row i.
// What is left behind the groups of 64 is taken in blocks of 16, one element per lane (head_dim 80: 20 products per block of
// 16 rows and operand instead of 32).
//
// A wavefront copies 16 rows with its lanes along the rows (a "block"), 1 KiB per instruction, and turns them in its own
// LDS into the forms it needs.  Loaded in row form straight from memory, 16 neighbouring lanes touch 16 rows, which the
// address unit takes one by one: 16 bytes per clock and CU instead of 64, and all three kernels waited for that (4 heads of
// head_dim 64, 256 rows at position 768: forward 17.2 -> 14.8 us, backward 22.0 -> 18.3; 97 rows at 900: 16.9 -> 14.7 and 21.0 ->
// 18.2).  What bounds them now: the products and vector instructions of the CUs that have a row tile (2 us per 256 cache
// rows of products alone), and 4 - 6 us of launch, first loads and last sums.
// Positions past head_dim repeat the row's last four elements and are multiplied by zero (row form) or dropped (col form);
// rows past the end repeat the last one and are masked.
#include <type_traits>

#include "mfma_tiles.h"
#include "seco_internal.h"

namespace seco {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kRows = 16;   // rows a workgroup owns
// blocks of 16 that every head_dim that NT blocks are used for (SECO_F32_DISPATCH) fills; past head_dim lie later ones
template <int NT> constexpr int kWhole = NT <= 2 ? 0 : NT <= 4 ? 2 : NT <= 5 ? 4 : NT <= 8 ? 5 : NT <= 12 ? 8 : 12;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// LDS image of 16 rows: rows of 16 NT floats, padded by 4
template <int NT> constexpr int kPartRow = 16 * NT + 4;
template <int NT> constexpr int kPart = kRows * kPartRow<NT>;

// ---- a wavefront's copy of 16 rows: lane l takes the 16-byte pieces l, l + 64, ..
template <int NT> struct Block { f32x4 v[NT]; };
// This lane's pieces.  Where a row is a power of two pieces long, piece l + 64 j lies kStep j rows below piece l.
template <int NT> struct Pieces {
  static constexpr bool kEven = 64 % (4 * NT) == 0;
  static constexpr bool kFixed = kEven || NT <= 8;      // offsets kept (twelve of them do not leave the registers)
  static constexpr int kStep = 64 / (4 * NT), kN = kEven ? 1 : kFixed ? NT : 0;
  int lane, D;
  uint32_t off[kN > 0 ? kN : 1];   // bytes from the first row, in a matrix of the given stride
  __device__ __forceinline__ int row(int j) const { return (lane + 64 * j) / (4 * NT); }
  __device__ __forceinline__ int col(int j) const { return min((lane + 64 * j) % (4 * NT) * 4, D - 4); }   // element
  __device__ __forceinline__ Pieces(int lane_, int64_t stride, int D_) : lane(lane_), D(D_) {
#pragma unroll
    for (int j = 0; j < kN; ++j) off[j] = ((uint32_t)row(j) * (uint32_t)stride + (uint32_t)col(j)) * 4u;
  }
  // rows base, base + stride, ..; n of them (at least one): rows past them repeat the last.  (All scalar but the lane.)
  __device__ __forceinline__ void load(Block<NT>& b, const float* base, int64_t stride, int n) const {
    if (kFixed && n >= kRows) {
      const char* from = reinterpret_cast<const char*>(base);
      int step = kEven ? kStep * 4 * (int)stride : 0;
      asm volatile("" : "+s"(step));       // (its multiples are not worth registers of their own throughout a loop)
#pragma unroll
      for (int j = 0; j < NT; ++j) b.v[j] = *reinterpret_cast<const f32x4*>(from + (int64_t)j * step + off[kEven ? 0 : j % (kN > 0 ? kN : 1)]);
    } else {
#pragma unroll
      for (int j = 0; j < NT; ++j) b.v[j] = load4(base + min(row(j), n - 1) * stride + col(j));
    }
  }
  __device__ __forceinline__ void put(float* own, const Block<NT>& b, int lane) const {
#pragma unroll
    for (int j = 0; j < NT; ++j)
      *reinterpret_cast<f32x4*>(own + (lane + 64 * j) / (4 * NT) * kPartRow<NT> + (lane + 64 * j) % (4 * NT) * 4) = b.v[j];
    asm volatile("" : : : "memory");     // (read back by other lanes; a wavefront's LDS accesses are in order)
  }
};
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
// row form of a block in LDS
template <int NT>
__device__ __forceinline__ void rows_of(const float* own, int i, int g, f32x4 (&x)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) x[t] = load4(own + i * kPartRow<NT> + 16 * t + 4 * g);
  asm volatile("" : : : "memory");
}
// ... to be kept as the second operand of a score tile: zero past head_dim
template <int NT>
__device__ __forceinline__ void mask_kept(int D, int g, f32x4 (&x)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) x[t][j] = 16 * t + 4 * g < D ? x[t][j] : 0.f;
}
// (two chains: a tile's products are dependent, 32 cycles each)
template <int NT>
__device__ __forceinline__ f32x4 score(const f32x4 (&x)[NT], const f32x4 (&kept)[NT]) {
  f32x4 s[2] = {zero4(), zero4()};
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j & 1] = mfma4(x[t][j], kept[t][j], s[j & 1]);
  return s[0] + s[1];
}
// 16 rows in col form
template <int NT> struct Cols {
  static constexpr int kF = NT / 4, kR = NT % 4;
  f32x4 full[4][kF > 0 ? kF : 1];
  float rest[4][kR > 0 ? kR : 1];
  // row(r): of this lane's rows 4 g + r, from its first element on; width: elements that are there
  template <typename Row> __device__ __forceinline__ void load(const Row& row, int width, int i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int n = 0; n < kF; ++n) full[r][n] = load4(row(r) + min(64 * n + 4 * i, width - 4));
#pragma unroll
      for (int m = 0; m < kR; ++m) rest[r][m] = row(r)[min(64 * kF + 16 * m + i, width - 1)];
    }
  }
  // of a block in LDS
  __device__ __forceinline__ void of(const float* own, int i, int g) {
    load([&](int r) { return own + (4 * g + r) * kPartRow<NT>; }, 16 * NT, i);
    asm volatile("" : : : "memory");
  }
};
// 16 rows of results: element 64 n + 16 g + 4 r + j of the lane's row i in full[n][j][r], 64 kF + 16 m + 4 g + r in rest[m][r]
template <int NT> struct Acc {
  static constexpr int kF = NT / 4, kR = NT % 4;
  f32x4 full[kF > 0 ? kF : 1][4];
  f32x4 rest[kR > 0 ? kR : 1];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int n = 0; n < kF; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) full[n][j] = zero4();
#pragma unroll
    for (int m = 0; m < kR; ++m) rest[m] = zero4();
  }
  __device__ __forceinline__ void scale(float f) {
#pragma unroll
    for (int n = 0; n < kF; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) full[n][j] *= f;
#pragma unroll
    for (int m = 0; m < kR; ++m) rest[m] *= f;
  }
  __device__ __forceinline__ void add(const Cols<NT>& x, const f32x4& w) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int n = 0; n < kF; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) full[n][j] = mfma4(x.full[r][n][j], w[r], full[n][j]);
#pragma unroll
      for (int m = 0; m < kR; ++m) rest[m] = mfma4(x.rest[r][m], w[r], rest[m]);
    }
  }
  // into an LDS image
  __device__ __forceinline__ void store(float* own, int i, int g) const {
    float* row = own + i * kPartRow<NT>;
#pragma unroll
    for (int n = 0; n < kF; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x4 v = {full[n][0][r], full[n][1][r], full[n][2][r], full[n][3][r]};
        *reinterpret_cast<f32x4*>(row + 64 * n + 16 * g + 4 * r) = v;
      }
#pragma unroll
    for (int m = 0; m < kR; ++m) *reinterpret_cast<f32x4*>(row + 64 * kF + 16 * m + 4 * g) = rest[m];
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

// O = softmax(s Q K^T) V and LSE, of O the columns of NO of the NT blocks (fwd_nt).  The next block's K and V are requested before the present one is worked on.
template <int NT, int NO, int NW>
__global__ __launch_bounds__(NW * 64, NT <= 12 ? 2 : 1) void fwd_f32_kernel(AttnParams p) {
  constexpr int kParts = (NT + NO - 1) / NO;
  constexpr bool kAhead = NT <= 8;                      // (longer rows do not leave the registers)
  extern __shared__ float part[];                       // an image per wavefront; then its (reference, sum) per row
  float* ml = part + NW * kPart<NT>;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;
  const int turn = gridDim.x - 1 - blockIdx.x, r0 = turn / kParts * kRows, h = blockIdx.y, b = blockIdx.z, D = p.D;
  const int o0 = turn % kParts * (16 * NO), n_o = min(D - o0, 16 * NO);   // this workgroup's columns of O
  if (n_o <= 0) return;
  const float* K = static_cast<const float*>(p.k) + b * p.kvs[0] + (h / p.G) * p.kvs[1];
  const float* V = static_cast<const float*>(p.v) + b * p.kvs[0] + (h / p.G) * p.kvs[1] + o0;
  const int64_t row = p.kvs[2];
  const int qpos = p.q_start + r0 + i, kv_end = p.q_start + min(r0 + kRows, p.C);
  float* own = part + w * kPart<NT>;
  Block<NT> kb;
  Cols<NO> vx;
  const Pieces<NT> pk(lane, row, D);
  const uint32_t v_off = (uint32_t)(4 * g) * (uint32_t)row;   // elements
  auto load_k = [&](int c0) { pk.load(kb, K + c0 * row, row, kv_end - c0); };
  auto load_v = [&](int c0) {
    const float* from = V + c0 * row;
    if (c0 + kRows <= kv_end)
      vx.load([&](int r) { return from + r * row + v_off; }, n_o, i);
    else
      vx.load([&](int r) { return V + min(c0 + 4 * g + r, kv_end - 1) * row; }, n_o, i);
  };
  f32x4 qf[NT];
  {
    // (every wavefront brings Q for itself: a barrier here sets them all on the same phase, 15.4 us instead of 14.8)
    Block<NT> qb;
    Pieces<NT>(lane, p.qs[2], D).load(qb, static_cast<const float*>(p.q) + b * p.qs[0] + h * p.qs[1] + r0 * p.qs[2], p.qs[2], p.C - r0);
    if (kAhead && w * 16 < kv_end) load_k(w * 16), load_v(w * 16);
    pk.put(own, qb, lane);
    rows_of<NT>(own, i, g, qf);
    mask_kept<NT>(D, g, qf);
  }
  const float c = p.scale * kLog2e;
  // m: the row's reference in log2 units (-inf before it has seen anything), ref: the same with 0 for -inf; l: this lane's
  // share of the row's sum.  The reference only guards against overflow, so it moves only when a score lies more than
  // kSlack above it.  (Vector instructions and fp32 products take turns on a SIMD, whichever wavefront they come from, so
  // every instruction of the loop counts: with the maximum and the rescaling in every block a call over 1024 rows took
  // 15.5 us, 14.8 without.)
  constexpr float kSlack = 32.f;
  float m = -INFINITY, ref = 0.f, l = 0.f;
  Acc<NO> o;
  o.clear();
#pragma unroll 1
  for (int c0 = w * 16; c0 < kv_end; c0 += NW * 16) {
    if (!kAhead) load_k(c0);
    const bool more = kAhead && c0 + NW * 16 < kv_end;
    f32x4 s;
    {
      f32x4 kx[NT];
      pk.put(own, kb, lane);
      if (more) load_k(c0 + NW * 16);
      rows_of<NT>(own, i, g, kx);
      s = score<NT>(kx, qf);
    }
    if (!kAhead) {                                      // (behind the products: K, its row form and V do not fit together)
      asm volatile("" : "+v"(s) : : "memory");
      load_v(c0);
    }
    s *= c;
    if (c0 + kRows > p.q_start + r0) {                  // a block on the diagonal
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] = c0 + 4 * g + r <= qpos ? s[r] : -INFINITY;
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    if (__builtin_amdgcn_ballot_w64(mx > m + kSlack)) {
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32)));
      ref = mx == -INFINITY ? 0.f : mx;
      const float alpha = fast_exp2(m - ref);
      m = mx;
      l *= alpha;
      o.scale(alpha);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = fast_exp2(s[r] - ref);
      l += s[r];
    }
    o.add(vx, s);
    if (more) load_v(c0 + NW * 16);
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  o.store(own, i, g);
  if (g == 0) {
    ml[(w * kRows + i) * 2] = m;
    ml[(w * kRows + i) * 2 + 1] = l;
  }
  __syncthreads();
  // a wavefront finishes whole rows: its lane (i, g) adds the partials of wavefronts g NW / 4 .. of elements 4 i ..
  for (int r = w; r < min(kRows, p.C - r0); r += NW) {
    float M = -INFINITY, a[NW / 4], L = 0.f;
#pragma unroll
    for (int v = 0; v < NW / 4; ++v) a[v] = ml[((g * (NW / 4) + v) * kRows + r) * 2], M = fmaxf(M, a[v]);
    M = fmaxf(M, __shfl_xor(M, 16));
    M = fmaxf(M, __shfl_xor(M, 32));                    // finite: column 0 is always visible
#pragma unroll
    for (int v = 0; v < NW / 4; ++v) {
      a[v] = fast_exp2(a[v] - M);
      L += a[v] * ml[((g * (NW / 4) + v) * kRows + r) * 2 + 1];
    }
    L += __shfl_xor(L, 16);
    L += __shfl_xor(L, 32);
    float* out = static_cast<float*>(p.o_out) + b * p.os[0] + h * p.os[1] + (r0 + r) * p.os[2] + o0;
#pragma unroll
    for (int d0 = 0; d0 < 16 * NO; d0 += 64) {
      const int d = d0 + 4 * i;
      f32x4 acc = zero4();
#pragma unroll
      for (int v = 0; v < NW / 4; ++v) acc += a[v] * load4(part + (g * (NW / 4) + v) * kPart<NT> + r * kPartRow<NO> + min(d, 16 * NO - 4));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[j] += __shfl_xor(acc[j], 16);
        acc[j] += __shfl_xor(acc[j], 32);
      }
      if (g == 0 && d < n_o) *reinterpret_cast<f32x4*>(out + d) = acc * (1.f / L);
    }
    if (lane == 0 && o0 == 0) p.lse[((int64_t)b * p.Hq + h) * p.C + r0 + r] = (M + __log2f(L)) * kLn2;
  }
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
__device__ __forceinline__ void dq_f32(const AttnParams& p, const Runs& runs, int item_part, float* part) {
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
__device__ __forceinline__ void dkdv_f32(const AttnParams& p, const Runs& runs, int item, float* part) {
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
__global__ __launch_bounds__(NW * 64) void bwd_f32_kernel(AttnParams p, Runs dq_runs, Runs seg, int n_dq) {
  extern __shared__ float part[];                       // two images per wavefront
  if ((int)blockIdx.x < n_dq)
    dq_f32<NT, NO, NW>(p, dq_runs, blockIdx.x, part);
  else
    dkdv_f32<NT, NW>(p, seg, blockIdx.x - n_dq, part);
}

// Wavefronts per workgroup: as many as the register file holds of the kernel at that head_dim.
template <int NT> constexpr int kFwdWaves = NT <= 4 ? 16 : NT <= 8 ? 8 : 4;
template <int NT> constexpr int kBwdWaves = NT <= 8 ? 8 : 4;

template <int NT, int NO>
int fwd_launch(const AttnParams& p, hipStream_t s) {
  constexpr int NW = kFwdWaves<NT>, smem = NW * (kPart<NT> + 2 * kRows) * 4;
  auto kern = fwd_f32_kernel<NT, NO, NW>;
  static std::atomic<uint64_t> ready{0};
  if (!allow_lds(ready, reinterpret_cast<const void*>(kern), smem)) return SECO_ERR_LAUNCH;
  ProfScope prof(kKernelFwd, s);
  hipLaunchKernelGGL(kern, dim3((p.C + kRows - 1) / kRows * ((NT + NO - 1) / NO), p.Hq, p.B), dim3(NW * 64), smem, s, p);
  return launch_status();
}
// Few row tiles: two or four workgroups for each, on CUs that had none, which all compute its scores but only a part of the
// columns of O (or dQ), whose products are half of the work (a third).  As long as that leaves every workgroup a CU: beyond, the
// scores computed again cost more than they save (88 tiles of head_dim 64 by four: 24 us, by two 17.3, whole 18.7).  Forward of 4
// heads of 64, 256 rows at 768: 14.9 -> 11.7 us; 3 heads of 128, 76 rows at 560: 18.2 -> 13.8; 4 of 256, 200 at 400: 37.5 -> 25.0.
// Backward: 64 + 128 tiles of head_dim 64 10.9 -> 10.1 us; 15 + 120 of 128 23.3 -> 19.1 (four); 28 + 252 of 64 18.1 -> 16.5 (two: the
// others' CUs may be shared a little, 64 + 256 gain nothing); 120 + 120 of 128 by two 26.2 -> 28.1.
// Not where O is written over an input: each of them would read query rows that another has overwritten.
template <int NT>
int fwd_nt(const AttnParams& p, hipStream_t s) {
  const int64_t n = (int64_t)((p.C + kRows - 1) / kRows) * p.Hq * p.B, cus = device_cus();
  if (o_over_inputs(p, sizeof(float))) return fwd_launch<NT, NT>(p, s);
  if (n * 4 <= cus) return fwd_launch<NT, (NT + 3) / 4>(p, s);
  if (n * 2 <= cus) return fwd_launch<NT, (NT + 1) / 2>(p, s);
  return fwd_launch<NT, NT>(p, s);
}
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
template <int NT, typename Runs>
int bwd_parts(const AttnParams& p, const Runs& dq_runs, const Runs& seg, int64_t n_dq, int64_t n_kv, hipStream_t s) {
  const int64_t cus = device_cus();
  if constexpr (NT < 16 || std::is_same<Runs, OneRun>::value) {    // (with the table scalar registers are short at the longest rows)
    if (dq_over_inputs(p, sizeof(float))) return bwd_launch<NT, NT>(p, dq_runs, seg, n_dq, n_kv, s);
    if (n_dq * 4 + n_kv <= cus) return bwd_launch<NT, (NT + 3) / 4>(p, dq_runs, seg, n_dq, n_kv, s);
    if (n_dq * 2 + n_kv <= cus + cus / 4) return bwd_launch<NT, (NT + 1) / 2>(p, dq_runs, seg, n_dq, n_kv, s);
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

// head_dim in blocks of 16: the sizes in use exactly, others by the next larger one
#define SECO_F32_DISPATCH(F, ...)                       \
  switch ((p.D + 15) / 16) {                            \
    case 1: case 2: return F<2>(__VA_ARGS__);           \
    case 3: case 4: return F<4>(__VA_ARGS__);           \
    case 5: return F<5>(__VA_ARGS__);                   \
    case 6: case 7: case 8: return F<8>(__VA_ARGS__);   \
    case 9: case 10: case 11: case 12: return F<12>(__VA_ARGS__); \
    default: return F<16>(__VA_ARGS__);                 \
  }

int launch_fwd_f32(const AttnParams& p, hipStream_t s) { SECO_F32_DISPATCH(fwd_nt, p, s) }

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
