// Row kernels of the decoder around the attention: residual add + RMSNorm, its backward, SiLU, cross-entropy and the
// embedding gradient.  All are bound by memory at large sizes and by the number of launches at the sizes of a chunk:
// written as separate framework operators a norm was six launches forward and about twelve backward (convert, square,
// mean, rsqrt, two products ...), and a two-layer training step spent 9 of its 14 ms of GPU time and nearly all of its
// 27 ms of host time on them.  Here each is one launch: a workgroup per row, 16-byte accesses where the row
// length allows, the row kept in registers between the two passes up to kKeep * 256 * V elements.  Sums are fp32 in a
// fixed order (reproducible); rounding follows the operators' (the normalised row is rounded before the gain).
#include "decoder.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "seco.h"

namespace {

constexpr int kThreads = 256, kKeep = 4;

template <typename T, int V> struct alignas(sizeof(T) * V) Vec {
  T v[V];
  __device__ void get(float* f) const {
#pragma unroll
    for (int j = 0; j < V; ++j) f[j] = (float)v[j];
  }
  __device__ void set(const float* f) {
#pragma unroll
    for (int j = 0; j < V; ++j) v[j] = (T)f[j];
  }
};
template <typename T, int V> __device__ __forceinline__ void load(const T* p, float* f) {
  reinterpret_cast<const Vec<T, V>*>(p)->get(f);
}
template <typename T, int V> __device__ __forceinline__ void store(T* p, const float* f) {
  Vec<T, V> x;
  x.set(f);
  *reinterpret_cast<Vec<T, V>*>(p) = x;
}

// Rows in bf16 take the hardware's exponential and logarithm, whose argument is first multiplied by log2(e) in fp32: a
// relative error of about |x| 2^-24, far below the rounding to bf16.  fp32 rows take the full-precision functions.
template <typename T> __device__ __forceinline__ float exp_of(float x) { return sizeof(T) == 4 ? expf(x) : __expf(x); }
template <typename T> __device__ __forceinline__ float log_of(float x) { return sizeof(T) == 4 ? logf(x) : __logf(x); }

struct Sum {
  __device__ static float of(float a, float b) { return a + b; }
};
struct Max {
  __device__ static float of(float a, float b) { return fmaxf(a, b); }
};
// over the workgroup; every thread gets the result.  The barrier at the end frees the scratch for the next call.
template <typename Op> __device__ __forceinline__ float block_reduce(float x) {
  __shared__ float sh[kThreads / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = Op::of(x, __shfl_xor(x, o));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
  __syncthreads();
  x = sh[0];
#pragma unroll
  for (int i = 1; i < kThreads / 64; ++i) x = Op::of(x, sh[i]);
  __syncthreads();
  return x;
}

// Block k of a row, this thread's words: loads are issued for every lane (past the row's end: its last words, dropped), all
// of a row's before the first is used.  Behind a per-lane condition the compiler waits for each load before the next,
// which made a norm three to six memory latencies long.
// KB: blocks of a row kept in registers, as many as the row has, at most kKeep.
template <typename T, int V> __device__ __forceinline__ Vec<T, V> fetch(const T* row, int64_t c, int64_t d) {
  return *reinterpret_cast<const Vec<T, V>*>(row + (c < d ? c : d - V));
}

// EMBED: row r of x is row token[r] of a table of v rows (the embedding of a chunk, which took a launch of its own for rows that
// this one reads anyway: 512 x 1024 3.1 + 3.5 us -> 4.4); a token outside it gives NaN, and 1 in *outside where that is asked for.
template <typename T, int V, int KB, bool EMBED>
__global__ __launch_bounds__(kThreads) void add_rmsnorm_kernel(const T* x, const T* y, const T* gain, T* x_out, T* h,
                                                               float* rstd, int64_t d, const int64_t* token, int64_t v,
                                                               float* outside) {   // (x_out may be x)
  const int64_t row = (int64_t)blockIdx.x * d;
  float kept[KB][V], sum = 0.f;
  bool bad = false;
  if constexpr (EMBED) {
    int64_t t = token[blockIdx.x];
    t += t < 0 ? v : 0;                                  // negative: counted from the end
    bad = t < 0 || t >= v;
    if (bad && outside && threadIdx.x == 0) *outside = 1.f;
    x += (bad ? 0 : t) * d - row;                        // (x + row is then the table's row)
  }
  const bool kept_out = EMBED || y;
  Vec<T, V> xv[KB], yv[KB], gv[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    const int64_t c = ((int64_t)k * kThreads + threadIdx.x) * V;
    xv[k] = fetch<T, V>(x + row, c, d);
    if (!EMBED) yv[k] = fetch<T, V>((y ? y : x) + row, c, d);
    gv[k] = fetch<T, V>(gain, c, d);
  }
#pragma unroll
  for (int k = 0; k < KB; ++k) {                       // first pass: the row, with y added (and rounded) to it
    const int64_t c = ((int64_t)k * kThreads + threadIdx.x) * V;
    if (c < d) {
      xv[k].get(kept[k]);
      if (EMBED) {
#pragma unroll
        for (int j = 0; j < V; ++j) kept[k][j] = bad ? NAN : kept[k][j];
        store<T, V>(x_out + row + c, kept[k]);
      } else if (y) {
        float g[V];
        yv[k].get(g);
#pragma unroll
        for (int j = 0; j < V; ++j) kept[k][j] = (float)(T)(kept[k][j] + g[j]);
        store<T, V>(x_out + row + c, kept[k]);
      }
#pragma unroll
      for (int j = 0; j < V; ++j) sum += kept[k][j] * kept[k][j];
    }
  }
  for (int64_t c = ((int64_t)KB * kThreads + threadIdx.x) * V; c < d; c += kThreads * V) {
    float f[V];
    load<T, V>(x + row + c, f);
    if (EMBED) {
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] = bad ? NAN : f[j];
      store<T, V>(x_out + row + c, f);
    } else if (y) {
      float g[V];
      load<T, V>(y + row + c, g);
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] = (float)(T)(f[j] + g[j]);
      store<T, V>(x_out + row + c, f);
    }
#pragma unroll
    for (int j = 0; j < V; ++j) sum += f[j] * f[j];
  }
  const float r = rsqrtf(block_reduce<Sum>(sum) / (float)d + 1e-6f);
  if (threadIdx.x == 0) rstd[blockIdx.x] = r;
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    const int64_t c = ((int64_t)k * kThreads + threadIdx.x) * V;
    if (c < d) {
      float g[V];
      gv[k].get(g);
#pragma unroll
      for (int j = 0; j < V; ++j) kept[k][j] = (float)(T)(kept[k][j] * r) * g[j];
      store<T, V>(h + row + c, kept[k]);
    }
  }
  for (int64_t c = ((int64_t)KB * kThreads + threadIdx.x) * V; c < d; c += kThreads * V) {
    float f[V], g[V];
    load<T, V>((kept_out ? x_out : x) + row + c, f);      // this thread's own words
    load<T, V>(gain + c, g);
#pragma unroll
    for (int j = 0; j < V; ++j) f[j] = (float)(T)(f[j] * r) * g[j];
    store<T, V>(h + row + c, f);
  }
}

// With n = x rstd and e = d_h gain:  d_x = d_in + rstd (e - n mean(e n)),  d_gain = sum over rows of d_h round(n).
// More rows than workgroups, of up to 256 V elements: a wavefront per row, so that the only barrier is the one before the
// workgroup's share of d_gain leaves (its wavefronts' sums in their order).  Bound by memory latency: a workgroup per row, one row
// after the other, takes a round trip for each of its rows.  bf16, rows x elements: 2048 x 1024 9.7 -> 5.4 us, 8192 x 1024
// 40.5 -> 17.3, 2048 x 2048 11.6 -> 9.6; 256 x 2048 4.1 -> 5.0 and, fp32, 512 x 1024 3.9 -> 4.1: those keep a workgroup per row.
template <typename T, int V, int KB>
__global__ __launch_bounds__(kThreads) void rmsnorm_bwd_rows_kernel(const T* x, const T* gain, const float* rstd, const T* d_h,
                                                                    const T* d_in, T* d_x, float* gain_part, int64_t rows, int64_t d) {
  constexpr int kWaves = kThreads / 64;
  constexpr int kOld = (KB * 64 * V + kThreads - 1) / kThreads;
  __shared__ float sh[kWaves][KB * 64 * V];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* part = gain_part + (int64_t)blockIdx.x * d;
  float dg[KB][V], old[kOld];                             // old: of this thread's elements of the share, under the rows' loads
#pragma unroll
  for (int k = 0; k < kOld; ++k) {
    const int64_t c = k * kThreads + threadIdx.x;
    old[k] = part[c < d ? c : d - 1];
  }
  Vec<T, V> gv[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    gv[k] = fetch<T, V>(gain, (k * 64 + lane) * V, d);
#pragma unroll
    for (int j = 0; j < V; ++j) dg[k][j] = 0.f;
  }
  for (int64_t rr = (int64_t)blockIdx.x * kWaves + wave; rr < rows; rr += (int64_t)DEC_GAIN_BLOCKS * kWaves) {
    const int64_t row = rr * d;
    const float r = rstd[rr];
    Vec<T, V> xv[KB], hv[KB], iv[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int64_t c = (k * 64 + lane) * V;
      xv[k] = fetch<T, V>(x + row, c, d);
      hv[k] = fetch<T, V>(d_h + row, c, d);
      iv[k] = fetch<T, V>((d_in ? d_in : x) + row, c, d);  // (d_x may be d_in: this thread's own words)
    }
    float n[KB][V], e[KB][V], sum = 0.f;
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      if ((k * 64 + lane) * V >= d) continue;
      float g[V];
      xv[k].get(n[k]);
      hv[k].get(e[k]);
      gv[k].get(g);
#pragma unroll
      for (int j = 0; j < V; ++j) {
        n[k][j] *= r;
        dg[k][j] += e[k][j] * (float)(T)n[k][j];
        e[k][j] *= g[j];
        sum += e[k][j] * n[k][j];
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    const float mean = sum / (float)d;
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int64_t c = (k * 64 + lane) * V;
      if (c >= d) continue;
      float f[V];
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] = 0.f;
      if (d_in) iv[k].get(f);
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] += r * (e[k][j] - n[k][j] * mean);
      store<T, V>(d_x + row + c, f);
    }
  }
#pragma unroll
  for (int k = 0; k < KB; ++k)
#pragma unroll
    for (int j = 0; j < V; ++j) sh[wave][(k * 64 + lane) * V + j] = dg[k][j];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOld; ++k) {
    const int64_t c = k * kThreads + threadIdx.x;
    if (c >= d) break;
    float f = old[k];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) f += sh[w][c];
    part[c] = f;
  }
}

// Otherwise a workgroup takes every DEC_GAIN_BLOCKS-th row and adds its share of d_gain to its own row of gain_part.
template <typename T, int V, int KB>
__global__ __launch_bounds__(kThreads) void rmsnorm_bwd_kernel(const T* x, const T* gain, const float* rstd, const T* d_h,
                                                               const T* d_in, T* d_x, float* gain_part, int64_t rows,
                                                               int64_t d) {
  float dg[KB][V];
  Vec<T, V> gv[KB];
  Vec<float, V> old[KB];
  float* part = gain_part + (int64_t)blockIdx.x * d;
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    const int64_t c = ((int64_t)k * kThreads + threadIdx.x) * V;
    gv[k] = fetch<T, V>(gain, c, d);
    old[k] = fetch<float, V>(part, c, d);
#pragma unroll
    for (int j = 0; j < V; ++j) dg[k][j] = 0.f;
  }
  for (int64_t rr = blockIdx.x; rr < rows; rr += DEC_GAIN_BLOCKS) {
    const int64_t row = rr * d;
    const float r = rstd[rr];
    float n[KB][V], e[KB][V], sum = 0.f;
    Vec<T, V> xv[KB], hv[KB], iv[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int64_t c = ((int64_t)k * kThreads + threadIdx.x) * V;
      xv[k] = fetch<T, V>(x + row, c, d);
      hv[k] = fetch<T, V>(d_h + row, c, d);
      iv[k] = fetch<T, V>((d_in ? d_in : x) + row, c, d);  // (d_x may be d_in: this thread's own words)
    }
    auto terms = [&](float* nn, float* ee, const float* g, float* gg) {   // nn = x, ee = d_h on entry
#pragma unroll
      for (int j = 0; j < V; ++j) {
        nn[j] *= r;
        if (gg) gg[j] += ee[j] * (float)(T)nn[j];
        ee[j] *= g[j];
        sum += ee[j] * nn[j];
      }
    };
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int64_t c = ((int64_t)k * kThreads + threadIdx.x) * V;
      if (c < d) {
        float g[V];
        xv[k].get(n[k]);
        hv[k].get(e[k]);
        gv[k].get(g);
        terms(n[k], e[k], g, dg[k]);
      }
    }
    auto far = [&](int64_t c, float* nn, float* ee, float* gg) {           // past what is kept in registers
      float g[V];
      load<T, V>(x + row + c, nn);
      load<T, V>(d_h + row + c, ee);
      load<T, V>(gain + c, g);
      terms(nn, ee, g, gg);
    };
    for (int64_t c = ((int64_t)KB * kThreads + threadIdx.x) * V; c < d; c += kThreads * V) {
      float nn[V], ee[V], gg[V];
      load<float, V>(part + c, gg);
      far(c, nn, ee, gg);
      store<float, V>(part + c, gg);
    }
    const float mean = block_reduce<Sum>(sum) / (float)d;
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int64_t c = ((int64_t)k * kThreads + threadIdx.x) * V;
      if (c < d) {
        float f[V];
#pragma unroll
        for (int j = 0; j < V; ++j) f[j] = 0.f;
        if (d_in) iv[k].get(f);
#pragma unroll
        for (int j = 0; j < V; ++j) f[j] += r * (e[k][j] - n[k][j] * mean);
        store<T, V>(d_x + row + c, f);
      }
    }
    for (int64_t c = ((int64_t)KB * kThreads + threadIdx.x) * V; c < d; c += kThreads * V) {
      float nn[V], ee[V], f[V];
      far(c, nn, ee, nullptr);
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] = 0.f;
      if (d_in) load<T, V>(d_in + row + c, f);
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] += r * (ee[j] - nn[j] * mean);
      store<T, V>(d_x + row + c, f);
    }
  }
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    const int64_t c = ((int64_t)k * kThreads + threadIdx.x) * V;
    if (c < d) {
      float f[V];
      old[k].get(f);
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] += dg[k][j];
      store<float, V>(part + c, f);
    }
  }
}

template <typename T, int V, bool BWD>
__global__ __launch_bounds__(kThreads) void silu_kernel(const T* u, T* a, int64_t n) {   // BWD: a is d_a, in and out
  for (int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * V; i < n; i += (int64_t)gridDim.x * kThreads * V) {
    float f[V], g[V];
    load<T, V>(u + i, f);
    if (BWD) load<T, V>(a + i, g);
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const float s = 1.f / (1.f + exp_of<T>(-f[j]));
      f[j] = BWD ? g[j] * (s * (1.f + f[j] * (1.f - s))) : f[j] * s;
    }
    store<T, V>(a + i, f);
  }
}

template <typename T, int V>
__global__ __launch_bounds__(kThreads) void cross_entropy_kernel(T* logits, const int64_t* target, float* loss, bool grad, int64_t v) {
  const int64_t row = (int64_t)blockIdx.x * v, t = target[blockIdx.x];
  T* l = logits + row;
  float m = -INFINITY;
  for (int64_t c = threadIdx.x * V; c < v; c += kThreads * V) {
    float f[V];
    load<T, V>(l + c, f);
#pragma unroll
    for (int j = 0; j < V; ++j) m = fmaxf(m, f[j]);
  }
  m = block_reduce<Max>(m);
  float sum = 0.f;
  for (int64_t c = threadIdx.x * V; c < v; c += kThreads * V) {
    float f[V];
    load<T, V>(l + c, f);
#pragma unroll
    for (int j = 0; j < V; ++j) sum += exp_of<T>(f[j] - m);
  }
  const bool bad = t != -100 && (t < 0 || t >= v);
  float at_target = 0.f;                       // read in front of the barriers behind which the row is overwritten
  if (loss && threadIdx.x == 0 && t != -100 && !bad) at_target = (float)l[t];
  sum = block_reduce<Sum>(sum);
  if (loss && threadIdx.x == 0) loss[blockIdx.x] = t == -100 ? 0.f : bad ? NAN : m + log_of<T>(sum) - at_target;
  if (!grad) return;
  const float inv = t == -100 ? 0.f : bad ? NAN : 1.f / sum;
  for (int64_t c = threadIdx.x * V; c < v; c += kThreads * V) {
    float f[V];
    load<T, V>(l + c, f);
#pragma unroll
    for (int j = 0; j < V; ++j) f[j] = exp_of<T>(f[j] - m) * inv - (c + j == t ? 1.f : 0.f);
    store<T, V>(l + c, f);
  }
}

// One workgroup per row r; the one of a token's first row adds up all of the token's rows, in order, the others leave.
// What bounds it is the token that occurs most often (padding, a frequent word): one workgroup adds up all of its rows.
// So the rows are first listed, kScan tokens at a time, and then taken kAhead at a time, their loads in flight
// together.  Measured at 1024 columns of bf16, walked one by one, each load behind the last -> here: 4096 rows of one token
// 1275 -> 257 us, of which 5 % are one token 52 -> 21, uniform tokens 17 -> 15; 512 rows 85 -> 33, 8.7 -> 7.2, 4.8 -> 4.9.
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void embedding_bwd_kernel(const T* d_x, const int64_t* token, T* grad, int64_t rows,
                                                                 int64_t d, int64_t v) {
  constexpr int kWaves = kThreads / 64, kTurns = 8, kScan = kTurns * kThreads, kAhead = 16;
  __shared__ int list[kScan], found[kTurns * kWaves];
  auto index = [&](int64_t i) { return token[i] < 0 ? token[i] + v : token[i]; };   // negative: counted from the end
  const int64_t r = blockIdx.x, t = index(r);
  if (t < 0 || t >= v) return;
  float earlier = 0.f;
  for (int64_t i = threadIdx.x; i < r; i += kThreads)
    if (index(i) == t) earlier = 1.f;
  if (block_reduce<Sum>(earlier) != 0.f) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T* out = grad + t * d;
  for (int64_t c0 = 0; c0 < d; c0 += kThreads * V) {
    const int64_t c = c0 + threadIdx.x * V;
    float f[V], x[V];
#pragma unroll
    for (int j = 0; j < V; ++j) f[j] = 0.f;
    for (int64_t i0 = r; i0 < rows; i0 += kScan) {
      uint64_t hit[kTurns];
#pragma unroll
      for (int u = 0; u < kTurns; ++u) {
        const int64_t i = i0 + u * kThreads + threadIdx.x;
        hit[u] = __builtin_amdgcn_ballot_w64(i < rows && index(i < rows ? i : r) == t);
        if (lane == 0) found[u * kWaves + wave] = __builtin_popcountll(hit[u]);
      }
      __syncthreads();
      int n = 0, mine[kTurns];
#pragma unroll
      for (int k = 0; k < kTurns * kWaves; ++k) {        // positions in ascending order of the rows
        if (k % kWaves == wave) mine[k / kWaves] = n;
        n += found[k];
      }
#pragma unroll
      for (int u = 0; u < kTurns; ++u)
        if (hit[u] >> lane & 1)
          list[mine[u] + __builtin_popcountll(hit[u] & (((uint64_t)1 << lane) - 1))] = u * kThreads + threadIdx.x;
      __syncthreads();
      n = __builtin_amdgcn_readfirstlane(n);
      const int64_t at = c < d ? c : d - V;
      auto add = [&](auto ahead, int k0, int there) {     // there: how many are left (uniform, like the row numbers)
        constexpr int A = decltype(ahead)::value;
        Vec<T, V> w[A];
#pragma unroll
        for (int k = 0; k < A; ++k)
          w[k] = *reinterpret_cast<const Vec<T, V>*>(d_x + (i0 + __builtin_amdgcn_readfirstlane(list[k0 + (k < there ? k : 0)])) * d + at);
#pragma unroll
        for (int k = 0; k < A; ++k)
          if (k < there) {
            w[k].get(x);
#pragma unroll
            for (int j = 0; j < V; ++j) f[j] += x[j];
          }
      };
      int k0 = 0;
      for (; n - k0 >= kAhead; k0 += kAhead) add(std::integral_constant<int, kAhead>{}, k0, kAhead);
      for (; k0 < n; k0 += 2) add(std::integral_constant<int, 2>{}, k0, n - k0);
      __syncthreads();                                   // the list and the counts are free again
    }
    if (c < d) {
      load<T, V>(out + c, x);
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] += x[j];
      store<T, V>(out + c, f);
    }
  }
}

// sums[i][c] = the rows of parts[i], added up (n sets of DEC_GAIN_BLOCKS rows of d), and the same rounded.  Bound by latency: a
// workgroup takes 64 columns, its 16 groups of lanes every 16th row each, all of a lane's loads in flight; then the groups in
// order.  (2.5 MB of five gains of 1024: 18 us as a framework sum and 2 for the rounding, 4.5 here.)
template <typename T>
__global__ __launch_bounds__(kThreads) void gain_sums_kernel(const float* parts, float* sums, T* rounded, int64_t d) {
  constexpr int kGroups = 16, kPer = DEC_GAIN_BLOCKS / kGroups;
  __shared__ float sh[kGroups][64];
  const int group = threadIdx.x >> 4, l16 = threadIdx.x & 15;
  const int64_t c0 = (int64_t)blockIdx.x * 64;
  const float* from = parts + (int64_t)blockIdx.y * DEC_GAIN_BLOCKS * d + (int64_t)group * d;
  float x[kPer][4];
#pragma unroll
  for (int k = 0; k < kPer; ++k)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t c = c0 + l16 + 16 * j;
      x[k][j] = from[(int64_t)k * kGroups * d + (c < d ? c : d - 1)];
    }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float f = x[0][j];
#pragma unroll
    for (int k = 1; k < kPer; ++k) f += x[k][j];
    sh[group][l16 + 16 * j] = f;
  }
  __syncthreads();
  const int64_t c = c0 + threadIdx.x;
  if (threadIdx.x >= 64 || c >= d) return;
  float f = sh[0][threadIdx.x];
#pragma unroll
  for (int k = 1; k < kGroups; ++k) f += sh[k][threadIdx.x];
  sums[blockIdx.y * d + c] = f;
  if (rounded) rounded[blockIdx.y * d + c] = (T)f;
}

// Three runs of columns of a matrix to matrices of their own, 16 bytes per thread (u: 16-byte units of a row, u0 and u1 of them in the
// first two runs)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(kThreads) void split_columns_kernel(const u32x4* src, u32x4* a, u32x4* b, u32x4* c, int64_t n, int u, int u0, int u1) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const int64_t row = i / u;
  const int col = (int)(i - row * u);
  const u32x4 x = src[i];
  if (col < u0) a[row * u0 + col] = x;
  else if (col < u0 + u1) b[row * u1 + (col - u0)] = x;
  else c[row * (u - u0 - u1) + (col - u0 - u1)] = x;
}

int status() { return hipGetLastError() == hipSuccess ? SECO_OK : SECO_ERR_LAUNCH; }
bool sizes_ok(int dtype, int64_t rows, int64_t d) {
  return (dtype == SECO_BF16 || dtype == SECO_F32) && rows >= 0 && rows < ((int64_t)1 << 31) && d >= 1;
}
template <typename... P> bool words(P... p) { return (((reinterpret_cast<uintptr_t>(p) & 15u) == 0) && ...); }

}  // namespace

// 16-byte accesses when every row starts on a 16-byte boundary, else element by element
#define DEC_DISPATCH(d, aligned, LAUNCH)                                        \
  if (dtype == SECO_BF16) {                                                     \
    if ((d) % 8 == 0 && (aligned)) { LAUNCH(__bf16, 8); }                       \
    else { LAUNCH(__bf16, 1); }                                                 \
  } else {                                                                      \
    if ((d) % 4 == 0 && (aligned)) { LAUNCH(float, 4); }                        \
    else { LAUNCH(float, 1); }                                                  \
  }

#define DEC_BLOCKS(kernel, T, V, grid, ...)                                                                                \
  if (d <= kThreads * V)                                                                                                  \
    hipLaunchKernelGGL((kernel<T, V, 1>), dim3(grid), dim3(kThreads), 0, (hipStream_t)stream, __VA_ARGS__);               \
  else if (d <= 2 * kThreads * V)                                                                                         \
    hipLaunchKernelGGL((kernel<T, V, 2>), dim3(grid), dim3(kThreads), 0, (hipStream_t)stream, __VA_ARGS__);               \
  else                                                                                                                    \
    hipLaunchKernelGGL((kernel<T, V, kKeep>), dim3(grid), dim3(kThreads), 0, (hipStream_t)stream, __VA_ARGS__)

template <typename T, int V, bool EMBED>
static void launch_norm(const void* x, const void* y, const void* gain, void* x_out, void* h, float* rstd, int64_t rows, int64_t d,
                        const int64_t* token, int64_t v, float* outside, void* stream) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)rows), dim3(kThreads), 0, (hipStream_t)stream, (const T*)x, (const T*)y, (const T*)gain,
                       (T*)x_out, (T*)h, rstd, d, token, v, outside);
  };
  if (d <= kThreads * V) go(add_rmsnorm_kernel<T, V, 1, EMBED>);
  else if (d <= 2 * kThreads * V) go(add_rmsnorm_kernel<T, V, 2, EMBED>);
  else go(add_rmsnorm_kernel<T, V, kKeep, EMBED>);
}

extern "C" int dec_embed_rmsnorm_checked(int dtype, const void* table, const int64_t* token, const void* gain, void* x_out, void* h, float* rstd,
                                         int64_t rows, int64_t d, int64_t v, float* outside, void* stream) {
  if (!sizes_ok(dtype, rows, d) || v < 1) return SECO_ERR_SHAPE;
  if (rows == 0) return SECO_OK;
#define L(T, V) launch_norm<T, V, true>(table, nullptr, gain, x_out, h, rstd, rows, d, token, v, outside, stream)
  DEC_DISPATCH(d, words(table, gain, x_out, h), L)
#undef L
  return status();
}

extern "C" int dec_embed_rmsnorm(int dtype, const void* table, const int64_t* token, const void* gain, void* x_out, void* h, float* rstd,
                                 int64_t rows, int64_t d, int64_t v, void* stream) {
  return dec_embed_rmsnorm_checked(dtype, table, token, gain, x_out, h, rstd, rows, d, v, nullptr, stream);
}

extern "C" int dec_add_rmsnorm(int dtype, const void* x, const void* y, const void* gain, void* x_out, void* h, float* rstd,
                               int64_t rows, int64_t d, void* stream) {
  if (!sizes_ok(dtype, rows, d)) return SECO_ERR_SHAPE;
  if (rows == 0) return SECO_OK;
#define L(T, V) launch_norm<T, V, false>(x, y, gain, x_out, h, rstd, rows, d, nullptr, 0, nullptr, stream)
  DEC_DISPATCH(d, words(x, y, gain, x_out, h), L)
#undef L
  return status();
}

extern "C" int dec_rmsnorm_bwd(int dtype, const void* x, const void* gain, const float* rstd, const void* d_h,
                               const void* d_in, void* d_x, float* gain_part, int64_t rows, int64_t d, void* stream) {
  if (!sizes_ok(dtype, rows, d)) return SECO_ERR_SHAPE;
  if (rows == 0) return SECO_OK;
  const unsigned blocks = rows < DEC_GAIN_BLOCKS ? (unsigned)rows : DEC_GAIN_BLOCKS;
  const unsigned by_wave = (unsigned)std::min<int64_t>(DEC_GAIN_BLOCKS, (rows + kThreads / 64 - 1) / (kThreads / 64));
#define ROWS(T, V, KB)                                                                                                      \
  hipLaunchKernelGGL((rmsnorm_bwd_rows_kernel<T, V, KB>), dim3(by_wave), dim3(kThreads), 0, (hipStream_t)stream, (const T*)x,  \
                     (const T*)gain, rstd, (const T*)d_h, (const T*)d_in, (T*)d_x, gain_part, rows, d)
#define L(T, V)                                                                                                             \
  if (rows > DEC_GAIN_BLOCKS && d <= 64 * V) ROWS(T, V, 1);                                                                 \
  else if (rows > DEC_GAIN_BLOCKS && d <= 128 * V) ROWS(T, V, 2);                                                           \
  else if (rows > 2 * DEC_GAIN_BLOCKS && d <= 256 * V) ROWS(T, V, 4);                                                       \
  else DEC_BLOCKS(rmsnorm_bwd_kernel, T, V, blocks, (const T*)x, (const T*)gain, rstd, (const T*)d_h, (const T*)d_in, (T*)d_x, \
                  gain_part, rows, d)
  DEC_DISPATCH(d, words(x, gain, d_h, d_in, d_x, gain_part), L)
#undef L
#undef ROWS
  return status();
}

extern "C" int dec_gain_sums(int dtype, const float* parts, float* sums, void* rounded, int64_t n, int64_t d, void* stream) {
  if (!sizes_ok(dtype, n, d) || n > 65535) return SECO_ERR_SHAPE;
  if (n == 0) return SECO_OK;
  const dim3 grid((unsigned)((d + 63) / 64), (unsigned)n);
  if (dtype == SECO_BF16)
    hipLaunchKernelGGL(gain_sums_kernel<__bf16>, grid, dim3(kThreads), 0, (hipStream_t)stream, parts, sums, (__bf16*)rounded, d);
  else
    hipLaunchKernelGGL(gain_sums_kernel<float>, grid, dim3(kThreads), 0, (hipStream_t)stream, parts, sums, (float*)rounded, d);
  return status();
}

extern "C" int dec_split_columns(const void* src, void* a, void* b, void* c, int64_t rows, int64_t bytes_a, int64_t bytes_b, int64_t bytes_c,
                                 void* stream) {
  if (rows < 0 || bytes_a < 0 || bytes_b < 0 || bytes_c < 0 || (bytes_a | bytes_b | bytes_c) & 15) return SECO_ERR_SHAPE;
  if (!words(src, a, b, c)) return SECO_ERR_ALIGN;
  const int64_t u = (bytes_a + bytes_b + bytes_c) / 16, n = rows * u;
  if (u > 0x7fffffff || (n + kThreads - 1) / kThreads > 0x7fffffff) return SECO_ERR_TOO_LARGE;
  if (n == 0) return SECO_OK;
  hipLaunchKernelGGL(split_columns_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, (hipStream_t)stream,
                     (const u32x4*)src, (u32x4*)a, (u32x4*)b, (u32x4*)c, n, (int)u, (int)(bytes_a / 16), (int)(bytes_b / 16));
  return status();
}

template <bool BWD> static int silu(int dtype, const void* u, void* a, int64_t n, void* stream) {
  if ((dtype != SECO_BF16 && dtype != SECO_F32) || n < 0) return SECO_ERR_SHAPE;
  if (n == 0) return SECO_OK;
#define L(T, V)                                                                                                        \
  {                                                                                                                    \
    const int64_t blocks = (n + kThreads * V - 1) / (kThreads * V);                                                    \
    hipLaunchKernelGGL((silu_kernel<T, V, BWD>), dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(kThreads), 0,  \
                       (hipStream_t)stream, (const T*)u, (T*)a, n);                                                    \
  }
  DEC_DISPATCH(n, words(u, a), L)
#undef L
  return status();
}
extern "C" int dec_silu(int dtype, const void* u, void* a, int64_t n, void* stream) { return silu<false>(dtype, u, a, n, stream); }
extern "C" int dec_silu_bwd(int dtype, const void* u, void* d_a, int64_t n, void* stream) {
  return silu<true>(dtype, u, d_a, n, stream);
}

static int cross_entropy(int dtype, void* logits, const int64_t* target, float* loss, bool grad, int64_t rows, int64_t v, void* stream) {
  if (!sizes_ok(dtype, rows, v)) return SECO_ERR_SHAPE;
  if (rows == 0) return SECO_OK;
#define L(T, V)                                                                                                     \
  hipLaunchKernelGGL((cross_entropy_kernel<T, V>), dim3((unsigned)rows), dim3(kThreads), 0, (hipStream_t)stream,    \
                     (T*)logits, target, loss, grad, v)
  DEC_DISPATCH(v, words(logits), L)
#undef L
  return status();
}
extern "C" int dec_cross_entropy(int dtype, void* logits, const int64_t* target, float* loss, int64_t rows, int64_t v,
                                 void* stream) {
  return cross_entropy(dtype, logits, target, loss, !loss, rows, v, stream);
}
extern "C" int dec_cross_entropy_both(int dtype, void* logits, const int64_t* target, float* loss, int64_t rows, int64_t v,
                                      void* stream) {
  return cross_entropy(dtype, logits, target, loss, true, rows, v, stream);
}

extern "C" int dec_embedding_bwd(int dtype, const void* d_x, const int64_t* token, void* grad, int64_t rows, int64_t d,
                                 int64_t v, void* stream) {
  if (!sizes_ok(dtype, rows, d)) return SECO_ERR_SHAPE;
  if (rows == 0) return SECO_OK;
#define L(T, V)                                                                                                     \
  hipLaunchKernelGGL((embedding_bwd_kernel<T, V>), dim3((unsigned)rows), dim3(kThreads), 0, (hipStream_t)stream,    \
                     (const T*)d_x, token, (T*)grad, rows, d, v)
  DEC_DISPATCH(d, words(d_x, grad), L)
#undef L
  return status();
}
