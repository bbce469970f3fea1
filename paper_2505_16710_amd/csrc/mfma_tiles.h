// Device-side building blocks for the bf16 matrix-core kernels (gfx950, wave64, head_dim 128).
//
// Operand layouts of v_mfma_f32_32x32x16_bf16 (D = A[32x16] * B[16x32] + C), lane l, g = l / 32:
//   A: row  l % 32, contraction slots 8g .. 8g+7
//   B: col  l % 32, contraction slots 8g .. 8g+7
//   C: col  l % 32, register r holds row 8*(r/4) + 4g + r%4
// so a C tile can be fed back as an A or B operand over 16 contraction steps by taking
// registers 8t .. 8t+7: slot s then stands for index 16t + 8*(s/4) + 4g + s%4 of the
// contracted dimension.  The other operand must present the same slot -> index map; when it
// comes from a row-major LDS tile whose ROWS are contracted, the LDS transpose read
// (ds_read_b64_tr_b16: lane i of a 16-lane group receives element i%4 of the 8 bytes
// addressed by lanes i/4, 4+i/4, 8+i/4, 12+i/4) delivers exactly that.
//
// Operand layouts of v_mfma_f32_16x16x32_bf16 (D = A[16x32] * B[32x16] + C), lane l, g = l / 16:
//   A: row  l % 16, contraction slots 8g .. 8g+7
//   B: col  l % 16, contraction slots 8g .. 8g+7
//   C: col  l % 16, register r holds row 4g + r
// so two C tiles of 16 rows each make an operand over 32 contraction steps (pack44): slots 0-3 of group g are the first
// tile's rows 4g .. 4g+3, slots 4-7 the second's.  Which row of an LDS tile stands for which row of A is free as long as
// both products agree: row 4q + i of A is tile row 4 pi(q) + i, pi = 0, 2, 3, 1, the order in which neither the row
// reads (served in groups of lanes 0-3, 12-15, 20-23, 24-27 and so on) nor the transpose reads (half-waves) have two
// lanes on a bank; in plain order both took twice the LDS cycles.
//
// LDS tiles are row-major, 256 bytes per row (128 bf16), with the sixteen 16-byte chunks of a
// row XOR-swizzled by a function of the row number so that the access patterns are free of
// bank conflicts: 16 lanes reading the same chunk of 16 consecutive rows, the transpose
// read's 4 rows x 64 bytes per half-wave, and those of the 16-row operands above.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "xcd_map.h"

namespace seco {

// Lets a kernel use more than the default 64 KiB of dynamic LDS.  The attribute belongs to the kernel on a device:
// set by the first launch there (`ready`: one bit per device, one variable per kernel), not by every launch.
inline bool allow_lds(std::atomic<uint64_t>& ready, const void* kernel, int bytes) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  const uint64_t bit = (uint64_t)1 << (dev & 63);
  if (dev < 64 && (ready.load(std::memory_order_acquire) & bit)) return true;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return false;
  ready.fetch_or(bit, std::memory_order_release);
  return true;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

#define SECO_LDS __attribute__((address_space(3)))
typedef SECO_LDS char lds_char;

constexpr int kHeadDim = 128;
constexpr int kRowBytes = kHeadDim * 2;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ int swz(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

// byte offset of 16-byte chunk `chunk` (0..15) of row `row` inside a tile
__device__ __forceinline__ int tile_off(int row, int chunk) { return row * kRowBytes + ((chunk ^ swz(row)) << 4); }

// 8 consecutive head_dim elements of one row (operand whose contraction runs along head_dim)
__device__ __forceinline__ bf16x8 lds_row8(lds_char* tile, int row, int chunk) {
  return *reinterpret_cast<SECO_LDS bf16x8*>(tile + tile_off(row, chunk));
}

__device__ __forceinline__ void lds_store16(lds_char* tile, int row, int chunk, bf16x8 v) {
  *reinterpret_cast<SECO_LDS bf16x8*>(tile + tile_off(row, chunk)) = v;
}

// Operand whose contraction runs along the tile's ROWS: for head_dim column 32*db + lane%32,
// slots s = 0..7 hold rows row0 + 8*(s/4) + 4*(lane/32) + s%4.
__device__ __forceinline__ bf16x8 lds_tr8(lds_char* tile, int row0, int db, int lane) {
  const int ii = lane & 15, half = (lane >> 4) & 1, g = lane >> 5;
  const int row = row0 + 4 * g + (ii >> 2);
  const int chunk = 4 * db + 2 * half + ((ii & 3) >> 1);
  const int sub = (ii & 1) << 3;
  s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<SECO_LDS s16x4*>(tile + tile_off(row, chunk) + sub));
  s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      reinterpret_cast<SECO_LDS s16x4*>(tile + tile_off(row + 8, chunk) + sub));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  s16x8 r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, r);
}

// The same two reads with the lane-dependent part of the address taken out of the loop.  tile_off(row0 + r, chunk)
// = row0 * kRowBytes + tile_off(r, chunk) whenever row0 is a multiple of 16 (the swizzle looks at the low four row
// bits only), so a kernel can compute these offsets once; an access in its main loop is then
// tile base + per-lane offset (one add per tile and offset) + a compile-time constant folded into the instruction.
struct TrOff { int lo, hi; };     // rows r and r + 8 of lds_tr8
__device__ __forceinline__ int row8_lane_off(int l32, int chunk) { return tile_off(l32, chunk); }
__device__ __forceinline__ TrOff tr8_lane_off(int db, int lane) {
  const int ii = lane & 15, half = (lane >> 4) & 1, g = lane >> 5;
  const int row = 4 * g + (ii >> 2);
  const int chunk = 4 * db + 2 * half + ((ii & 3) >> 1);
  const int sub = (ii & 1) << 3;
  return {tile_off(row, chunk) + sub, tile_off(row + 8, chunk) + sub};
}
__device__ __forceinline__ bf16x8 lds_row8_at(lds_char* tile_plus_off, int row0) {   // row0: multiple of 32
  return *reinterpret_cast<SECO_LDS bf16x8*>(tile_plus_off + row0 * kRowBytes);
}
__device__ __forceinline__ bf16x8 lds_tr8_at(lds_char* tile, TrOff off, int row0) {   // row0: multiple of 16
  s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<SECO_LDS s16x4*>(tile + off.lo + row0 * kRowBytes));
  s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<SECO_LDS s16x4*>(tile + off.hi + row0 * kRowBytes));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  s16x8 r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// (pi of the operand layouts above, of a lane group)
__device__ __forceinline__ int pi4(int group) { return ((group & 1) << 1) ^ ((group >> 1) * 3); }
// operand over 32 contraction rows from two C tiles of 16 of them
__device__ __forceinline__ bf16x8 pack44(const f32x4& x, const f32x4& y) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x2 v = i < 2 ? f32x2{x[2 * i], x[2 * i + 1]} : f32x2{y[2 * i - 4], y[2 * i - 3]};
    r[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  }
  return __builtin_bit_cast(bf16x8, r);
}
// Per-lane offsets of operands in a tile, constant for a whole kernel, and the reads themselves (row0: multiple of 16):
// 16 rows (lane: row pi(l % 16)), contraction 32 t .. 32 t + 31 of head_dim
__device__ __forceinline__ int row16_lane_off(int t, int lane) {
  return tile_off(4 * pi4((lane >> 2) & 3) + (lane & 3), 4 * t + (lane >> 4));
}
__device__ __forceinline__ bf16x8 lds_at(lds_char* tile_plus_off, int row0) {
  return *reinterpret_cast<SECO_LDS bf16x8*>(tile_plus_off + row0 * kRowBytes);
}
// head_dim column 16 db + lane % 16, contraction over the 32 rows from row0 on, slots as pack44's
__device__ __forceinline__ int tr16_lane_off(int db, int lane) {
  const int ii = lane & 15;
  return tile_off(4 * pi4(lane >> 4) + (ii >> 2), 2 * db + ((ii & 3) >> 1)) + ((ii & 1) << 3);
}
__device__ __forceinline__ bf16x8 lds_tr16_at(lds_char* tile_plus_off, int row0) {
  lds_char* a = tile_plus_off + row0 * kRowBytes;
  const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<SECO_LDS s16x4*>(a));
  const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<SECO_LDS s16x4*>(a + 16 * kRowBytes));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x8 r = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
  return __builtin_bit_cast(bf16x8, r);
}
__device__ __forceinline__ bf16x8 lds_row16(lds_char* tile, int row0, int t, int lane) { return lds_at(tile + row16_lane_off(t, lane), row0); }
__device__ __forceinline__ bf16x8 lds_tr16(lds_char* tile, int row0, int db, int lane) { return lds_tr16_at(tile + tr16_lane_off(db, lane), row0); }

// registers 8t .. 8t+7 of a C tile, rounded to bf16 (pairwise, one v_cvt_pk_bf16_f32 per pair),
// as an operand over 16 contraction steps
__device__ __forceinline__ bf16x8 pack8(const f32x16& x, int t) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x2 v = {x[8 * t + 2 * i], x[8 * t + 2 * i + 1]};
    r[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  }
  return __builtin_bit_cast(bf16x8, r);
}

// Asynchronous copy of four 256-byte rows (rows r .. r+3 of a swizzled tile, r wavefront-uniform)
// from global memory straight into LDS with global_load_lds_dwordx4: lane i's 16 bytes land at
// dst + 16*i, so the swizzle is applied by choosing which 16-byte chunk of its source row the
// lane fetches.  `row_ptr` is this lane's source row (lane / 16 selects the row), already
// clamped by the caller.  The copy is tracked by vmcnt only: the issuing wavefront must call
// dma_wait_all() before the barrier that publishes the tile.  (Issued as inline assembly on
// purpose: with the compiler builtin every later LDS read in the loop is made to wait for the
// copy, because the destination cannot be told apart from the tiles being read.)
__device__ __forceinline__ void dma4rows(lds_char* dst_tile, int r, const __bf16* row_ptr, int lane) {
  const int row = r + (lane >> 4);
  const int chunk = (lane & 15) ^ swz(row);
  const uint32_t m = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(dst_tile + r * kRowBytes));
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(row_ptr + chunk * 8), "s"(m) : "memory", "m0");
}
// Same copy with the address split into a wavefront-uniform 64-bit base (held in scalar registers) and a per-lane
// 32-bit byte offset that does not change from tile to tile: no vector arithmetic per copy.  `lds_dst` must be
// wavefront-uniform and already in a scalar register (e.g. derived from __builtin_amdgcn_readfirstlane).
__device__ __forceinline__ void dma16_sbase(const void* base_uniform, uint32_t lane_off_bytes, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_off_bytes), "s"(base_uniform), "s"(lds_dst) : "memory", "m0");
}
// per-lane byte offset of the 16-byte chunk this lane fetches when rows r .. r+3 (r % 4 == 0) of a tile whose
// source rows are `row_stride_bytes` apart are copied by one dma16_sbase
__device__ __forceinline__ uint32_t dma_lane_offset(int r, int64_t row_stride_bytes, int lane) {
  const int row = r + (lane >> 4);
  return (uint32_t)(row * row_stride_bytes) + (uint32_t)((((lane & 15) ^ swz(row))) << 4);
}
// The same value to the compiler's eyes a new one: destinations derived from it are added up where they are used instead
// of being kept, one scalar register each, over a whole loop (where scalar registers run out, in the kernel that holds
// both passes of the backward).
__device__ __forceinline__ uint32_t opaque(uint32_t scalar) {
  asm volatile("" : "+s"(scalar));
  return scalar;
}
__device__ __forceinline__ void dma_wait_all() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// rowsum(x * y) of 16 rows, x and y as operands (lane l: some row for l % 16, the same in both; fragment t: chunk 4 t + l / 16): the
// diagonal of X Y^T.  Every lane gets the sum of its row.  Four matrix instructions and a dozen others, where products in fp32 and a
// sum over lanes take a hundred; all kernels that need such sums take this one, so that they have the same bits.
__device__ __forceinline__ float row16_dot(const bf16x8* x, const bf16x8* y, int lane) {
  f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 4; ++t) d = mfma16(x[t], y[t], d);
  // element (i, i) is register i % 4 of lane i + 16 (i / 4)
  const float mine = lane & 2 ? (lane & 1 ? d[3] : d[2]) : lane & 1 ? d[1] : d[0];
  return __shfl(mine, (lane & 15) + 4 * (lane & 12));
}

// An address that is the same for all lanes of a wavefront, in scalar registers, and a load from there with a 32-bit lane offset
typedef __attribute__((address_space(1))) const char* global_bytes;
__device__ __forceinline__ global_bytes scalar_address(const void* p) {
  const uint64_t at = (uint64_t)(uintptr_t)p;
  return (global_bytes)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(at >> 32)) << 32 |
                        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)at));
}
__device__ __forceinline__ bf16x8 global_load16(global_bytes from, uint32_t lane_off) {
  return *reinterpret_cast<__attribute__((address_space(1))) const bf16x8*>(from + lane_off);
}

// Make the compiler wait, here, for the load that produces `v`.  Used on operand fragments that are
// loaded once before a loop: otherwise the first use inside the loop carries a conservative vmcnt wait
// on every iteration, which would also wait for the asynchronous tile copies issued in the loop.
__device__ __forceinline__ void settle(const bf16x8& v) { asm volatile("" : : "v"(v)); }
// ... for eight of them at once: all eight loads are in flight before the first one is waited for
__device__ __forceinline__ void settle8(const bf16x8 (&v)[8]) {
  asm volatile("" : : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
}

// Fragments of 32 rows (lane: row l % 32, chunks 2 t + l / 32), taken from memory with whole 256-byte rows per 16 lanes
// and turned through 8 KiB of LDS that belong to the wavefront (no barrier: a wavefront's LDS accesses are in order).
// Loaded straight into their layout the fragments are 32 bytes of each of 32 rows per instruction, which the address
// unit takes one cache line at a time: about 57 cycles per instruction and CU, 11e3 cycles before a dQ workgroup of
// 8 wavefronts could start; whole rows take 16.
// (base, row0: the same for a wavefront.  From a scalar address and 32-bit lane offsets, a row stride being less than 2^24 bytes: with
// 64-bit row numbers times strides the 24 loads of a dQ wavefront are 240 vector instructions.)
__device__ __forceinline__ void load_rows32(bf16x8 (&x)[8], const __bf16* base, int64_t stride, int row0, int last_row, int lane) {
  const int first = __builtin_amdgcn_readfirstlane(min(row0, last_row));
  global_bytes from = scalar_address(base + first * stride);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t r = (uint32_t)min(4 * j + (lane >> 4), last_row - first);
    x[j] = global_load16(from, __umul24(r, (uint32_t)stride * 2u) + (uint32_t)(lane & 15) * 16u);
  }
}
__device__ __forceinline__ void rows32_to_frags(bf16x8 (&f)[8], const bf16x8 (&x)[8], lds_char* own8k, int lane) {
#pragma unroll
  for (int j = 0; j < 8; ++j) lds_store16(own8k, 4 * j + (lane >> 4), lane & 15, x[j]);
#pragma unroll
  for (int t = 0; t < 8; ++t) f[t] = lds_row8(own8k, lane & 31, 2 * t + (lane >> 5));
}
// As operands over 32 contraction steps: fragment 4 qb + t is rows 16 qb + l % 16, chunks 4 t + l / 16
__device__ __forceinline__ void rows16_to_frags(bf16x8 (&f)[8], const bf16x8 (&x)[8], lds_char* own8k, int lane) {
#pragma unroll
  for (int j = 0; j < 8; ++j) lds_store16(own8k, 4 * j + (lane >> 4), lane & 15, x[j]);
#pragma unroll
  for (int t = 0; t < 8; ++t) f[t] = lds_row8(own8k, 16 * (t >> 2) + (lane & 15), 4 * (t & 3) + (lane >> 4));
}
// The way back: a 128 x 32 accumulator whose lanes own rows (lane: row l % 32, register 4 r4 + i of block db: column
// 32 db + 8 r4 + 4 (l / 32) + i) as bf16 to rows of memory, whole rows at a time.
template <typename F>
__device__ __forceinline__ void store_rows32(const F& value, __bf16* base, int64_t stride, int row0, int n_rows,
                                             lds_char* own8k) {   // value(db, register): the element
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));        // (derived again here, so that no address is kept in registers across the main loop)
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (__bf16)value(db, 4 * r4 + i);
      *reinterpret_cast<SECO_LDS bf16x4*>(own8k + tile_off(lane & 31, 4 * db + r4) + 8 * (lane >> 5)) = v;
    }
  const int r0 = row0 + (lane >> 4);
  __bf16* dst = base + (int64_t)r0 * stride + (lane & 15) * 8;
#pragma unroll
  for (int j = 0; j < 8; ++j, dst += 4 * stride)
    if (r0 + 4 * j < n_rows) *reinterpret_cast<bf16x8*>(dst) = lds_row8(own8k, 4 * j + (lane >> 4), lane & 15);
}

// The same for an accumulator of 16 x 16 tiles: value(db, qb, i) is column 16 db + 4 (l / 16) + i of row 16 qb + l % 16
template <typename F>
__device__ __forceinline__ void store_rows16(const F& value, __bf16* base, int64_t stride, int row0, int n_rows, lds_char* own8k) {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int qb = 0; qb < 2; ++qb)
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (__bf16)value(db, qb, i);
      *reinterpret_cast<SECO_LDS bf16x4*>(own8k + tile_off(16 * qb + (lane & 15), 2 * db + (lane >> 5)) + 8 * ((lane >> 4) & 1)) = v;
    }
  const int r0 = row0 + (lane >> 4);
  __bf16* dst = base + (int64_t)r0 * stride + (lane & 15) * 8;
#pragma unroll
  for (int j = 0; j < 8; ++j, dst += 4 * stride)
    if (r0 + 4 * j < n_rows) *reinterpret_cast<bf16x8*>(dst) = lds_row8(own8k, 4 * j + (lane >> 4), lane & 15);
}

// The same accumulator, fp32 and unscaled, to consecutive 512-byte rows (16.5 KiB of LDS)
__device__ __forceinline__ void store_part32(const f32x16 (&acc)[4], float* base, int n_rows, lds_char* own) {
  constexpr int kRow = 528;             // bytes; 16 of padding
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const f32x4 v = {acc[db][4 * r4], acc[db][4 * r4 + 1], acc[db][4 * r4 + 2], acc[db][4 * r4 + 3]};
      *reinterpret_cast<SECO_LDS f32x4*>(own + (lane & 31) * kRow + (32 * db + 8 * r4 + 4 * (lane >> 5)) * 4) = v;
    }
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int r = 2 * j + (lane >> 5);
    const f32x4 v = *reinterpret_cast<SECO_LDS f32x4*>(own + r * kRow + (lane & 31) * 16);
    if (r < n_rows) *reinterpret_cast<f32x4*>(base + r * kHeadDim + (lane & 31) * 4) = v;
  }
}

// ... of 16 x 16 tiles (as store_rows16)
__device__ __forceinline__ void store_part16(const f32x4 (&acc)[8][2], float* base, int n_rows, lds_char* own) {
  constexpr int kRow = 528;             // bytes; 16 of padding
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int db = 0; db < 8; ++db)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
      *reinterpret_cast<SECO_LDS f32x4*>(own + (16 * qb + (lane & 15)) * kRow + (16 * db + 4 * (lane >> 4)) * 4) = acc[db][qb];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int r = 2 * j + (lane >> 5);
    const f32x4 v = *reinterpret_cast<SECO_LDS f32x4*>(own + r * kRow + (lane & 31) * 16);
    if (r < n_rows) *reinterpret_cast<f32x4*>(base + r * kHeadDim + (lane & 31) * 4) = v;
  }
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// How a kernel that owns row tiles divides them among workgroups: not at all; every packed row tile into p.n_splits; only
// those beyond the first round (row_shares)
enum { kWholeTiles = 0, kDivided = 1, kShares = 2 };

}  // namespace seco
