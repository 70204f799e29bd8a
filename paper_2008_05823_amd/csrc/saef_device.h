// Device helpers shared by the kernel translation units of the SAEF library.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "saef_internal.h"

namespace saef {

typedef unsigned long long u64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
}

// Streaming accesses: nothing is re-read soon enough to profit from the caches.
__device__ __forceinline__ float ld_nt(const float* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void st_nt(float* p, float v) { __builtin_nontemporal_store(v, p); }

// Word 3 of a raw buffer descriptor on gfx9 parts (32-bit data format, no
// swizzle, no index stride).  A load through a raw buffer resource of n
// bytes returns 0 for a byte offset at or past n, without touching memory,
// and a store there is dropped.
constexpr int kBufWord3 = 0x00020000;
// Cache policy of a buffer access on gfx940 and later: bit 1 = nt (streaming).
constexpr int kAuxNT = 2;

typedef __amdgpu_buffer_rsrc_t Buf;

// A raw buffer resource over [p, p + bytes), bytes < 2^31.  Accesses through
// it take a 32-bit byte offset (a lane offset in a VGPR plus an immediate),
// so no 64-bit address arithmetic is spent per element, and the range check
// in the hardware replaces the per-lane guards of a ragged tail.
__device__ __forceinline__ Buf buf_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kBufWord3);
}
__device__ __forceinline__ float buf_ld(Buf r, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kAuxNT));
}
// x is re-read by the K workers of a tile through one XCD's L2: cached load.
__device__ __forceinline__ float buf_ld_cached(Buf r, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ void buf_st(Buf r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, 0, kAuxNT);
}
// A 64-bit sign word at a wave-uniform byte offset (passed as the scalar
// offset of the access, so no vector register holds the address).
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u64 buf_ld_word(Buf r, uint32_t off) {
  const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, 0, off, 0);
  return ((u64)v.y << 32) | v.x;
}
__device__ __forceinline__ void buf_st_word(Buf r, uint32_t off, u64 w) {
  u32x2 v;
  v.x = (uint32_t)w;
  v.y = (uint32_t)(w >> 32);
  __builtin_amdgcn_raw_buffer_store_b64(v, r, 0, off, 0);
}

// The same with a byte offset of each lane's own.
__device__ __forceinline__ void buf_st_lane_word(Buf r, uint32_t off, uint32_t lo, uint32_t hi) {
  u32x2 v;
  v.x = lo;
  v.y = hi;
  __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 0);
}

// Sign words of a buffer that no wave writes during the kernel, at a
// wave-uniform address: read through the scalar cache (s_load), straight
// into the scalar registers the inline v_cndmask takes as its mask.
typedef __attribute__((address_space(4))) const u64 ConstWord;
__device__ __forceinline__ u64 ld_word_ro(const uint64_t* p) {
  return *(ConstWord*)p;  // an address-space cast (same address)
}

// n consecutive sign words (n a power of two <= 64) of a buffer that the
// kernel also writes: one vector load, lane i holding word w0 + (i mod n)
// (vector loads see this kernel's own earlier stores; the scalar cache
// would not); word_of picks word u out of it into scalar registers.
__device__ __forceinline__ u64 buf_ld_words(Buf r, int w0, int n) {
  const uint32_t off = (uint32_t)(w0 + (int)(threadIdx.x & (unsigned)(n - 1))) * 8u;
  const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
  return ((u64)v.y << 32) | v.x;
}
__device__ __forceinline__ u64 word_of(u64 v, int u) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, u);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), u);
  return ((u64)hi << 32) | lo;
}

// v in a vector register the compiler cannot trace back to a scalar one: a
// loop-invariant operand of the inline v_cndmask (which takes only vector
// registers besides its mask) then stays in a VGPR instead of being copied
// from an SGPR at every use.
__device__ __forceinline__ float in_vgpr(float v) {
  asm volatile("" : "+v"(v));
  return v;
}

// ---- exact layer-wise L1 sum ------------------------------------------------
// S = sum_i floor(|v_i| 2^80), an integer below 2^127 when every |v_i| < 2^19
// and a tensor has at most 2^28 elements.  Per lane the terms are split in
// binary64 so that two plain fp64 sums stay exact (8 VALU operations per
// value instead of a 128-bit integer addition with shifts):
//   a = |v| (exact in binary64), t = a + 1.5 2^22 rounds a to H, a multiple
//   of 2^-30 (a < 2^21 keeps a + 1.5 2^22 in [2^22, 2^23), whose spacing is
//   2^-30); C - t = -H and a - H = a + (C - t) are exact (Sterbenz),
//   |a - H| <= 2^-31.  floor(a 2^80) = H 2^80 + floor((a - H) 2^80), and
//   the floor is a truncation: a - H < 0 only when a >= 2^-31, where a is a
//   multiple of 2^-80 (fp32 spacing at that size), so (a - H) 2^80 is an
//   integer; below 2^-57 the bits under 2^-80 are truncated as the
//   definition says (H = 0 there, a - H = a >= 0).
// With at most 16 values per lane between flushes, -sum H 2^30 <= 2^53 and
// |sum trunc((a - H) 2^80)| <= 16 2^49 = 2^53: both fp64 sums are exact.
// They are then integers h and q, S = h 2^50 + q, and a tile of at most 2^13
// elements keeps |h|, |q| <= 2^62, so lanes and waves are added as two plain
// 64-bit sums; one thread per tile forms the 128-bit integer.  In a build with
// larger tiles h and q are 128-bit.
using TileSum = std::conditional_t<(kTileElems <= 8192), int64_t, __int128>;
struct ExactSum {
  double nh = 0.0;   // -sum of H
  double lq = 0.0;   // sum of trunc((a - H) 2^80)
  float mx = 0.0f;   // largest |v| seen (range check; NaN shows in nh)
  int terms = 0;     // values since the last flush (wave-uniform)
  TileSum h = 0, q = 0;  // flushed sums
  bool bad = false;

  __device__ __forceinline__ void add(float v) {
    const double a = (double)fabsf(v);
    const double t = a + 0x1.8p22;
    const double n = 0x1.8p22 - t;
    nh += n;
    lq += trunc((a + n) * 0x1p80);
    mx = fmaxf(mx, fabsf(v));
  }

  // Moves the two fp64 sums into the integers and clears them.
  __device__ __forceinline__ void flush() {
    bad = bad || !(nh == nh) || !(lq == lq);
    h += to_i64(-nh * 0x1p30);
    q += to_i64(lq);
    nh = 0.0;
    lq = 0.0;
    terms = 0;
  }

  // After `count` more values: flush when another pass could break the
  // 16-values-per-lane bound.
  __device__ __forceinline__ void added(int count) {
    terms += count;
    if (terms > 8) flush();
  }

  __device__ __forceinline__ void finish() {
    flush();
    bad = bad || !(mx < 0x1p19f);
  }

  // An integer of magnitude at most 2^53 held in binary64.
  static __device__ __forceinline__ int64_t to_i64(double v) {
    const double hd = floor(v * 0x1p-32);
    const int32_t hi = (int32_t)hd;
    const uint32_t lo = (uint32_t)(v - hd * 0x1p32);
    return (int64_t)(((u64)(uint32_t)hi << 32) | lo);
  }
};

// Sum of v over the wave, in lane 63: each step adds the lane `ctrl` names
// with a DPP operand (no LDS round trip: the __shfl_xor form cost six).
template <int kCtrl, int kRows>
__device__ __forceinline__ int64_t dpp_add(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, kCtrl, kRows,
                                                            0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)((u64)v >> 32),
                                                            kCtrl, kRows, 0xf, false);
  return v + (int64_t)(((u64)hi << 32) | lo);
}
__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
  v = dpp_add<0x111, 0xf>(v);  // row_shr:1
  v = dpp_add<0x112, 0xf>(v);  // row_shr:2
  v = dpp_add<0x114, 0xf>(v);  // row_shr:4
  v = dpp_add<0x118, 0xf>(v);  // row_shr:8: lane 15 of each row holds its sum
  v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

__device__ __forceinline__ int64_t wave_sum_tile(int64_t v) { return wave_sum_i64(v); }
// The 128-bit form (in every lane).
__device__ __forceinline__ __int128 wave_sum_tile(__int128 v) {
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) {
    const u64 lo = __shfl_xor((unsigned long long)v, off);
    const u64 hi = __shfl_xor((unsigned long long)((unsigned __int128)v >> 64), off);
    v += (__int128)(((unsigned __int128)hi << 64) | lo);
  }
  return v;
}

// A workgroup barrier that orders LDS accesses only, whatever the compiler makes
// of __syncthreads(): no wait for the global stores in flight, which would keep a
// streaming workgroup on its CU until its last store is acknowledged.  (In the
// compression kernels the two measure alike: this compiler's __syncthreads()
// waits for LDS only.)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Per lane: bit `lane` of the 64-bit mask ? if1 : if0, in one VALU op
// (v_cndmask with the mask as its lane condition).  The mask must be the
// same in every lane (a sign word read at a wave-uniform address); it is
// moved to scalar registers explicitly, which costs nothing when it already
// is in one.
__device__ __forceinline__ uint32_t sel_by_bit(u64 mask, uint32_t if1, uint32_t if0) {
  const uint32_t mlo = __builtin_amdgcn_readfirstlane((uint32_t)mask);
  const uint32_t mhi = __builtin_amdgcn_readfirstlane((uint32_t)(mask >> 32));
  const u64 m = ((u64)mhi << 32) | mlo;
  uint32_t r;
  asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(if0), "v"(if1), "s"(m));
  return r;
}
__device__ __forceinline__ float sel_by_bit(u64 mask, float if1, float if0) {
  return __uint_as_float(sel_by_bit(mask, __float_as_uint(if1), __float_as_uint(if0)));
}

// (1/K) * acc, binary64; inv_k is 1/K when K is a power of two (exact), else 0.
__device__ __forceinline__ double mean_of(double acc, double inv_k, int K) {
  return (inv_k != 0.0) ? acc * inv_k : acc / (double)K;
}

// Host: 1/K when K is a power of two (then acc * inv_k == acc / K exactly), else 0.
inline double inv_pow2(int K) { return (K & (K - 1)) == 0 ? 1.0 / (double)K : 0.0; }

// The (row, tile) of workgroup b when each tile has `rows` workgroups: along
// a run, tile by tile, then the next row on the same run.  ti may be past the
// last tile (the grid is rounded up to whole groups).
__device__ __forceinline__ void run_tile_of(unsigned b, int rows, int s, int& row, int64_t& ti) {
  const unsigned xcd = b % kXcds, r = b / kXcds;
  const unsigned j = r & ((1u << s) - 1u);
  const unsigned u = r >> s;
  row = (int)(u % (unsigned)rows);
  const int64_t grp = u / (unsigned)rows;
  ti = ((grp * kXcds + xcd) << s) + j;
}

// Workgroups of 4 waves, one wave per tile.
inline unsigned per_wave_grid(const DevLayout& lay) {
  return (unsigned)((lay.n_tiles + kWaves - 1) / kWaves);
}

}  // namespace saef

// All launches go through hipExtLaunchKernelGGL so that an optional event
// pair (a LaunchEvents `ev` in scope) is stamped by the dispatch itself.
#define SAEF_LAUNCH(kernel, grid, block, shmem, stream, ...) \
  hipExtLaunchKernelGGL(kernel, grid, block, shmem, stream, ev.start, ev.stop, 0, __VA_ARGS__)
