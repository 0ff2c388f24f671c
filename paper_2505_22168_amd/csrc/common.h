// Shared device helpers of the GMNN HIP library (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../../include/gmnn.h"

#define GMNN_WAVE 64

namespace gmnn {

// ---------------------------------------------------------------------------
// packed image vector: three int8 in the low 24 bits
// ---------------------------------------------------------------------------
__host__ __device__ inline int32_t pack_shift(int sx, int sy, int sz) {
  return (sx & 0xff) | ((sy & 0xff) << 8) | ((sz & 0xff) << 16);
}
__host__ __device__ inline void unpack_shift(int32_t p, int& sx, int& sy, int& sz) {
  sx = (int)(int8_t)(p & 0xff);
  sy = (int)(int8_t)((p >> 8) & 0xff);
  sz = (int)(int8_t)((p >> 16) & 0xff);
}
// canonical sort key of a pair inside a row: (j, Sx, Sy, Sz) ascending
__host__ __device__ inline uint64_t pair_key(int j, int sx, int sy, int sz) {
  return ((uint64_t)(uint32_t)j << 24) | ((uint64_t)(sx + 128) << 16) |
         ((uint64_t)(sy + 128) << 8) | (uint64_t)(sz + 128);
}

// ---------------------------------------------------------------------------
// XCD-aware block order.  The 8 XCDs of the chip (each with its own L2) take
// workgroups round-robin by block index; xcd_block maps the launch so that
// XCD x processes one contiguous run of logical blocks (nb split as evenly
// as possible), keeping the neighbour rows that nearby atoms share in one
// L2.  A bijection of [0, nb).
// ---------------------------------------------------------------------------
constexpr int kXcds = 8;
constexpr int kComputeUnits = 256;
__device__ inline int xcd_block(int b, int nb) {
  const int q = nb / kXcds, r = nb % kXcds;
  const int x = b % kXcds, k = b / kXcds;
  return x * q + (x < r ? x : r) + k;
}

// ---------------------------------------------------------------------------
// Dynamic-LDS limit of a kernel on the current device, raised to `bytes` the
// first time a launch needs it.  One process-wide table of (device, kernel)
// -> limit set (fixed size, no heap allocation), guarded by a mutex: safe
// from several host threads, and each device gets its own attribute call.
// ---------------------------------------------------------------------------
inline gmnn_status ensure_lds_limit(const void* kernel, size_t bytes) {
  struct Rec {
    int dev;
    const void* kernel;
    size_t bytes;
  };
  constexpr int kRecs = 512;
  static Rec recs[kRecs];
  static int n_recs = 0;
  static std::mutex mu;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return GMNN_ERR_HIP;
  std::lock_guard<std::mutex> lock(mu);
  int r = 0;
  while (r < n_recs && !(recs[r].dev == dev && recs[r].kernel == kernel)) ++r;
  if (r < n_recs && recs[r].bytes >= bytes) return GMNN_OK;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
    return GMNN_ERR_HIP;
  if (r < n_recs) recs[r].bytes = bytes;
  else if (n_recs < kRecs) recs[n_recs++] = Rec{dev, kernel, bytes};  // a full table only costs repeated calls
  return GMNN_OK;
}

// ---------------------------------------------------------------------------
// split-BF16 operands
// ---------------------------------------------------------------------------
// v - hi for the low bf16 part of v (hi = bf16(v)), with v taken as the
// rounded FP32 value: the empty asm keeps the compiler from fusing the
// product that produced v into the subtraction (an FMA there would give the
// low part of the unrounded product, and kernels that fuse differently would
// disagree in the last bits)
__device__ inline float split_low(float v, __bf16 hi) {
  asm("" : "+v"(v));
  return v - (float)hi;
}

// the three bf16 parts of an FP32 value, 8 significant bits each, nearest even,
// so each remainder is exact in FP32: h + m + l = v exactly for 2^-103 <= |v| <
// 3.396e38 (below, the last parts leave the range of normal bf16 values; above,
// where h rounds to infinity, and for infinities the parts are NaN, so what is
// not finite stays so.  Clamps that keep those values cost 1-2% of an FP32
// evaluation: 2195 -> 2234 us for ten MD steps of 10,626 atoms)
__device__ inline void split3(float v, __bf16& h, __bf16& m, __bf16& l) {
  h = (__bf16)v;
  const float r = split_low(v, h);
  m = (__bf16)r;
  l = (__bf16)(r - (float)m);
}

// split3 of two values at once: the parts come out packed, and one conversion
// makes both parts of a pair (three conversions instead of nine)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ inline void split3_pair(float a, float b, bf16x2& h, bf16x2& m, bf16x2& l) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  asm("" : "+v"(a));  // as in split_low
  asm("" : "+v"(b));
  h = __builtin_convertvector((f32x2{a, b}), bf16x2);
  const float ra = a - (float)h[0], rb = b - (float)h[1];
  m = __builtin_convertvector((f32x2{ra, rb}), bf16x2);
  l = __builtin_convertvector((f32x2{ra - (float)m[0], rb - (float)m[1]}), bf16x2);
}

// ---------------------------------------------------------------------------
// wave-level helpers
// ---------------------------------------------------------------------------
__device__ inline int lane_id() { return __lane_id(); }

// a block barrier that orders LDS accesses only: global loads in flight
// (operands prefetched for a later phase) stay in flight across it, where
// __syncthreads() would wait for them
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The value held by lane l ^ 32 (lane_xor32) or l ^ 16 (lane_xor16), in
// registers: a permlane swap of the value with itself hands every lane its
// partner's copy in one of the two outputs (no LDS round trip, unlike a
// shuffle).
__device__ inline float lane_xor32(float v) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(lane_id() < 32 ? r[1] : r[0]);
}
__device__ inline float lane_xor16(float v) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __uint_as_float(((lane_id() >> 4) & 1) ? r[0] : r[1]);
}

// Sum over the 16 lanes of a row by DPP row rotations (8, 4, 2, 1), in
// registers.  Lane 0 of the row ends with the same value, bit for bit, as
// an xor butterfly over the row (at each level it adds the same two partial
// sums); other lanes hold other orderings of the row sum.
__device__ inline float row16_rot_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, false));  // row_ror:8
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xf, 0xf, false));  // row_ror:4
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x122, 0xf, 0xf, false));  // row_ror:2
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x121, 0xf, 0xf, false));  // row_ror:1
  return v;
}

template <typename T>
__device__ inline T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, GMNN_WAVE);
  return v;
}

// inclusive prefix sum over the 64 lanes
__device__ inline int wave_incl_scan(int v) {
  const int l = lane_id();
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(v, o, GMNN_WAVE);
    if (l >= o) v += t;
  }
  return v;
}

__device__ inline void raise_flag(uint32_t* status, uint32_t f) { atomicOr(status, f); }

}  // namespace gmnn
