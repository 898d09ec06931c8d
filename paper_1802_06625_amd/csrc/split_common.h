// Building blocks of the kernels on the half-precision matrix cores with split
// operands: fp32 values as the sum of two half-precision parts.
#pragma once
#include <hip/hip_runtime.h>

#include "prune_internal.h"

namespace prune {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
// two complex samples at 8-byte alignment (frames start at any sample)
typedef float pair_u __attribute__((ext_vector_type(4), aligned(8)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4_u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ pair_u ld_pair(const float2 *p) {
  typedef __attribute__((address_space(1))) const pair_u gpair;
  return *(const gpair *)(const pair_u *)p;
}
__device__ __forceinline__ void st_pair(float2 *p, pair_u v) {
  typedef __attribute__((address_space(1))) pair_u gpair;
  *(gpair *)(pair_u *)p = v;
}

// Compiler ordering between the lanes' LDS stores and loads of one wave (the
// hardware runs a wave's LDS instructions in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Largest value of a wave, by cross-lane moves within the vector unit (a
// shuffle would go through the LDS, six dependent round trips).
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_max(int v) {
  return max(v, __builtin_amdgcn_update_dpp(v, v, CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ int wave_max(int v) {
  v = dpp_max<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: lane 15 of each row of 16
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  v = dpp_max<0x142, 0xa>(v);   // row_bcast 15 into rows 1 and 3
  v = dpp_max<0x143, 0xc>(v);   // row_bcast 31 into rows 2 and 3
  return __builtin_amdgcn_readlane(v, 63);
}

// |re + i im| as every forward kernel rounds it (written out: the compiler may
// fuse either square of re * re + im * im).
__device__ __forceinline__ float magnitude(float re, float im) { return sqrtf(fmaf(re, re, im * im)); }

// Sum over a wave, in a fixed order.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_sum(float v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);
  v = dpp_add<0x143, 0xc>(v);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

__device__ __forceinline__ uint32_t abs_bits(float v) { return __builtin_bit_cast(uint32_t, v) & 0x7fffffffu; }

// magnitudes (as bits) that the scaling by powers of two covers
constexpr uint32_t kInf = 0x7f800000u, kLow = 30u << 23, kHigh = 220u << 23;

// Two complex samples (re, im, re, im) as high and low half-precision parts:
// v = high + low to 2^-24 of v, both parts rounded to nearest.  neg1 is -1,
// opaque to the compiler so that the remainder is one mixed-precision FMA.
__device__ __forceinline__ void split_pair(const pair_u v, float neg1, uint32_t *hi, uint32_t *lo) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const floatx2 z = q ? floatx2{v.z, v.w} : floatx2{v.x, v.y};
    const half2v h = __builtin_convertvector(z, half2v);
    const floatx2 r = {fmaf((float)h.x, neg1, z.x), fmaf((float)h.y, neg1, z.y)};
    hi[q] = __builtin_bit_cast(uint32_t, h);
    lo[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, half2v));
  }
}

}  // namespace prune
