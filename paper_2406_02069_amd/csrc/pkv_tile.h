// Lane-level pieces shared by the scoring kernels that multiply 32 x 32 tiles of keys and query rows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pkv_lds.h"

namespace pkv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned long long u64;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ bf16x8 as_frag(u32x4 u) { return __builtin_bit_cast(bf16x8, u); }
#define PKV_MFMA32(A, B, C) __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, B, C, 0, 0, 0)
// A value the compiler must treat as new: lane constants derived from it are recomputed where they are used instead of
// being kept (and spilled) across the whole item loop.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
template <bool MAX>
__device__ __forceinline__ float both_halves(float x) {
  const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false));
  const float p = __uint_as_float(r[0]), q = __uint_as_float(r[1]);
  return MAX ? fmaxf(p, q) : p + q;
}
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
// Row of a product's element v in lane half 0 (4 more in the other half).
__device__ __forceinline__ constexpr int mrow0(int v) { return 8 * (v >> 2) + (v & 3); }

// Sums of 16 registers over the 32 lanes of a wave half: the sum of register 8 b4 + 4 b3 + 2 b2 + b1 arrives in the lanes
// whose number has these bits.
__device__ __forceinline__ float transpose_sum(const f32x16& t, int lane) {
  float u[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(t[v]), __float_as_uint(t[v + 8]), false, false));
    u[v] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const float mine = b3 ? u[v + 4] : u[v], other = b3 ? u[v] : u[v + 4];
    u[v] = mine + dpp<0x128>(other);  // row_ror:8
  }
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const float mine = b2 ? u[v + 2] : u[v], other = b2 ? u[v] : u[v + 2];
    u[v] = mine + dpp<0x141>(other);  // row_half_mirror
  }
  const float mine = b1 ? u[1] : u[0], other = b1 ? u[0] : u[1];
  const float s = mine + dpp<0x4E>(other);  // quad_perm 2,3,0,1
  return s + dpp<0xB1>(s);                  // quad_perm 1,0,3,2
}
// ... of a product whose rows are keys: the key (of the tile's 32) whose sum arrives in a lane.
__device__ __forceinline__ int transpose_key(int lane) { return (lane & 24) + 4 * (lane >> 5) + ((lane & 6) >> 1); }

// Sums of exponentials as integers, so that the order in which they are added does not show; large ones in further words.
constexpr float kSumUnits = 0x1p30f, kSumUnits2 = 0x1p11f, kSumUnits3 = 0x1p-19f, kSumUnits4 = 0x1p-49f;  // to the 1
constexpr float kSumLimit = 0x1p13f, kSumLimit2 = 0x1p43f, kSumLimit3 = 0x1p73f, kSumLimit4 = 0x1p103f;   // of an item's sum (256 of them stay below bit 52)
__device__ __forceinline__ u64 fixed_point(float z, float scale) {
  const float y = rintf(z * scale);
  const float hi = floorf(y * 0x1p-32f);
  return (u64)(uint32_t)hi << 32 | (uint32_t)__builtin_fmaf(hi, -0x1p32f, y);
}
__device__ __forceinline__ float as_float(u64 w) { return __builtin_fmaf((float)(uint32_t)(w >> 32), 0x1p32f, (float)(uint32_t)w); }
// The sum of all words (first: the one of small sums, as a float).
__device__ __forceinline__ float sum_of_words(float first, u64 b2, u64 b3, u64 b4) {
  const float z = __builtin_fmaf(as_float(b2), 1.f / kSumUnits2, first * (1.f / kSumUnits));
  return __builtin_fmaf(as_float(b4), 1.f / kSumUnits4, __builtin_fmaf(as_float(b3), 1.f / kSumUnits3, z));
}

}  // namespace
}  // namespace pkv
