// fp32 values as three bfloat16 pieces, for fp32 products on the bf16 matrix cores (Dekker's splitting, with bf16 as the short format).
//
// Every piece is the rest rounded to the nearest bf16 (ties to even), and the rests are exact fp32 differences, so the three pieces add
// up to the value exactly: |p1 - v| <= 2^-8 and |p3| <= 2^-17 of the value's power of two.  (True for magnitudes from 2^-100 to 2^127:
// smaller ones lose what lies below 2^-133, larger ones may round to infinity.)
// A product of two values is then nine products of pieces.  The six from the leading one down to p1 q3, p2 q2 and p3 q1 are taken; what is left
// out, p2 q3 + p3 q2 + p3 q3, is at most 2^-24 of the product, the bound of ONE fp32 rounding, and has either sign.  Pieces cut off by
// truncation would leave out up to 2^-21, always towards zero.
#pragma once
#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#endif
#include <stdint.h>
#include <string.h>

namespace moqe {

#if defined(__HIP_DEVICE_COMPILE__)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
static __device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {   // round to nearest even, a in the low half
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
static __device__ __forceinline__ float float_of_bits(uint32_t u) { return __uint_as_float(u); }
#else
static inline __host__ __device__ uint32_t pack_bf16x2(float a, float b) {
  uint32_t u[2];
  memcpy(&u[0], &a, 4);
  memcpy(&u[1], &b, 4);
  for (int i = 0; i < 2; ++i) u[i] = (u[i] + 0x7fffu + ((u[i] >> 16) & 1u)) >> 16;     // finite values
  return u[0] | u[1] << 16;
}
static inline __host__ __device__ float float_of_bits(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
#endif

// The pieces of a (low halves) and b (high halves).
static __host__ __device__ __forceinline__ void cut3_pair(float a, float b, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
  p1 = pack_bf16x2(a, b);
  a -= float_of_bits(p1 << 16);
  b -= float_of_bits(p1 & 0xffff0000u);
  p2 = pack_bf16x2(a, b);
  a -= float_of_bits(p2 << 16);
  b -= float_of_bits(p2 & 0xffff0000u);
  p3 = pack_bf16x2(a, b);
}

}  // namespace moqe
