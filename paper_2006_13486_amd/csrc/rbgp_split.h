// fp32 operands as sums of three bf16 numbers, for kernels that multiply them on the bf16 matrix core.
#ifndef RBGP_SPLIT_H
#define RBGP_SPLIT_H

#include "rbgp_reg_common.h"

namespace rbgp_split {

using namespace rbgp_reg;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));

// The operands are split as 2^23 times their value: every fp32 number is a multiple of 2^-149, so every part is zero or a
// normal bf16 number however small the operand is.  The sums leave with the factor of both operands taken off.
constexpr float kUp = 0x1p23f, kDown = 0x1p-46f;

// the three bf16 parts of eight fp32 values, times kUp (nearest even each; the differences are exact)
struct Split {
  bf16x8 p[3];
};
__device__ __forceinline__ float bf16_lo(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }
// the parts of two values, a pair each
__device__ __forceinline__ void split2(float y0, float y1, uint32_t (&p)[3]) {
#pragma clang fp contract(off)   // (x * kUp is needed by itself, and a subtraction runs at twice the rate of a fused one)
  const float x0 = y0 * kUp, x1 = y1 * kUp;
  p[0] = bf16_pair(x0, x1);
  const float a = x0 - bf16_lo(p[0]), b = x1 - bf16_hi(p[0]);
  p[1] = bf16_pair(a, b);
  p[2] = bf16_pair(a - bf16_lo(p[1]), b - bf16_hi(p[1]));
}
__device__ __forceinline__ Split split8(const float (&x)[8]) {
  u32x4 p0, p1, p2;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t p[3];
    split2(x[2 * e], x[2 * e + 1], p);
    p0[e] = p[0];
    p1[e] = p[1];
    p2[e] = p[2];
  }
  return Split{{__builtin_bit_cast(bf16x8, p0), __builtin_bit_cast(bf16x8, p1), __builtin_bit_cast(bf16x8, p2)}};
}

__device__ __forceinline__ bf16x16 joined(const u32x4 &lo, const u32x4 &hi) {
  return __builtin_shufflevector(__builtin_bit_cast(bf16x8, lo), __builtin_bit_cast(bf16x8, hi), 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11,
                                 12, 13, 14, 15);
}

// Adds the small products and takes the operands' factors off.  True: one of the sums is not finite, and the fp32 pass has
// to give it.
__device__ __forceinline__ bool add_up(f32x16 &acc, const f32x16 &cor) {
  float zero = 0.f;   // 0, or NaN where a sum is not finite
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    acc[i] = (acc[i] + cor[i]) * kDown;
    zero = __builtin_fmaf(acc[i], 0.f, zero);
  }
  return zero != 0.f;
}
// (every finite sum stays as it is, bit for bit)
__device__ __forceinline__ void take_not_finite(f32x16 &acc, const f32x16 &second) {
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = acc[i] * 0.f == 0.f ? acc[i] : second[i];
}

}  // namespace rbgp_split

#endif
