// fp32 operands as sums of three bf16 numbers, for kernels that multiply them on the bf16 matrix core.
#ifndef RBGP_SPLIT_H
#define RBGP_SPLIT_H

#include "rbgp_reg_common.h"

namespace rbgp_split {

using namespace rbgp_reg;

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
__device__ __forceinline__ Split split8(const float (&x)[8]) {
#pragma clang fp contract(off)   // (x * kUp is needed by itself, and a subtraction runs at twice the rate of a fused one)
  u32x4 p0, p1, p2;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x0 = x[2 * e] * kUp, x1 = x[2 * e + 1] * kUp;
    p0[e] = bf16_pair(x0, x1);
    const float a = x0 - bf16_lo(p0[e]), b = x1 - bf16_hi(p0[e]);
    p1[e] = bf16_pair(a, b);
    p2[e] = bf16_pair(a - bf16_lo(p1[e]), b - bf16_hi(p1[e]));
  }
  return Split{{__builtin_bit_cast(bf16x8, p0), __builtin_bit_cast(bf16x8, p1), __builtin_bit_cast(bf16x8, p2)}};
}

}  // namespace rbgp_split

#endif
