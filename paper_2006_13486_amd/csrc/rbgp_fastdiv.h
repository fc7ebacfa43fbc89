// Division by a number that is known when a kernel is launched, without a division.
//
// A kernel finds its tile, rows and steps by dividing its block and thread numbers by sizes of the mask.  The compiler turns
// such a division into a reciprocal in vector registers and some 25 dependent instructions, two or three times a
// prologue -- before the first table load can be issued, in kernels of 4 to 15 us.  The host computes
// the multiplier instead: three scalar instructions.  Together with the kernel arguments of a prologue in one go (grid_args,
// rbgp_reg_common.h) 800 to 1300 of a wave's 30 000 cycles in the register kernels; us, before -> after: VGG19 conv3 bf16, 8192 columns 13.4 -> 13.0, its fused training step 36.1 -> 35.0, layer 13
// at 1/2 fp32, 512 columns 14.6 -> 14.1, kernels of 5 to 7 us 0.2 to 0.35.
#ifndef RBGP_FASTDIV_H
#define RBGP_FASTDIV_H

#include <cstdint>

namespace rbgp_fast {

// n / d for 0 <= n < 2^31, 1 <= d < 2^31.  With l = ceil(log2 d) and mul = floor(2^(31 + l) / d) + 1 < 2^32 the quotient is
// floor(n mul / 2^(31 + l)): mul d exceeds 2^(31 + l) by at most d <= 2^l, which is what n < 2^31 needs (Granlund and Montgomery,
// Division by Invariant Integers using Multiplication, theorem 4.2).
struct Div {
  uint32_t mul, shift;
};

inline Div div_by(int64_t d) {
  const uint32_t l = d > 1 ? uint32_t(64 - __builtin_clzll(uint64_t(d - 1))) : 0;
  return Div{uint32_t((uint64_t(1) << (31 + l)) / uint64_t(d) + 1), l};
}

__host__ __device__ __forceinline__ int quotient(int n, Div d) {
  return int(uint32_t((uint64_t(uint32_t(n) << 1) * d.mul) >> 32) >> d.shift);
}

}  // namespace rbgp_fast

#endif
