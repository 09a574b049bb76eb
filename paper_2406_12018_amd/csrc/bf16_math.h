// Conversions of f32 numbers to bf16 words, shared by the attention kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace citrus {

__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) __bf16 pair_bf16;
  typedef __attribute__((ext_vector_type(2))) float pair_f32;
  const pair_f32 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, pair_bf16));  // round to nearest even
}

// Two numbers as the sums of two bf16 each: hi is the number rounded to nearest, rest what that left, rounded.  Together
// they keep 17 bits of a number (2^-18 relative).
__device__ inline void split_bf16x2(float a, float b, uint32_t& hi, uint32_t& rest) {
  hi = pack_bf16x2(a, b);
  rest = pack_bf16x2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

}  // namespace citrus
