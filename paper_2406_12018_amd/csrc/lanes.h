// Exchanges between lanes in the vector registers: a data-parallel-primitive move or a row swap is one vector instruction, where
// __shfl_xor is a round trip through the LDS unit of about a hundred cycles.  us with round trips | so: instruction score, 64 rows
// over 1280 keys, 1 layer of 32/8 heads 12.6 | 11.8, 16 layers 31.9 | 30.1, head_dim 64, 64 layers 86.9 | 80.8; f32, 8 rows over 96
// keys 8.8 | 8.3; the tiny f32 document 198 | 191.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace citrus {
namespace {

// What lane f(l) holds, f a move within rows of 16 lanes.
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor3 = 0x1B, kXor7 = 0x141, kXor8 = 0x128;  // l ^ 1, l ^ 2, ...
constexpr int kBack4 = 0x124;  // lane l - 4 of the row (its own inverse where lanes 8 apart hold the same)
template <int F>
__device__ __forceinline__ float from_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), F, 0xf, 0xf, true));
}
// The rows of 16 lanes of a and b, even ones in the first and odd ones in the second: {a0, b0, a2, b2}, {a1, b1, a3, b3}.
__device__ __forceinline__ void swap_rows(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
  a = __int_as_float(r[0]);
  b = __int_as_float(r[1]);
}
// v of lanes l and l ^ 16, l and l ^ 32 (in some order)
__device__ __forceinline__ void both_of_rows(float v, float& a, float& b) {
  a = b = v;
  swap_rows(a, b);
}
__device__ __forceinline__ void both_of_halves(float v, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
  a = __int_as_float(r[0]);
  b = __int_as_float(r[1]);
}
// Sums grow in one order, lanes 16, 8, 4, 2 and 1 apart: which of two nearly equal scores is the larger one depends on it.
// over the 16 lanes of a row
__device__ __forceinline__ float row_sum(float v) {
  v += from_lane<kXor8>(v);
  v += from_lane<kBack4>(v);  // l ^ 4, or l ^ 12, which holds the same
  v += from_lane<kXor2>(v);
  return v + from_lane<kXor1>(v);
}

// Sum of 16 per-lane values over the 32 lanes that share lane / 32: each step
// halves the values a lane still carries (the lane keeps the half its own bit selects and takes
// the partner's partial sum of the same half).  On return lane c holds, for value index c / 2,
// the total over its 32 lanes.  (col: lane % 32)
__device__ __forceinline__ float reduce16_over32(const float (&v)[16], int col) {
  float a[8], b[4], c[2];
  const bool u8 = col & 8, u4 = col & 4, u2 = col & 2;
#pragma unroll
  for (int x = 0; x < 8; ++x) {  // a lane of an even row keeps the lower half of the values
    float lo = v[x], hi = v[x + 8];
    swap_rows(lo, hi);
    a[x] = lo + hi;
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) b[x] = (u8 ? a[x + 4] : a[x]) + from_lane<kXor8>(u8 ? a[x] : a[x + 4]);
#pragma unroll
  for (int x = 0; x < 2; ++x) c[x] = (u4 ? b[x + 2] : b[x]) + from_lane<kXor3>(from_lane<kXor7>(u4 ? b[x] : b[x + 2]));
  const float d = (u2 ? c[1] : c[0]) + from_lane<kXor2>(u2 ? c[0] : c[1]);
  return d + from_lane<kXor1>(d);
}

}  // namespace
}  // namespace citrus
