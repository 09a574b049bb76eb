// Attention of one query row on the vector units of one wave, head_dim 64: lane e holds element e.
//
// The matrix-core kernels form every product of a tile, 0 x v among them: for states a row does not see, for rows of a
// tile past the last state, and for the second bf16 part of a probability.  An infinite or NaN value then makes the
// row's outputs NaN.  Rows whose outputs are not finite (nothing else costs time) are computed again here, where a state
// that the row does not see is not touched and a probability is one f32 number.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace citrus {

__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }
__device__ inline float read_lane(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// q: this lane's element of the row; states 0 .. limit are seen; key_row(j) / value_row(j): their bf16 rows.  Called by
// whole waves.  Returns this lane's element of the output; lse: the row's log-sum-exp.
template <typename KeyRow, typename ValueRow>
__device__ float attn_row_64(float q, int limit, float scale, KeyRow&& key_row, ValueRow&& value_row, float& lse) {
  const int lane = threadIdx.x % 64;
  float m = -INFINITY, lsum = 0.f, acc = 0.f;
  for (int j0 = 0; j0 <= limit; j0 += 64) {
    const bool seen = j0 + lane <= limit;
    const uint4* const key = reinterpret_cast<const uint4*>(key_row(min(j0 + lane, limit)));
    float dot = 0.f;
    for (int x = 0; x < 8; ++x) {
      const uint4 words = key[x];
      const uint32_t w[4] = {words.x, words.y, words.z, words.w};
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        dot = fmaf(read_lane(q, 8 * x + 2 * y), __uint_as_float(w[y] << 16), dot);
        dot = fmaf(read_lane(q, 8 * x + 2 * y + 1), __uint_as_float(w[y] & 0xffff0000u), dot);
      }
    }
    const float s = seen ? dot * scale : -INFINITY;
    float mx = s;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    const float m_new = fmaxf(m, mx);
    const float p = seen ? expf(s - m_new) : 0.f;
    float psum = p;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) psum += __shfl_xor(psum, o, 64);
    const float corr = expf(m - m_new);
    lsum = lsum * corr + psum;
    acc *= corr;
    m = m_new;
    const int count = min(64, limit + 1 - j0);
    for (int x = 0; x < count; ++x) acc = fmaf(read_lane(p, x), bf16_to_f32(value_row(j0 + x)[lane]), acc);
  }
  lse = m + logf(lsum);
  return acc / lsum;
}

}  // namespace citrus
