// Attention of one query row on the vector units of one wave, head_dim 64.
//
// The matrix-core kernels form every product of a tile, 0 x v among them: for states a row does not see, for rows of a
// tile past the last state, and for the second bf16 part of a probability.  An infinite or NaN value then makes the
// row's outputs NaN.  Rows whose outputs are not finite (nothing else costs time) are computed again here, where a state
// that the row does not see is not touched and a probability is one f32 number.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace citrus {

struct Floats8 {
  float x[8];
};
__device__ inline Floats8 bf16x8_to_f32(const uint4& v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  Floats8 f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f.x[2 * i] = __uint_as_float(w[i] << 16);
    f.x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
  return f;
}

// Eight lanes share a state (lane % 8: their 16-byte piece of its row), so a load instruction reads eight whole rows; the
// sixteen loads of 64 states are in flight together.  q: elements 8 (lane % 8) .. + 7 of the query row; states 0 .. limit are
// seen; key_row(j) / value_row(j): their bf16 rows.  Called by whole waves.  Returns the same elements of the output in
// every group of eight lanes; lse: the row's log-sum-exp.
// A launch all of whose rows come here (an infinite value in the first state; 8 layers of 32/8 heads, 512 rows over 768 +
// 512 states) takes 3.0 ms, with one state per load instruction 10.8, on the vector kernels of before 4.9; one token 37 us
// (97).  A wave takes its 32 rows one after the other: a launch of few row tiles is slower than with a wave per row (one
// layer of 8/2 heads, 500 rows over 3000 + 500 states: 3.1 ms, 0.6).
template <typename KeyRow, typename ValueRow>
__device__ Floats8 attn_row_64(const Floats8& q, int limit, float scale, KeyRow&& key_row, ValueRow&& value_row, float& lse) {
  constexpr int kBatch = 8;  // states per lane and step
  const int lane = threadIdx.x % 64, state = lane / 8, piece = lane % 8;
  float m = -INFINITY, lsum = 0.f;
  Floats8 acc = {};
  for (int j0 = 0; j0 <= limit; j0 += 8 * kBatch) {
    uint4 key[kBatch], value[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) key[i] = reinterpret_cast<const uint4*>(key_row(min(j0 + 8 * i + state, limit)))[piece];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) value[i] = reinterpret_cast<const uint4*>(value_row(min(j0 + 8 * i + state, limit)))[piece];
    float s[kBatch], mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const Floats8 k = bf16x8_to_f32(key[i]);
      float dot = 0.f;
#pragma unroll
      for (int x = 0; x < 8; ++x) dot = fmaf(q.x[x], k.x[x], dot);
#pragma unroll
      for (int o = 4; o > 0; o >>= 1) dot += __shfl_xor(dot, o, 64);
      s[i] = j0 + 8 * i + state <= limit ? dot * scale : -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
#pragma unroll
    for (int o = 32; o >= 8; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    const float m_new = fmaxf(m, mx), corr = expf(m - m_new);
#pragma unroll
    for (int x = 0; x < 8; ++x) acc.x[x] *= corr;
    float psum = 0.f;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const bool seen = j0 + 8 * i + state <= limit;
      const float p = seen ? expf(s[i] - m_new) : 0.f;
      const Floats8 v = bf16x8_to_f32(value[i]);
      psum += p;
#pragma unroll
      for (int x = 0; x < 8; ++x) acc.x[x] = seen ? fmaf(p, v.x[x], acc.x[x]) : acc.x[x];
    }
#pragma unroll
    for (int o = 32; o >= 8; o >>= 1) psum += __shfl_xor(psum, o, 64);
    lsum = lsum * corr + psum;
    m = m_new;
  }
#pragma unroll
  for (int x = 0; x < 8; ++x) {
#pragma unroll
    for (int o = 32; o >= 8; o >>= 1) acc.x[x] += __shfl_xor(acc.x[x], o, 64);
    acc.x[x] /= lsum;
  }
  lse = m + logf(lsum);
  return acc;
}

}  // namespace citrus
