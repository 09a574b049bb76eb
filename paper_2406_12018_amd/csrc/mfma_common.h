// What the bf16 matrix-core kernels share: operand types, tile geometry, small helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "citrus_internal.h"
#include "lanes.h"

namespace citrus {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short i16x4;

typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr int kTileN = 64;              // keys per LDS tile of the kernels whose waves share their tiles
constexpr int kXcds = 8;
constexpr int kBufferFlags = 0x00020000;  // raw buffer resource word 3 on CDNA: 32-bit data format, no swizzle

// Geometry of K/V tiles in LDS for one head dimension (64 or 128).  Rows are unpadded; the 16-byte segment `seg` of
// tile row `row` lives at segment position seg ^ swz(row), which keeps both read patterns (key rows as an operand,
// transpose reads of value columns) free of bank conflicts.  swz is linear under XOR in the row's bits, so the
// swizzle of a sum of disjoint bit ranges is the XOR of their swizzles, and 16 rows leave it unchanged.
//   128: a row spans the 256 bytes of a 16-byte read cycle: sixteen consecutive rows take sixteen positions.
//   64:  two rows span them: eight rows of one parity take the eight positions of a row, and the four rows of a
//        transpose read (8-byte pieces of two neighbouring segments each) fall into four different 32-byte pairs.
template <int D>
struct Geo {
  static constexpr int kSegs = D / 8;                    // 16-byte segments of a row
  static constexpr int kRowBytes = 2 * D;
  static constexpr int kTileBytes = kTileN * kRowBytes;
  static constexpr int kRowsPerLoad = 1024 / kRowBytes;  // rows one wave-level LDS-direct load moves
  static constexpr int kKk = D / 16;                     // contraction steps of K.Q^T
  static constexpr int kOut = D / 32;                    // 32-row tiles of O^T
  // bf16 parts of a probability in P.V.  One (the probability rounded to bf16) at 128.  Two at 64, where the results keep
  // the accuracy of f32 probabilities: what is left of their error is the rounding of the output (relative error
  // against f64 over 512 rows x 1280 states 0.00166, of the rounded f64 result 0.00166, with one part 0.00234).
  static constexpr int kParts = D == 64 ? 2 : 1;
  static constexpr int kPitchK = D + 8;                  // padded row pitch (bf16) of query rows staged by ordinary writes
  __device__ static constexpr int swz(int row) {
    return D == 128 ? (2 * (row % 8)) ^ ((row / 8) % 2) : (2 * ((row / 2) % 4)) ^ ((row / 8) % 2) ^ (4 * (row % 2));
  }
};
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMaxSlack = 8.0f;  // probabilities stay below 2^8: exact in f32, same relative rounding in bf16

union Pack8 {
  bf16x8 v;
  uint4 u;
  uint32_t w[4];
  i16x4 h[2];
};

__device__ inline const uint16_t* unit_ptr(const View& v, int b, int l, int h) {
  return static_cast<const uint16_t*>(v.ptr) + (b * v.sb + l * v.sl + h * v.sh);
}

// a fence for the optimiser
__device__ inline void no_memory_motion() { asm volatile("" ::: "memory"); }

// Division by a number that is known at launch: n / divisor for 0 <= n < 2^31 by a multiplication.
struct FastDiv {
  int divisor;
  uint32_t mul;
  int shift;
  __device__ int quotient(int n) const {
    return static_cast<int>((__umulhi(static_cast<uint32_t>(n), mul) + static_cast<uint32_t>(n)) >> shift);
  }
};
inline FastDiv fast_div(int d) {
  FastDiv f{d, 0, 0};
  while ((int64_t{1} << f.shift) < d) ++f.shift;
  f.mul = static_cast<uint32_t>(((uint64_t{1} << 32) * ((uint64_t{1} << f.shift) - d)) / d + 1);
  return f;
}

}  // namespace
}  // namespace citrus
