// Software pipelines of MFMAs and vector instructions inside one wave, and the LDS tiles they read: what the kernels with
// a hand-fixed issue order share.
#pragma once

#pragma clang diagnostic ignored "-Winline-asm"
#include <type_traits>

#include "mfma_common.h"

namespace citrus {
namespace {

// Instructions whose issue ORDER matters (a software pipeline that overlaps the matrix pipe with
// the exponentials inside one wave) are written as volatile asm statements: the compiler keeps
// volatile statements in source order and allocates their registers, but does not see inside
// them, so the software-managed hazards are handled here: v_exp_f32 is followed by the one wait
// state a non-transcendental consumer needs, and no vector instruction may read an MFMA result
// sooner than the MFMA takes to complete (callers keep a whole MFMA group in between).
__device__ inline f32x16 mfma_pinned_first(const bf16x8& a, const bf16x8& b) {  // accumulator starts at zero
  f32x16 d;
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0"
               : "=&v"(d)
               : "v"(__builtin_bit_cast(i32x4, a)), "v"(__builtin_bit_cast(i32x4, b)));
  return d;
}
// Enough wait states for every MFMA issued through the pinned helpers above to have written its result.  What is read behind the
// wait passes through it: other arithmetic is not bound to volatile statements, and was scheduled ahead of them.
template <typename... Results>
__device__ inline void wait_for_pinned_mfmas(Results&... results) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  auto pass = [](f32x16& r) { asm volatile("" : "+v"(r)); };
  (pass(results), ...);
}

// One LDS-direct load (64 lanes x 16 bytes of global memory to 1 KB of consecutive LDS) as asm: the compiler waits
// for every such load it can see (vmcnt(0)) in front of the next LDS read that might alias it, i.e. a tile requested
// between the MFMAs of one half step would be waited for at the start of the next, long before the barrier that
// publishes it.  Loads issued here are waited for by the barrier helpers alone.  lds + LDS_OFF: byte address.
template <int LDS_OFF>
__device__ inline void load_lds_unwatched(const i32x4& rsrc, uint32_t lds, int lane_off, int scalar_off) {
  asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds), "v"(lane_off), "s"(rsrc), "s"(scalar_off), "n"(LDS_OFF)
               : "m0", "scc");
}
// Buffer resource of `bytes` bytes at p as the four words the asm above takes.
__device__ inline i32x4 buffer_words(const void* p, int bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  i32x4 words = {static_cast<int>(a), static_cast<int>(a >> 32) & 0xffff, bytes, kBufferFlags};
  asm volatile("" : "+s"(words));  // one value: known to be constant, the last word was moved in place in front of each use
  return words;
}


// All but the newest LEFT loads of this wave have landed, and then every wave's have (PUBLISH: its LDS accesses are
// through as well).
template <int LEFT, bool PUBLISH>
__device__ inline void wait_loads_and_barrier() {
  if constexpr (PUBLISH)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(LEFT) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"(LEFT) : "memory");
}
__device__ inline void lds_writes_and_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// K and V tiles of the attention kernel in LDS.  A 1 KB load instruction fills one block of kR whole rows (a lane group
// reads one row of global memory: lanes of different rows next to each other would cost the address path a multiple);
// inside a row, segment seg (16 bytes) is at position seg ^ (kStep x (row / kRowStep % 4)), and blocks are 16 bytes
// further apart than they are long.  The XOR touches two bits of the segment only, so the operand reads of a lane need
// four (K) and two (V) base registers, and every address in the key loop is one of them plus a constant: no instruction
// of the loop forms an address.  Sixteen consecutive rows of one segment (a cycle of a key operand) fall into different
// banks, and so do the four rows of two segments of a 16-lane group of a transpose read; but two such groups go through
// the LDS at a time, and at head_dim 128 rows r and r ^ 2 of the two meet in the same banks: two extra LDS cycles per
// transpose read (SQ_LDS_BANK_CONFLICT, 31 % of the cycles the LDS works, which is 41 % of the launch's).
template <int D>
struct Lay {
  static constexpr int kR = Geo<D>::kRowsPerLoad;
  static constexpr int kStep = D == 128 ? 4 : 2, kRowStep = D == 128 ? 1 : 2;
  static constexpr int kBlock = 1024 + 16;
  static constexpr int kHalf = 32 / kR * kBlock;  // 32 rows
  static constexpr int kTile = 2 * kHalf;
  __device__ static constexpr int swz(int row) { return kStep * (row / kRowStep % 4); }
  __device__ static constexpr int at(int row, int seg) {
    return row / kR * kBlock + row % kR * Geo<D>::kRowBytes + (seg ^ swz(row)) * 16;
  }
};

}  // namespace
}  // namespace citrus
