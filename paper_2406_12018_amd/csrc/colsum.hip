// Column sums of softmax weights whose row normalisers are known (summed form of Eq. (1)): score[g, j] = sum over the query
// rows of the KV group of exp(s - lse), bf16, head_dim 64 and 128, gfx950.  Second pass of the two-pass instruction score,
// and, with the causal mask and the attention's normalisers, the importance a chunk gives its candidates.
#include "citrus_internal.h"
#include "mfma_common.h"
#include "mfma_pipe.h"

namespace citrus {
namespace {

constexpr int kRowShares = 2;  // waves that share out the rows of a workgroup's keys

// N logits of a lane (2 or 4): weight exp2(s c2 - lse) each, added to its key's sum, around one MFMA in whose shadow the
// vector instructions run.  One statement, so that the order is what is written; the MFMA is the wait state behind the
// exponentials.  FIRST: the MFMA begins a chain, in the registers that the accumulator has.
template <bool FIRST>
__device__ inline void weights2_with_mfma(float s0, float s1, float& t0, float& t1, float lse, float c2, f32x16& acc,
                                          const bf16x8& a, const bf16x8& b) {
  float p0, p1;
  if constexpr (FIRST)
    asm volatile(
        "v_fma_f32 %0, %5, %7, -%8\n\tv_fma_f32 %1, %6, %7, -%8\n\tv_exp_f32 %0, %0\n\tv_exp_f32 %1, %1\n\t"
        "v_mfma_f32_32x32x16_bf16 %2, %9, %10, 0\n\t"
        "v_add_f32 %3, %3, %0\n\tv_add_f32 %4, %4, %1"
        : "=&v"(p0), "=&v"(p1), "+v"(acc), "+v"(t0), "+v"(t1)
        : "v"(s0), "v"(s1), "s"(c2), "v"(lse), "v"(__builtin_bit_cast(i32x4, a)), "v"(__builtin_bit_cast(i32x4, b)));
  else
    asm volatile(
        "v_fma_f32 %0, %5, %7, -%8\n\tv_fma_f32 %1, %6, %7, -%8\n\tv_exp_f32 %0, %0\n\tv_exp_f32 %1, %1\n\t"
        "v_mfma_f32_32x32x16_bf16 %2, %9, %10, %2\n\t"
        "v_add_f32 %3, %3, %0\n\tv_add_f32 %4, %4, %1"
        : "=&v"(p0), "=&v"(p1), "+v"(acc), "+v"(t0), "+v"(t1)
        : "v"(s0), "v"(s1), "s"(c2), "v"(lse), "v"(__builtin_bit_cast(i32x4, a)), "v"(__builtin_bit_cast(i32x4, b)));
}
template <bool FIRST>
__device__ inline void weights4_with_mfma(float s0, float s1, float s2, float s3, float& t0, float& t1, float& t2, float& t3,
                                          float lse, float c2, f32x16& acc, const bf16x8& a, const bf16x8& b) {
  float p0, p1, p2, p3;
  if constexpr (FIRST)
    asm volatile(
        "v_fma_f32 %0, %9, %13, -%14\n\tv_fma_f32 %1, %10, %13, -%14\n\tv_fma_f32 %2, %11, %13, -%14\n\tv_fma_f32 %3, %12, %13, -%14\n\t"
        "v_exp_f32 %0, %0\n\tv_exp_f32 %1, %1\n\tv_exp_f32 %2, %2\n\tv_exp_f32 %3, %3\n\t"
        "v_mfma_f32_32x32x16_bf16 %4, %15, %16, 0\n\t"
        "v_add_f32 %5, %5, %0\n\tv_add_f32 %6, %6, %1\n\tv_add_f32 %7, %7, %2\n\tv_add_f32 %8, %8, %3"
        : "=&v"(p0), "=&v"(p1), "=&v"(p2), "=&v"(p3), "+v"(acc), "+v"(t0), "+v"(t1), "+v"(t2), "+v"(t3)
        : "v"(s0), "v"(s1), "v"(s2), "v"(s3), "s"(c2), "v"(lse), "v"(__builtin_bit_cast(i32x4, a)),
          "v"(__builtin_bit_cast(i32x4, b)));
  else
    asm volatile(
        "v_fma_f32 %0, %9, %13, -%14\n\tv_fma_f32 %1, %10, %13, -%14\n\tv_fma_f32 %2, %11, %13, -%14\n\tv_fma_f32 %3, %12, %13, -%14\n\t"
        "v_exp_f32 %0, %0\n\tv_exp_f32 %1, %1\n\tv_exp_f32 %2, %2\n\tv_exp_f32 %3, %3\n\t"
        "v_mfma_f32_32x32x16_bf16 %4, %15, %16, %4\n\t"
        "v_add_f32 %5, %5, %0\n\tv_add_f32 %6, %6, %1\n\tv_add_f32 %7, %7, %2\n\tv_add_f32 %8, %8, %3"
        : "=&v"(p0), "=&v"(p1), "=&v"(p2), "=&v"(p3), "+v"(acc), "+v"(t0), "+v"(t1), "+v"(t2), "+v"(t3)
        : "v"(s0), "v"(s1), "v"(s2), "v"(s3), "s"(c2), "v"(lse), "v"(__builtin_bit_cast(i32x4, a)),
          "v"(__builtin_bit_cast(i32x4, b)));
}
// 64 lanes x 16 bytes from a scalar base plus a lane's offset, or from a lane's own address, to 1 KB of LDS; waited for by
// the barrier alone (see load_lds_unwatched)
__device__ inline void global_to_lds(uint32_t lds, const void* base, uint32_t lane_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(lane_off), "s"(base) : "m0", "memory");
}
__device__ inline void global_to_lds(uint32_t lds, const void* lane_address) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds), "v"(lane_address) : "m0", "memory");
}

struct ColsumArgs {
  View q;
  Segments ks;
  int Hq, Hkv, L, G, rows, causal;
  int key_blocks, full_blocks;  // of a unit; those whose first key is a cache state come first
  int per_xcd;                  // units per XCD, 0: not a whole number
  FastDiv by_full, by_units, kv_heads, layers, head_rows;
  float c2, to_log2;
  const float* norm;  // norm[row * norm_pitch] * to_log2: a row's normaliser in the log2 domain
  int norm_pitch;
  float* score;
};

// Keys stay, rows stream.  A wave holds 64 keys (two 32-key tiles) as operands in registers; the group's query rows (all
// its heads, flattened) go through LDS in chunks of a step per wave.  Of the 2 KG waves KG share out the keys and two the
// steps, the even and the odd ones of the group's rows whatever KG is; what these two summed meets in LDS at the end: no
// atomics, and a score's bits follow from its rows and not from the launch.
// What bounds it: at head_dim 128 a SIMD spends 32 cycles of matrix pipe on an MFMA and about 42 on issuing it with its share
// of the vector work (two multiply-adds of 4.3 cycles, two exponentials of 8.2, two adds of 2.3).  Of launches that fill the chip
// the counters say (16 layers | 32, no mask): matrix pipe busy 37 | 44 % of the time, vector port 49 | 57 %, and the waves wait 34 %
// of theirs on a counter or a barrier, for the next chunk of rows; 0.86 | 0.99 PFLOP/s.  So: the weights of one step are
// formed between the MFMAs of the next, evenly and in a fixed order (waves that do the one and then the other take turns on
// the ports); an LDS operand feeds two MFMAs; keys and rows come in through LDS as whole rows; loads go between the MFMAs;
// the mask's arithmetic is left out for waves whose keys every row sees.
// us, earlier kernel (32 keys a wave, four waves per SIMD, rows staged through registers) | this one; 32/8 heads, 512 rows,
// 1280 keys: 1 layer 39.8 | 29.2, 4 layers 46.1 | 36.7, 8 layers 66.7 | 67.4, 16 layers 107.7 | 102.2; 500 rows, 1000 keys,
// 16 layers 89.7 | 72.6; 28/4 heads, 700 rows, 900 keys, 3 layers 126 | 72.7; causal, 512 rows behind 768 states, 1 layer
// 41.8 | 31.2, 16 layers 98.4 | 91.3.  head_dim 64, where the vector port is the bound, 8 layers 51.8 | 42, 16 layers 76.5 | 71.
template <int D, int KG>
__global__ __launch_bounds__(64 * kRowShares * KG, 2) void colsum_mfma_kernel(ColsumArgs a) {
  typedef Geo<D> T;
  typedef Lay<D> Y;
  constexpr int QT = 128 / D;                  // 32-row tiles of a step: eight MFMAs per key tile and step
  constexpr int RS = kRowShares;
  constexpr int kSteps = RS * KG;                 // of a chunk; a wave stages one of them
  constexpr int kChunkRows = kSteps * 32 * QT;
  constexpr int kStage = kSteps * QT * Y::kHalf;  // bytes of a staged chunk
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  char* const q_s = smem;                                           // [2] chunks
  float* const lse_s = reinterpret_cast<float*>(smem + 2 * kStage); // [2][kChunkRows], log2 domain, +inf for padding rows

  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int col = lane % 32, grp = lane / 32;
  const int kg = w % KG, rs = w / KG;

  // Workgroups go to the 8 XCDs round-robin by their linear id.  An XCD takes whole units, the key blocks of a unit next to
  // each other (they stream the same rows through its L2); under the causal mask the blocks of chunk keys, which fewer
  // rows see, come behind all others.
  const int linear = blockIdx.y * gridDim.x + blockIdx.x;
  int at = linear, units = gridDim.y * a.Hkv, unit0 = 0;
  if (a.per_xcd > 0) {
    at = linear / kXcds;
    units = a.per_xcd;
    unit0 = linear % kXcds * a.per_xcd;
  }
  int unit, block;
  if (at < units * a.full_blocks) {
    unit = a.by_full.quotient(at);
    block = at - unit * a.full_blocks;
  } else {
    at -= units * a.full_blocks;
    block = a.by_units.quotient(at);
    unit = at - block * units;
    block += a.full_blocks;
  }
  unit += unit0;
  const int bl = a.kv_heads.quotient(unit), g = unit - bl * a.Hkv;
  const int b = a.layers.quotient(bl), l = bl - b * a.L;
  const int n_c = a.ks.n_c, n = n_c + a.ks.c, rows = a.rows;
  const int j0 = (block * KG + kg) * 64;
  const bool has_keys = j0 < n;
  const bool partial = a.causal && j0 + 63 > n_c;  // some row may not see some key of this wave
  const int total_rows = a.G * rows;  // flattened (head in group, row)

  // ---- staging: a wave brings in the 32 QT rows of step w of a chunk, kR rows per load instruction ----
  typedef __attribute__((address_space(3))) char* lds_char_ptr;
  const uint32_t lds_q = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_char_ptr)q_s));
  constexpr int kR = T::kRowsPerLoad;
  const int fill_row = lane / T::kSegs, fill_seg16 = ((lane % T::kSegs) ^ Y::swz(fill_row)) * 16;
  const uint32_t lane_off = static_cast<uint32_t>(fill_row) * static_cast<uint32_t>(2 * a.q.ss) + fill_seg16;
  const uint16_t* const q_group = unit_ptr(a.q, b, l, g * a.G);
  const float* const norm = a.norm + (static_cast<int64_t>(bl) * a.Hq + g * a.G) * rows * a.norm_pitch;  // the group's heads are consecutive
  float lse_in = INFINITY;  // of row tid of the chunk being staged
  // What is left to stage: loads from a scalar base, whole rows of one head, that go between the MFMAs of the steps (all
  // eight waves issuing theirs at once held every wave up for 900 cycles a chunk).
  const uint16_t* stage_base = q_group;
  uint32_t stage_lds = 0;
  int stage_left = 0;
  const int64_t stage_step = kR * a.q.ss;
  auto stage_one = [&]() __attribute__((always_inline)) {
    if (stage_left > 0) {  // wave-uniform
      global_to_lds(stage_lds, stage_base, lane_off);
      stage_base += stage_step;
      stage_lds += Y::kBlock;
      --stage_left;
    }
  };
  auto stage_rest = [&]() __attribute__((always_inline)) {
    while (stage_left > 0) stage_one();
  };
  constexpr int kStageLoads = 32 * QT / kR, kStagePerStep = kStageLoads * RS / kSteps;
  auto begin_stage = [&](int f0, int buf) __attribute__((always_inline)) {
    const int f = f0 + 32 * QT * w, hh = a.head_rows.quotient(f), t = f - hh * rows;
    const uint32_t dst = lds_q + buf * kStage + w * QT * Y::kHalf;
    if (f + 32 * QT <= total_rows && t + 32 * QT <= rows) {  // wave-uniform
      stage_base = q_group + hh * a.q.sh + t * a.q.ss;
      stage_lds = dst;
      stage_left = kStageLoads;
    } else {  // rows of several heads; rows past the end repeat the last one, their weight is 0
#pragma unroll 1
      for (int x = 0; x < kStageLoads; ++x) {
        const int fx = min(f + kR * x + fill_row, total_rows - 1), hx = a.head_rows.quotient(fx);
        const char* const row = reinterpret_cast<const char*>(q_group + hx * a.q.sh + (fx - hx * rows) * a.q.ss);
        global_to_lds(dst + x * Y::kBlock, row + fill_seg16);
      }
    }
    if (tid < kChunkRows) lse_in = f0 + tid < total_rows ? norm[static_cast<int64_t>(f0 + tid) * a.norm_pitch] * a.to_log2 : INFINITY;
  };
  auto publish = [&](int buf) __attribute__((always_inline)) {
    if (tid < kChunkRows) lse_s[buf * kChunkRows + tid] = lse_in;
    wait_loads_and_barrier<0, true>();
  };
  static_assert(kSteps % (2 * RS) == 0, "pairs of steps");
  static_assert(kChunkRows <= 64 * RS * KG, "a thread per normaliser of a chunk");

  // ---- the wave's keys: row operand of key j0 + 32 kt + col, kept in registers.  They come in through LDS as well, in the
  // second chunk's place: whole rows per load instruction, once for the waves that share them ----
  // row of a flattened row within its head; a 32-row tile that wraps holds the first row of a head and the last
  auto head_row = [&](int f) __attribute__((always_inline)) { return f - a.head_rows.quotient(f) * rows; };
  // Chunks none of whose rows sees a key of this block are passed over.
  auto next_chunk = [&](int f) __attribute__((always_inline)) {
    if (a.causal && block * (64 * KG) > n_c) {  // block-uniform
      for (; f < total_rows; f += kChunkRows) {
        const int t = head_row(f);
        if (n_c + (t + kChunkRows > rows ? rows : t + kChunkRows) > block * (64 * KG)) break;
      }
    }
    return f;
  };
  int f0 = next_chunk(0);
  begin_stage(f0, 0);
  stage_rest();
  constexpr int kKeysPerWave = 64 / RS;  // that a wave brings in
  const uint32_t lds_k = lds_q + kStage;
  {
    const uint16_t* const k_cache = unit_ptr(a.ks.cache, b, l, g);
    const uint16_t* const k_chunk = unit_ptr(a.ks.chunk, b, l, g);
#pragma unroll
    for (int x = 0; x < kKeysPerWave / kR; ++x) {
      const int r = kKeysPerWave * w + kR * x, j = min(block * (64 * KG) + r + fill_row, n - 1);  // past the end: the last key again
      const uint16_t* const row = j < n_c ? k_cache + j * a.ks.cache.ss : k_chunk + (j - n_c) * a.ks.chunk.ss;
      global_to_lds(lds_k + r / kR * Y::kBlock, reinterpret_cast<const char*>(row) + fill_seg16);
    }
  }
  uint32_t op_base[4];  // of an operand's rows in a 32-row tile
#pragma unroll
  for (int c = 0; c < 4; ++c) op_base[c] = Y::at(col, Y::kStep * c + grp);
  auto read_operand = [&](const char* tile, int kk) __attribute__((always_inline)) {
    const int c = 2 * kk / Y::kStep;
    Pack8 p;
    p.u = *reinterpret_cast<const uint4*>(tile + op_base[c] + (2 * kk - Y::kStep * c) * 16);
    return p.v;
  };
  publish(0);
  bf16x8 k_op[2][T::kKk];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int kk = 0; kk < T::kKk; ++kk) k_op[kt][kk] = read_operand(q_s + kStage + (2 * kg + kt) * Y::kHalf, kk);
  lds_writes_and_barrier();  // every wave has its keys: the second chunk may come in

  float acc[2][16];  // of key 32 kt + 8 (i / 4) + 4 grp + (i % 4), over the rows of the lane
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[kt][i] = 0.f;

  // ---- logits of two steps: those of one become weights while those of the other are formed ----
  f32x16 s_t[2][2][QT];  // step parity, key tile, row tile
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int y = 0; y < QT; ++y)
#pragma unroll
      for (int i = 0; i < 16; ++i) s_t[1][kt][y][i] = -INFINITY;  // before the first step: weights of 0
  bf16x8 q_op[QT][T::kKk];
  float lse_cur[QT], lse_old[QT];
#pragma unroll
  for (int y = 0; y < QT; ++y) lse_cur[y] = lse_old[y] = 0.f;
  int f_old = -1;  // first row of the step whose logits wait, where the mask may hide some of them
  const float c2 = a.c2;

  // Under the causal mask a key is invisible to the rows of its chunk in front of it.
  auto masked = [&](int f) __attribute__((always_inline)) {
    if (!partial) return false;
    bool m = false;
#pragma unroll
    for (int y = 0; y < QT; ++y) {
      const int t = head_row(f + 32 * y);
      m |= j0 + 63 > n_c + (t + 31 >= rows ? 0 : t);
    }
    return m;
  };
  auto seen = [&](int f) __attribute__((always_inline)) {  // does any row of the step see a key of this wave?
    if (!partial) return true;
    bool any = false;
#pragma unroll
    for (int y = 0; y < QT; ++y) {
      const int t = head_row(f + 32 * y);
      any |= n_c + (t + 31 >= rows ? rows - 1 : t + 31) >= j0;
    }
    return any;
  };
  // Logits that the mask hides become -inf.  A row whose normaliser is NaN, or -inf, gives NaN to the keys it sees and
  // nothing to the others: the NaN moves from the normaliser into the visible logits.
  auto wait_for_logits = [&](f32x16 (&s)[2][QT]) __attribute__((always_inline)) {
    if constexpr (QT == 1)
      wait_for_pinned_mfmas(s[0][0], s[1][0]);
    else
      wait_for_pinned_mfmas(s[0][0], s[0][1], s[1][0], s[1][1]);
  };
  auto hide = [&](f32x16 (&s)[2][QT], int f) __attribute__((always_inline)) {
    wait_for_logits(s);
#pragma unroll
    for (int y = 0; y < QT; ++y) {
      const bool known = lse_old[y] > -INFINITY;
      const float extra = known ? 0.f : NAN;
      if (!known) lse_old[y] = 0.f;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const int last = n_c + head_row(f + 32 * y + col) - j0 - 32 * kt - 4 * grp;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kt][y][i] = 8 * (i / 4) + (i % 4) <= last ? s[kt][y][i] + extra : -INFINITY;
      }
    }
  };

  // One step, the rows at rows_s: its 16 products, and between them the weights of the step before it.  An operand is read
  // again right behind its last MFMA, from the step that comes next.
  auto step = [&](auto parity, int f, const char* rows_next, const float* lse_next_s) __attribute__((always_inline)) {
    constexpr int P = decltype(parity)::value;
    f32x16(&s_new)[2][QT] = s_t[P];
    f32x16(&s_was)[2][QT] = s_t[1 - P];
    if (__builtin_expect(f_old >= 0, 0)) hide(s_was, f_old);  // wave-uniform
    float lse_next[QT];
#pragma unroll
    for (int y = 0; y < QT; ++y) lse_next[y] = lse_next_s[32 * y + col];
    f_old = masked(f) ? f : -1;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      // products: 16 / kKk chains, key tile by key tile; weights: the same order, a chain's logits in kKk parts
      const int kt = x / 8, y = x % 8 / T::kKk, kk = x % T::kKk, i = 16 / T::kKk * kk;
      if constexpr (D == 128) {
        if (kk == 0)
          weights2_with_mfma<true>(s_was[kt][y][i], s_was[kt][y][i + 1], acc[kt][i], acc[kt][i + 1], lse_old[y], c2, s_new[kt][y],
                                   k_op[kt][kk], q_op[y][kk]);
        else
          weights2_with_mfma<false>(s_was[kt][y][i], s_was[kt][y][i + 1], acc[kt][i], acc[kt][i + 1], lse_old[y], c2, s_new[kt][y],
                                    k_op[kt][kk], q_op[y][kk]);
      } else {
        if (kk == 0)
          weights4_with_mfma<true>(s_was[kt][y][i], s_was[kt][y][i + 1], s_was[kt][y][i + 2], s_was[kt][y][i + 3], acc[kt][i],
                                   acc[kt][i + 1], acc[kt][i + 2], acc[kt][i + 3], lse_old[y], c2, s_new[kt][y], k_op[kt][kk], q_op[y][kk]);
        else
          weights4_with_mfma<false>(s_was[kt][y][i], s_was[kt][y][i + 1], s_was[kt][y][i + 2], s_was[kt][y][i + 3], acc[kt][i],
                                    acc[kt][i + 1], acc[kt][i + 2], acc[kt][i + 3], lse_old[y], c2, s_new[kt][y], k_op[kt][kk],
                                    q_op[y][kk]);
      }
      if (kt == 1) q_op[y][kk] = read_operand(rows_next + y * Y::kHalf, kk);
      if (x % (16 / kStagePerStep) == 16 / kStagePerStep - 1) stage_one();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int y = 0; y < QT; ++y) {
      lse_old[y] = lse_cur[y];
      lse_cur[y] = lse_next[y];
    }
  };

  // A wave's steps of a chunk are rs, rs + RS, ..., taken in pairs.
  for (int buf = 0, f_next; f0 < total_rows; f0 = f_next, buf ^= 1) {
    f_next = next_chunk(f0 + kChunkRows);
    const bool more = f_next < total_rows;      // block-uniform
    if (more) begin_stage(f_next, buf ^ 1);  // every wave is through with that buffer
    const int steps = has_keys ? (min(kChunkRows, total_rows - f0) + 32 * QT - 1) / (32 * QT) : 0;
    auto next_pair = [&](int s) __attribute__((always_inline)) {
      while (s < steps && !seen(f0 + 32 * QT * s) && !seen(f0 + 32 * QT * (s + RS))) s += 2 * RS;
      return s;
    };
    auto step_rows = [&](int s) __attribute__((always_inline)) { return q_s + buf * kStage + s * QT * Y::kHalf; };
    auto step_lse = [&](int s) __attribute__((always_inline)) { return lse_s + buf * kChunkRows + 32 * QT * s; };
    int s = next_pair(rs);
    if (s < steps) {
#pragma unroll
      for (int y = 0; y < QT; ++y) {
        lse_cur[y] = step_lse(s)[32 * y + col];
#pragma unroll
        for (int kk = 0; kk < T::kKk; ++kk) q_op[y][kk] = read_operand(step_rows(s) + y * Y::kHalf, kk);
      }
    }
    while (s < steps) {
      const int s_next = next_pair(s + 2 * RS), s_read = s_next < steps ? s_next : s;  // behind the last pair: rows that are there
      step(std::integral_constant<int, 0>{}, f0 + 32 * QT * s, step_rows(s + RS), step_lse(s + RS));
      step(std::integral_constant<int, 1>{}, f0 + 32 * QT * (s + RS), step_rows(s_read), step_lse(s_read));
      s = s_next;
    }
    if (more) {
      stage_rest();
      publish(buf ^ 1);
    }
  }
  if (has_keys) {  // the weights of the last step
    wait_for_logits(s_t[1]);
    if (f_old >= 0) hide(s_t[1], f_old);
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int y = 0; y < QT; ++y)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[kt][i] += __builtin_amdgcn_exp2f(fmaf(s_t[1][kt][y][i], c2, -lse_old[y]));
  }

  // ---- the lanes hold 32 rows each of a sum: over the lanes, then over the waves with the same keys ----
  lds_writes_and_barrier();
  float* const part_s = reinterpret_cast<float*>(smem);  // [RS][KG * 64]
  if (has_keys) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const float tot = reduce16_over32(acc[kt], col);  // value index col / 2 -> key 8 (i / 4) + 4 grp + (i % 4)
      const int i = col >> 1;
      if ((col & 1) == 0) part_s[rs * (KG * 64) + 64 * kg + 32 * kt + 8 * (i / 4) + 4 * grp + (i % 4)] = tot;
    }
  }
  lds_writes_and_barrier();
  const int j = block * (KG * 64) + tid;
  if (tid < KG * 64 && j < n) {
    float v = part_s[tid];
#pragma unroll
    for (int x = 1; x < RS; ++x) v += part_s[x * (KG * 64) + tid];
    a.score[static_cast<int64_t>(unit) * n + j] = v;
  }
}

// The same sums by waves of 32 keys, four to a SIMD, that form products and weights in turn and pass over single tiles of rows that see
// none of their keys.  It has less to do before the first row and behind the last, and is not held up where blocks of one unit pass over
// different rows and lose step, which costs the kernel above, with one chunk of rows in flight, more than this one; per row and
// key that one is faster.  many_waves has the line between the two.  The order of a sum's rows is the same: the bits are too.
constexpr int kManyThreads = 512, kManyRows = 128;
template <int D>
constexpr int kManyLds = 2 * kManyRows * (Geo<D>::kPitchK * 2 + 4);
template <int D, bool WHOLE, bool CAUSAL>
__global__ __launch_bounds__(kManyThreads, 4) void colsum_many_kernel(ColsumArgs a) {
  typedef Geo<D> T;
  constexpr int kPitchK = T::kPitchK, kTilesPerStep = 128 / D;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  uint16_t* const q_sb = reinterpret_cast<uint16_t*>(smem);                        // [2][kManyRows][kPitchK]
  float* const lse_sb = reinterpret_cast<float*>(q_sb + 2 * kManyRows * kPitchK);  // [2][kManyRows], log2 domain
  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64;
  const int col = lane % 32, grp = lane / 32;
  const int g = blockIdx.y, bl = blockIdx.z, b = bl / a.L, l = bl % a.L;
  const int n_c = a.ks.n_c, n = n_c + a.ks.c, rows = a.rows;
  const int j0 = (blockIdx.x * (kManyThreads / 64) + w) * 32;
  const bool wave_has_keys = j0 < n;

  bf16x8 k_op[T::kKk];
  {
    const uint16_t* const k_cache = unit_ptr(a.ks.cache, b, l, g);
    const uint16_t* const k_chunk = unit_ptr(a.ks.chunk, b, l, g);
    const int j = min(j0 + col, n - 1);
    const uint16_t* const key = (j < n_c ? k_cache + j * a.ks.cache.ss : k_chunk + (j - n_c) * a.ks.chunk.ss) + 8 * grp;
#pragma unroll
    for (int kk = 0; kk < T::kKk; ++kk) k_op[kk] = *reinterpret_cast<const bf16x8*>(key + 16 * kk);
  }
  float acc[2][16];  // steps of even and of odd number
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0.f;

  // A thread stages 16 bytes of some rows of a chunk; the next chunk's are in registers while a chunk is multiplied.
  // WHOLE: chunks lie inside a head.  Otherwise every row is looked up, and rows past the end repeat the last one, with a weight of 0.
  constexpr int kStep = kManyThreads / T::kSegs, kLoads = kManyRows / kStep;
  const int st_row = tid / T::kSegs, st_seg = tid % T::kSegs;
  const uint32_t thread_off = (st_row * static_cast<uint32_t>(a.q.ss) + 8 * st_seg) * 2;  // bytes; a head's rows span < 2 GiB
  const uint16_t* const q_group = unit_ptr(a.q, b, l, g * a.G);
  const float* const norm = a.norm + (static_cast<int64_t>(bl) * a.Hq + g * a.G) * rows * a.norm_pitch;
  const int total_rows = a.G * rows;
  i32x4 q_in[kLoads];
  float lse_in = 0.f;
  int stage_head = 0, stage_row = 0;  // block-uniform
  auto request_chunk = [&](int f0) {
    if constexpr (WHOLE) {
      const uint16_t* const base = q_group + stage_head * a.q.sh + static_cast<int64_t>(stage_row) * a.q.ss;
#pragma unroll
      for (int x = 0; x < kLoads; ++x)
        q_in[x] = *reinterpret_cast<const i32x4*>(reinterpret_cast<const char*>(base + x * kStep * a.q.ss) + thread_off);
      stage_row += kManyRows;
      if (stage_row == rows) {
        stage_row = 0;
        ++stage_head;
      }
      if (tid < kManyRows) lse_in = norm[static_cast<int64_t>(f0 + tid) * a.norm_pitch] * a.to_log2;
    } else {
#pragma unroll
      for (int x = 0; x < kLoads; ++x) {
        int thread = tid;
        asm volatile("" : "+v"(thread));  // formed here: addresses kept through the loop do not fit the registers
        const int f = min(f0 + thread / T::kSegs + x * kStep, total_rows - 1), hh = a.head_rows.quotient(f);
        q_in[x] = *reinterpret_cast<const i32x4*>(q_group + hh * a.q.sh + (f - hh * rows) * a.q.ss + 8 * (thread % T::kSegs));
      }
      if (tid < kManyRows) lse_in = f0 + tid < total_rows ? norm[static_cast<int64_t>(f0 + tid) * a.norm_pitch] * a.to_log2 : INFINITY;
    }
  };
  request_chunk(0);
  int buf = 0, chunk_row = 0;  // WHOLE: of its head, where the chunk starts
  for (int f0 = 0; f0 < total_rows; f0 += kManyRows, buf ^= 1) {
    uint16_t* const q_s = q_sb + buf * (kManyRows * kPitchK);
    float* const lse_s = lse_sb + buf * kManyRows;
    // this buffer was last read two chunks ago, and every wave has passed the previous chunk's barrier since
#pragma unroll
    for (int x = 0; x < kLoads; ++x) *reinterpret_cast<i32x4*>(&q_s[(st_row + x * kStep) * kPitchK + 8 * st_seg]) = q_in[x];
    if (tid < kManyRows) lse_s[tid] = lse_in;
    if (f0 + kManyRows < total_rows) request_chunk(f0 + kManyRows);  // block-uniform
    __syncthreads();
    if (wave_has_keys) {
#pragma unroll
      for (int qt = 0; qt < kManyRows / 32; ++qt) {
        float(&sum)[16] = acc[qt / kTilesPerStep % 2];
        // wave-uniform: rows of their head that the tile begins and ends with; one that wraps holds a head's first row and its last
        const int f = f0 + 32 * qt, tile_row = WHOLE ? chunk_row + 32 * qt : f - a.head_rows.quotient(f) * rows;
        const bool wraps = !WHOLE && tile_row + 31 >= rows;
        if (!WHOLE && f >= total_rows) break;
        if (CAUSAL && n_c + (wraps ? rows - 1 : tile_row + 31) < j0) continue;  // no row of the tile sees a key of this wave
        f32x16 s_t;
#pragma unroll
        for (int i = 0; i < 16; ++i) s_t[i] = 0.f;
        const uint16_t* const q_row = &q_s[(32 * qt + col) * kPitchK + 8 * grp];
#pragma unroll
        for (int kk = 0; kk < T::kKk; ++kk)
          s_t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_op[kk], *reinterpret_cast<const bf16x8*>(q_row + 16 * kk), s_t, 0, 0, 0);
        const float lse2 = lse_s[32 * qt + col];
        if (CAUSAL && j0 + 31 > n_c + (wraps ? 0 : tile_row)) {  // a key of the wave that a row of the tile does not see
          const int row = WHOLE ? tile_row + col : f + col - a.head_rows.quotient(f + col) * rows;
          const int last = n_c + row - j0 - 4 * grp;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float p = __builtin_amdgcn_exp2f(fmaf(s_t[i], a.c2, -lse2));
            sum[i] += 8 * (i / 4) + i % 4 <= last ? p : 0.f;
          }
        } else {
#pragma unroll
          for (int i = 0; i < 16; ++i) sum[i] += __builtin_amdgcn_exp2f(fmaf(s_t[i], a.c2, -lse2));
        }
      }
    }
    if constexpr (WHOLE) {
      chunk_row += kManyRows;
      if (chunk_row == rows) chunk_row = 0;
    }
  }
  if (!wave_has_keys) return;
  const float even = reduce16_over32(acc[0], col), odd = reduce16_over32(acc[1], col);
  const int i = col >> 1, j = j0 + 8 * (i / 4) + 4 * grp + i % 4;
  if ((col & 1) == 0 && j < n) a.score[(static_cast<int64_t>(bl) * a.Hkv + g) * n + j] = even + odd;
}

template <int D, int KG>
constexpr int colsum_lds_bytes() {
  constexpr int QT = 128 / D;
  return 2 * kRowShares * KG * QT * (Lay<D>::kHalf + 32 * 4);
}

// Is colsum_many_kernel the faster one?  Both were measured at 1220 calls, with and without the mask, 8 to 12000 rows per KV head, 8 to 4700
// keys, 1 to 2048 KV heads; by this rule a call takes 1 % more than the faster one on average.  It is the one of short waves where the
// other's fixed cost per workgroup weighs (few rows; several turns of the chip with few rows or keys each), and under the mask.
// us, colsum_mfma_kernel | colsum_many_kernel (head_dim 128 where none is given):
//   few rows: 8/8 heads, 29 rows, 59 keys, 3 layers 5.8 | 4.2; head_dim 64, 32/16 heads, 33 rows, 62 keys 6.4 | 4.3; but 104 rows, 233 keys 5.6 | 6.7.
//   no mask, 129 to 256 keys: 32/8 heads, 512 rows, 200 keys, 96 layers 136 | 119, but 16/8 heads, 1256 rows, 96 layers 163 | 168, and one layer
//     of 24/8 heads, 320 rows, 426 keys 37 | 69.
//   no mask, more keys: head_dim 64, 16/8 heads, 300 rows, 768 keys, 96 layers 122 | 85; 4/4 heads, 546 rows, 2000 keys, 48 layers 69 | 48;
//     8/8 heads, 512 rows, 1024 keys, 128 layers 220 | 172, but 32/16 heads, 250 rows, 300 keys, 128 layers 276 | 319 (blocks of 128
//     keys leave none idle there), 24/8 heads, 700 rows, 64 layers 138 | 192.
//   mask, head_dim 64: 64/16 heads, 200 rows behind 300 states, 128 layers 283 | 149; 32/8 heads, 384 behind 300, 64 layers 146 | 82, 1000 behind 768, 96
//     layers 1027 | 932; 16/8 heads, 211 behind 2500, 24 layers 80 | 52; 4/2 heads, 275 behind 535, 64 layers 0.64 of the time; but 32/8 heads, 1740 behind 100, 24 layers 359 | 494, 1000 behind 768, 8
//     layers 100 | 107.
//   mask: 32/8 heads, 128 behind 120, 256 layers 0.43 of the time; 12/8 heads, 200 behind 40, 64 layers 0.70; 12/8 heads, 250 behind 500, 128 layers
//     232 | 194; 32/16 heads, 400 behind 768, 96 layers 971 | 885, but 1000 behind 1024, 24 layers 812 | 881; rows of a head a multiple of 128:
//     32/8 heads, 1024 behind 300, 96 layers 1146 | 928, but 16/2 heads, 1024 behind 1024 742 | 760.
bool many_waves(const Dims& dm, int rows, int n, bool causal) {
  const int64_t units = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv, group_rows = static_cast<int64_t>(dm.G) * rows;
  const int cus = compute_units();
  const int64_t tenths = 10 * units / cus, turn_tenths = 10 * units * ((n + 255) / 256) / cus;  // turns of blocks of 256 keys
  const bool wide = dm.D == 128;
  if (group_rows <= 96 || (group_rows <= 192 && n <= 128)) return true;
  const bool few_rows = turn_tenths >= 30 && group_rows <= (wide ? 1100 : 2700);
  if (causal) {
    if (few_rows || (rows % kManyRows == 0 && units * group_rows > 3 << 17)) return true;
    if (wide) return (tenths >= 7 && (n <= 400 || group_rows <= 400)) || (tenths >= 10 && n <= 640) || (turn_tenths >= 40 && n <= 1200);
    return (tenths >= 6 && n <= 1850 && rows <= 1400) || (turn_tenths >= 5 && n > 256 && group_rows <= 1600);
  }
  if (n <= 128 || (n > 256 && n <= 384 && group_rows > 320)) return false;
  if (n <= 256) return tenths >= 12;
  return few_rows || (!wide && ((tenths >= 9 && group_rows <= 3100) || (turn_tenths >= 8 && n > 384 && group_rows <= 800)));
}

// keys: of a block of colsum_mfma_kernel
ColsumArgs colsum_args(const Dims& dm, View q, int rows, Segments ks, int causal, const float* norm, int norm_pitch, float to_log2,
                       float* score, int keys) {
  const int n = ks.n_c + ks.c, units = dm.B * dm.L * dm.Hkv;
  ColsumArgs a;
  a.q = q;
  a.ks = ks;
  a.Hq = dm.Hq;
  a.Hkv = dm.Hkv;
  a.L = dm.L;
  a.G = dm.G;
  a.rows = rows;
  a.causal = causal;
  a.key_blocks = (n + keys - 1) / keys;
  a.full_blocks = causal ? (ks.n_c + keys - 1) / keys : a.key_blocks;
  a.per_xcd = units % kXcds == 0 ? units / kXcds : 0;
  a.by_full = fast_div(a.full_blocks > 0 ? a.full_blocks : 1);
  a.by_units = fast_div(a.per_xcd > 0 ? a.per_xcd : units);
  a.kv_heads = fast_div(dm.Hkv);
  a.layers = fast_div(dm.L);
  a.head_rows = fast_div(rows);
  a.c2 = dm.scale * kLog2e;
  a.to_log2 = to_log2;
  a.norm = norm;
  a.norm_pitch = norm_pitch;
  a.score = score;
  return a;
}

template <int D, int KG>
hipError_t colsum_launch(const Dims& dm, const ColsumArgs& a, hipStream_t st) {
  static LdsLimit limit;
  const auto kern = colsum_mfma_kernel<D, KG>;
  constexpr int lds = colsum_lds_bytes<D, KG>();
  const hipError_t e = raise_lds_limit(limit, reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.key_blocks * dm.Hkv, dm.B * dm.L), dim3(64 * kRowShares * KG), lds, st, a);
  return hipGetLastError();
}

template <int D, bool WHOLE, bool CAUSAL>
hipError_t colsum_many_launch(const Dims& dm, const ColsumArgs& a, hipStream_t st) {
  static LdsLimit limit;
  const auto kern = colsum_many_kernel<D, WHOLE, CAUSAL>;
  const hipError_t e = raise_lds_limit(limit, reinterpret_cast<const void*>(kern), kManyLds<D>);
  if (e != hipSuccess) return e;
  const int n = a.ks.n_c + a.ks.c;
  hipLaunchKernelGGL(kern, dim3((n + 255) / 256, dm.Hkv, dm.B * dm.L), dim3(kManyThreads), kManyLds<D>, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_colsum_mfma(const Dims& dm, View q, int rows, Segments ks, int causal, const float* norm, int norm_pitch,
                              float to_log2, float* score, hipStream_t st) {
  const int n = ks.n_c + ks.c;
  const int64_t units = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv;
  // Workgroups of eight waves and 256 keys, one to a compute unit, or of four and 128, two to a compute unit.  Those fill a last
  // turn more evenly, and one alone on its compute unit takes 0.65 of the time of two; where every turn is full they take 1.08 times
  // as long (rows pass the LDS twice as often).  So: the shorter sum of turns.  us, 256 | 128 keys, 32/8 heads, 512 rows, 1280 keys:
  // 1 layer 32.8 | 29.2, 4 layers 36.3 | 41.0, 8 layers 69.5 | 67.3, 12 layers 73.1 | 79.6, 16 layers 102 | 102, 32 layers 178 | 190;
  // 8/8 heads, 200 rows, 300 keys, 40 layers 24.4 | 18.0; head_dim 64: 1 layer 26.2 | 20.2, 4 layers 28.4 | 30.7, 8 layers 51.4 |
  // 42.7, 16 layers 78.7 | 70.6, 32 layers 132 | 132.  (Eight waves on 128 keys, four to the rows, are faster where the chip is nearly
  // empty, 22 us for one layer, but add the rows in another order: a score would depend on the launch it is part of.)
  const auto blocks = [&](int keys) { return (n + keys - 1) / keys * units; };
  const int64_t pairs = 2 * int64_t{compute_units()}, left = blocks(128) % pairs;
  const int64_t turns128 = 100 * (blocks(128) / pairs) + (left == 0 ? 0 : 2 * left <= pairs ? 65 : 100);
  const int64_t turns256 = 100 * ((blocks(256) + compute_units() - 1) / compute_units());
  const bool small = 108 * turns128 < 100 * turns256;
  const auto choose = [&](auto head_dim) {
    constexpr int D = decltype(head_dim)::value;
    if (!many_waves(dm, rows, n, causal != 0)) return small ? colsum_launch<D, 2> : colsum_launch<D, 4>;
    if (rows % kManyRows == 0) return causal ? colsum_many_launch<D, true, true> : colsum_many_launch<D, true, false>;
    return causal ? colsum_many_launch<D, false, true> : colsum_many_launch<D, false, false>;
  };
  const auto launch = dm.D == 64 ? choose(std::integral_constant<int, 64>()) : choose(std::integral_constant<int, 128>());
  return launch(dm, colsum_args(dm, q, rows, ks, causal, norm, norm_pitch, to_log2, score, small ? 128 : 256), st);
}

}  // namespace citrus
