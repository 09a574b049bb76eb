// bf16 MFMA kernels for head_dim 64 and 128 on gfx950 (CDNA4): templates over the head dimension.
// (head_dim 64 ran on one-wavefront-per-row vector kernels before, whose serial chain of key loads and f32
// multiply-adds reached 7 TFLOP/s: 8 layers of 32/8 heads, a document of 4096 tokens in chunks of 512, budget 768,
// took 37.6 ms; on these kernels 0.93 ms, 0.81 with probabilities rounded to bf16.)
//
//  attn_pipe_kernel    flash-style chunk attention (Section 4.1 step 1; softmax
//                      with the 1/sqrt(d_k) scaling of Eq. (1)): online softmax
//                      over 64-key tiles staged in LDS, S^T = K.Q^T and
//                      O^T = V^T.P^T on v_mfma_f32_32x32x16_bf16.
//  lse_mfma_kernel     the rows' log-sum-exp alone (first pass of the two-pass
//                      importance scores; the second is colsum.hip).
//
// Layout facts used throughout (wave64, v_mfma_f32_32x32x16_bf16):
//   A operand: lane l holds row (l % 32), contraction slots 8*(l / 32) .. +7
//   B operand: lane l holds column (l % 32), the same contraction slots
//   C/D:       lane l, register i holds column (l % 32),
//              row 8*(i / 4) + 4*(l / 32) + (i % 4)
// Computing S^T (keys x queries) puts one query per lane, so softmax row
// reductions are in-lane plus one exchange with lane l ^ 32, and the S^T
// accumulators are directly the B operand (P^T) of the second product.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "attn_row.h"
#include "bf16_math.h"
#include "citrus_internal.h"
#include "evict_body.h"
#include "mfma_common.h"
#include "mfma_pipe.h"
#include "rope_math.h"
#include "strip_score.h"


namespace citrus {
namespace {

constexpr int kWaves = 4;               // one wave per SIMD and block; two or more blocks share a CU
constexpr int kThreads = kWaves * 64;
constexpr int kRowsPerWave = 32;        // one 32-query column tile per wave

// LDS transpose read (ds_read_b64_tr_b16).  Within each group of 16 lanes, lane s passes the
// address of 4 consecutive bf16 and lane i receives element (i % 4) of lanes i/4, 4 + i/4,
// 8 + i/4, 12 + i/4.  With lane s pointing at &V[key(s / 4)][d0 + 4 (s % 4)], lane i gets
// V[key(0..3)][d0 + i]: four keys of one head_dim column, i.e. half of an MFMA A operand of V^T.
__device__ inline i16x4 lds_read_tr16(const char* p) {
  typedef i16x4 __attribute__((address_space(3))) * lds_ptr;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
}

__device__ inline float exp2_pinned(float x) {
  float y;
  asm volatile("v_exp_f32 %0, %1\n\ts_nop 0" : "=v"(y) : "v"(x));
  return y;
}

__device__ inline float max3_pinned(float a, float b, float c) {
  float y;
  asm volatile("v_max3_f32 %0, %1, %2, %3" : "=v"(y) : "v"(a), "v"(b), "v"(c));
  return y;
}
// v_exp_f32 followed by an MFMA that does not read its result: the MFMA is the wait state.
__device__ inline float exp2_then_mfma(float x, f32x16& acc, const bf16x8& a, const bf16x8& b) {
  float y;
  asm volatile("v_exp_f32 %0, %2\n\tv_mfma_f32_32x32x16_bf16 %1, %3, %4, %1"
               : "=&v"(y), "+v"(acc)
               : "v"(x), "v"(__builtin_bit_cast(i32x4, a)), "v"(__builtin_bit_cast(i32x4, b)));
  return y;
}

// two exponentials in front of one MFMA (head_dim 64: half the MFMAs per logit)
__device__ inline void exp2x2_then_mfma(float x0, float x1, float& y0, float& y1, f32x16& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_exp_f32 %0, %3\n\tv_exp_f32 %1, %4\n\tv_mfma_f32_32x32x16_bf16 %2, %5, %6, %2"
               : "=&v"(y0), "=&v"(y1), "+v"(acc)
               : "v"(x0), "v"(x1), "v"(__builtin_bit_cast(i32x4, a)), "v"(__builtin_bit_cast(i32x4, b)));
}

// Small fences for the optimiser, as functions so that kernel templates hold no asm of their own.
// -inf where n < 0, else x: three vector instructions.  (Sixteen comparisons whose results wait in scalar registers made
// the masked half step 40 instructions longer and spilled other scalars around it.)
__device__ inline float minus_inf_if_negative(int n, float x) {
  const int all_ones = n >> 31;
  asm("v_bfi_b32 %0, %1, %2, %0" : "+v"(x) : "v"(all_ones), "s"(0xff800000u));
  return x;
}
// the same number, of which the compiler knows nothing: what is formed from it is formed here, not ahead of a loop and
// kept in a register through it
__device__ inline uint32_t formed_here(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ inline void keep_values_here(uint32_t (&p)[8], float& l) {
  asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]), "+v"(p[4]), "+v"(p[5]), "+v"(p[6]), "+v"(p[7]), "+v"(l));
}
// Barrier that publishes tiles streamed into LDS by buffer_load ... lds.  Those writes are tracked
// by the issuing wave's vector-memory counter only, and the fence inside __syncthreads() covers
// ordinary LDS traffic: every wave has to drain its own loads before it arrives.
__device__ inline void barrier_after_lds_fill() {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), nothing else
  __syncthreads();
}

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
// lanes 0..31: first = own lo_half, second = lo_half of lane l + 32; lanes 32..63: first = hi_half of lane l - 32,
// second = own hi_half
__device__ inline void swap_halves(uint32_t lo_half, uint32_t hi_half, uint32_t& first, uint32_t& second) {
  const auto r = __builtin_amdgcn_permlane32_swap(lo_half, hi_half, false, false);
  first = r[0];
  second = r[1];
}

// How the waves of a block split (head, 32-row tile) tasks inside one KV group.
struct TaskShape {
  int heads_per_block;  // 4, 2 or 1 query heads of the group
  int tiles_per_block;  // kWaves / heads_per_block row tiles of 32
};
__host__ __device__ inline TaskShape task_shape(int G, int waves = kWaves) {
  const int hpb = (G % 4 == 0 && waves >= 4) ? 4 : ((G % 2 == 0 && waves >= 2) ? 2 : 1);
  return TaskShape{hpb, waves / hpb};
}

// Row normalisers only (no values, no output, no mask): one partial (running maximum, sum) pair per key range and
// row; with a single range the normaliser itself, as merge_partials_kernel leaves it.  First pass of the two-pass
// importance scores.
template <int D>
__global__ __launch_bounds__(kThreads, 2) void lse_mfma_kernel(Dims dm, View q, int rows, Segments ks, int key_splits,
                                                              float2* part) {
  typedef Geo<D> T;
  constexpr int kRowBytes = T::kRowBytes, kTileBytes = T::kTileBytes;
  __shared__ __attribute__((aligned(1024))) char k_s[2 * kTileBytes];  // double-buffered tiles

  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64;
  const int col = lane % 32, grp = lane / 32;
  const TaskShape ts = task_shape(dm.G);
  const int head_groups = dm.G / ts.heads_per_block;
  const int rows_per_block = ts.tiles_per_block * kRowsPerWave;
  const int row_blocks = (rows + rows_per_block - 1) / rows_per_block;
  // Workgroups are handed to the 8 XCDs round-robin by their linear id.  Remap so that the
  // workgroups of one (document, layer, KV head), which read the same K/V, land on ONE XCD and
  // share its L2.
  int logical = blockIdx.x;
  const int total = gridDim.x;
  if (total % kXcds == 0) logical = (blockIdx.x % kXcds) * (total / kXcds) + blockIdx.x / kXcds;
  // Each workgroup covers one contiguous range of key tiles and writes a partial (running maximum, sum) pair per row;
  // the consumer merges them.
  const int sp = logical % key_splits;
  logical /= key_splits;
  const int rb = row_blocks - 1 - logical % row_blocks;
  const int hg = (logical / row_blocks) % head_groups;
  const int g = (logical / (row_blocks * head_groups)) % dm.Hkv;
  const int bl = logical / (row_blocks * head_groups * dm.Hkv);
  const int b = bl / dm.L, l = bl % dm.L;
  const int h = g * dm.G + hg * ts.heads_per_block + (w % ts.heads_per_block);
  const int n_c = ks.n_c;
  const int n = n_c + ks.c;

  // ---- global -> LDS staging of one 64-key tile, without a stop in registers ----
  // buffer_load ... lds: a wave-level instruction moves 64 x 16 B from per-lane global addresses
  // to 1 KB of consecutive LDS, i.e. four (head_dim 64: eight) unpadded rows.  The swizzle of a row's
  // segments (Geo) is realised by the loading lane, which fetches global segment (its LDS position) ^ swz(row).
  // Wave w fills rows 16 w .. + 15.  Rows that fall outside the candidates re-read the last row
  // (finite values; their logits are masked).
  const int k_ss_cache = static_cast<int>(ks.cache.ss), k_ss_chunk = static_cast<int>(ks.chunk.ss);
  auto seg_bytes = [](int rows_, int ss_) { return rows_ > 0 ? ((rows_ - 1) * ss_ + D) * 2 : 0; };
  const __amdgpu_buffer_rsrc_t k_rs_cache = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(unit_ptr(ks.cache, b, l, g)), 0, seg_bytes(n_c, k_ss_cache), kBufferFlags);
  const __amdgpu_buffer_rsrc_t k_rs_chunk = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(unit_ptr(ks.chunk, b, l, g)), 0, seg_bytes(ks.c, k_ss_chunk), kBufferFlags);
  const int wu = __builtin_amdgcn_readfirstlane(w);
  constexpr int kFillRows = kTileN / kWaves, kR = T::kRowsPerLoad;
  const int fill_row = kFillRows * wu + lane / T::kSegs;                         // tile row this lane fills with load 0
  const int fill_seg16 = ((lane % T::kSegs) ^ T::swz(lane / T::kSegs)) * 16;  // byte offset of its segment, before ^ c_i
  typedef __attribute__((address_space(3))) void* lds_void_ptr;
  auto fill4 = [&](char* lds_tile, __amdgpu_buffer_rsrc_t rs_cache, __amdgpu_buffer_rsrc_t rs_chunk, int ss_cache,
                   int ss_chunk, int j0) {
    const bool simple = (j0 + kTileN <= n_c) || (j0 >= n_c && j0 + kTileN <= n);  // block-uniform
#pragma unroll
    for (int i = 0; i < kFillRows / kR; ++i) {
      const int ci16 = T::swz(kR * i) * 16;
      lds_void_ptr dst = (lds_void_ptr)(lds_tile + (kFillRows * wu + kR * i) * kRowBytes);
      if (simple) {
        const bool in_cache = j0 < n_c;
        const int ss = in_cache ? ss_cache : ss_chunk;
        const int r0 = in_cache ? j0 : j0 - n_c;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(in_cache ? rs_cache : rs_chunk, dst, 16,
                                                 fill_row * ss * 2 + (fill_seg16 ^ ci16), (r0 + kR * i) * ss * 2, 0, 0);
      } else {  // the tile straddles the cache / chunk boundary or the end of the candidates
        const int j = min(j0 + fill_row + kR * i, n - 1);
        if (j < n_c)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_cache, dst, 16, j * ss_cache * 2 + (fill_seg16 ^ ci16), 0, 0, 0);
        else
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_chunk, dst, 16, (j - n_c) * ss_chunk * 2 + (fill_seg16 ^ ci16),
                                                   0, 0, 0);
      }
    }
  };
  auto fetch_tile = [&](int j0_, int buf_) {
    fill4(k_s + buf_ * kTileBytes, k_rs_cache, k_rs_chunk, k_ss_cache, k_ss_chunk, j0_);
  };

  // per-lane LDS read offsets (bytes inside a tile buffer), swizzle included
  // A operand of S^T: key row `col`, head_dim segment 2 kk + grp
  const int f_col = T::swz(col);
  int k_off[T::kKk];
#pragma unroll
  for (int kk = 0; kk < T::kKk; ++kk) k_off[kk] = col * kRowBytes + (((2 * kk + grp) ^ f_col) * 16);
  const int row0 = (rb * ts.tiles_per_block + w / ts.heads_per_block) * kRowsPerWave;

  const int all_tiles = (n - 1) / kTileN + 1;
  const int tiles_per_split = (all_tiles + key_splits - 1) / key_splits;
  const int t_begin = sp * tiles_per_split;
  const int t_end = min(all_tiles, t_begin + tiles_per_split);
  const bool wave_active = row0 < rows;

  // ---- Q^T operand, kept in registers: q_op[kk] = Q[row0 + col][16 kk + 8 grp ..+7] ----
  bf16x8 q_op[T::kKk];
  const int t_lane = max(min(row0 + col, rows - 1), 0);
  {
    const uint16_t* qp = unit_ptr(q, b, l, h) + static_cast<int64_t>(t_lane) * q.ss + 8 * grp;
#pragma unroll
    for (int kk = 0; kk < T::kKk; ++kk) {
      Pack8 p;
      p.u = *reinterpret_cast<const uint4*>(qp + 16 * kk);
      q_op[kk] = p.v;
    }
  }

  // ---- running softmax state: one query per lane ----
  const float c2 = dm.scale * kLog2e;  // logits are kept in the log2 domain
  float m_run = -INFINITY, l_run = 0.f;

  if (t_begin < t_end) {  // block-uniform
  fetch_tile(t_begin * kTileN, 0);
  barrier_after_lds_fill();  // also: the Q operand loads have landed

  for (int jt = t_begin; jt < t_end; ++jt) {
    const int j0 = jt * kTileN;
    const int buf = (jt - t_begin) & 1;
    const char* k_t = k_s + buf * kTileBytes;
    // The other buffer was last read one iteration ago and every wave has passed the barrier that
    // ended that iteration: the next tile can stream into it while this one is computed.
    if (jt + 1 < t_end) fetch_tile(j0 + kTileN, buf ^ 1);

    if (wave_active) {
      // S^T = K . Q^T for 64 keys x 32 queries
      f32x16 s_acc[2];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) s_acc[mt][i] = 0.f;
#pragma unroll
      for (int kh = 0; kh < T::kKk / 4; ++kh) {  // the two 32-key halves are independent MFMA chains: interleave them
        Pack8 a[2][4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int mt = 0; mt < 2; ++mt)
            a[mt][kk].u = *reinterpret_cast<const uint4*>(k_t + 32 * mt * kRowBytes + k_off[4 * kh + kk]);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int mt = 0; mt < 2; ++mt)
            s_acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mt][kk].v, q_op[4 * kh + kk], s_acc[mt], 0, 0, 0);
      }

      if (j0 + kTileN > n) {  // wave-uniform: the last tile
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int j = j0 + 32 * mt + 8 * (i / 4) + 4 * grp + (i % 4);
            if (j >= n) s_acc[mt][i] = -INFINITY;
          }
      }
      // Running maximum, kept lazily: softmax is invariant to the subtracted value, so m_run only has
      // to stay within kMaxSlack (log2 units) of the true row maximum to keep exp2 in range.  The fast
      // path looks at this lane's own 32 logits only; the exchange with lane l ^ 32, the update of
      // m_run and the rescale of the running sum happen only when some row needs them.
      float mx = s_acc[0][0];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s_acc[mt][i]);
      if (__any(mx * c2 > m_run + kMaxSlack)) {  // wave-uniform and rare after the first tiles
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx * c2);
        // 0 on a row's first visible tile (m_run = -inf); 1 for a row that has seen nothing yet
        const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
        m_run = m_new;
      }
      float psum = 0.f;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) psum += __builtin_amdgcn_exp2f(fmaf(s_acc[mt][i], c2, -m_run));
      l_run += psum;
    }

    barrier_after_lds_fill();  // publishes the tile that streamed in; everyone is done with this one
  }
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const int t = row0 + col;
  if (wave_active && t < rows && grp == 0) {  // log2 domain; an empty range leaves (-inf, 0)
    const int64_t row_id = (static_cast<int64_t>(bl) * dm.Hq + h) * rows + t;
    part[static_cast<int64_t>(sp) * dm.B * dm.L * dm.Hq * rows + row_id] =
        key_splits == 1 ? make_float2(m_run + log2f(l_tot), 1.f) : make_float2(m_run, l_tot);
  }
}

// A tensor as the attention kernel addresses it: everything in bytes.
struct UnitView {
  const char* ptr;
  int64_t sb, sl, sh;
  int ss;
  uint32_t tile_step;  // of kTileN rows; kOutside if that is 2 GiB or more
};
// Byte offset outside every unit: the range check of a buffer resource drops a store to it and reads zeros from it.  Rows
// behind the last one are sent there; their own offset, row x stride modulo 2^32, may lie inside the unit again.
constexpr uint32_t kOutside = 0x80000000u;
// rows: sequence rows of a unit.  They span less than 2 GiB (checked at the entry points), so from two rows on the stride
// is an int; the stride of a single row has no such bound and means nothing.
inline UnitView unit_view(const View& v, int rows, int head_dim) {
  const int ss = rows > 1 ? static_cast<int>(2 * v.ss) : 2 * head_dim;
  return UnitView{static_cast<const char*>(v.ptr), 2 * v.sb, 2 * v.sl, 2 * v.sh, ss,
                  ss < static_cast<int>(kOutside / kTileN) ? static_cast<uint32_t>(kTileN * ss) : kOutside};
}
// What a workgroup of the attention kernel works on, prepared on the host: a wave issues one instruction in eight
// cycles, and with divisions by runtime numbers and per-element strides the set-up took 830 of them.
struct AttnArgs {
  UnitView q, out, k_cache, k_chunk, v_cache, v_chunk;
  int n_c, c, q_heads;  // c: chunk states and query rows
  int paired;      // a workgroup takes a row block and its mirror image
  int log_heads;   // 2^log_heads query heads of a group per workgroup
  int row_blocks;  // of a head
  int per_xcd;     // workgroups per XCD, 0: not a whole number
  FastDiv slots, head_groups, kv_heads, layers;  // workgroup -> (row block slot, head group, KV head, layer)
  float scale, c2, inv_c2;  // softmax scale, and in the log2 domain
  float *lse, *lse_cache;
  int q_rope_pos0;
  float rope_log2_base;
  FastDiv group;  // MIXED: query heads of a group
  int tasks;      // MIXED: (32-row tile, head) pairs of a unit
};

// The same attention, with output, as a software pipeline over half tiles of 32 keys: in step h the
// MFMAs of S^T(h + 1) = K.Q^T and of O^T += V^T.P^T(h - 1) are issued between the exponentials of
// half tile h, so that inside ONE wave the matrix pipe, the vector pipe and the LDS reads run at
// the same time instead of taking turns (the order is fixed with volatile asm statements, see above).
// K tiles are fetched one 64-key tile further ahead than V tiles; one barrier per 64 keys.
//
// What bounds it.  A wave issues at most one instruction, of whatever kind, per 8 cycles (measured: 64 independent
// v_fma, v_max or s_mov of one wave take 505 to 540 cycles, of two waves of a SIMD the same), next to the 32 that an MFMA
// holds the matrix pipe.  A 64-key tile is therefore kept at 245 instructions per wave, 32 of them MFMAs: LDS addresses are
// register + constant (Lay), a tile lies in one segment and is always fetched (out-of-range rows read as zeros), masks and
// segment changes sit behind branches that are not taken, the vote on the row maxima is taken a step early, and one wait
// covers all operands of a product.  Outside the loop it is the same count: set-up from host-made numbers (AttnArgs),
// output rows through buffer stores.  The two waves of a SIMD meet at a barrier every 64 keys; one of the two (waves 4..7)
// passes it in front of its vector-only tail, the other behind it, so that their MFMA phases alternate.
// Counters over a document of 32 layers, 32/8 heads, 512 rows over up to 768 + 512 states: the matrix pipe is busy 51 % of
// the cycles (44 % before), the vector port 45 %, waves wait for an issue slot 43 % and at a counter or barrier 23 % of
// their time; 527 k cycles in 271 us are 1.94 GHz, the clock a loop of MFMAs alone runs at: power takes the other fifth.
// Launches inside a loop with other kernels: 330 -> 305 us (steady state, 32 layers); empty cache 141 -> 128 us; back to
// back 16 layers of 32/32 heads, 1024 rows over 1024 + 1024 states 493 -> 451 us; 64/8 heads, 2048 rows over 4096 + 2048
// states 1286 -> 1227 us.  head_dim 64, two bf16 parts per probability: 8 layers of 32/8 heads back to back 59 us.
// block: the workgroup's number among a's.  ring: two K tiles, then two V tiles (double buffers).  q_stage: WAVES query row
// tiles, laid out like half a key tile.
template <int D>
constexpr int attn_ring_bytes() { return 4 * Lay<D>::kTile; }
template <int D, int WAVES>
constexpr int attn_stage_bytes() { return WAVES * Lay<D>::kHalf; }
// MIXED: a block is the next WAVES pairs of a 32-row tile and a head, the heads of a tile next to each other, whichever they are.
// Otherwise its waves are 4, 2 or 1 heads, whichever divides the group, and row tiles of these: a group of 7 heads then
// takes 256 rows of a head at a time, of which a chunk of 300 rows has 300 in 512.  MIXED holds more scalars through the key loop
// (readlanes in it, 3 to 6 % where nothing is wasted), so it is taken where it makes fewer blocks: us, 8 layers of 28/4 heads, 300 rows
// over 700 states 61.9 | 52.9, 16 layers, 100 rows over 200 states 29.5 | 18.4, 8 layers of 24/8 heads, 333 rows over 500 states
// 50.5 | 48.8.
template <int D, int WAVES, bool ROTATE_Q, bool SAVE_REGISTERS = ROTATE_Q, bool MIXED = false>
__device__ __forceinline__ void attn_pipe_body(const AttnArgs& a, const int block, char* const ring, char* const q_stage) {
  typedef Geo<D> T;
  typedef Lay<D> Y;
  constexpr int kRowBytes = T::kRowBytes;
  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64;
  const int col = lane % 32, grp = lane / 32;
  // The instance that rotates its queries is at the limit of its registers: it forms what the rare branches of the key loop
  // need of the lane's number there (227 registers; 256 and some in scratch otherwise: 16 layers, a document of 4000
  // tokens, 3.28 against 3.12 ms).  The other instances keep these numbers: 243 registers, and documents 0.3 to 0.6 %
  // faster than with 217.
  auto when_needed = [](uint32_t x) { return SAVE_REGISTERS ? formed_here(x) : x; };
  constexpr int kR = T::kRowsPerLoad;
  constexpr int kFillRows = kTileN / WAVES;             // rows of a tile each wave fetches
  constexpr int kPer = kFillRows / kR;                  // load instructions per wave and tile
  constexpr int kSlots = T::kKk / 2;                    // places between the MFMAs of a product that take loads
  constexpr int kPerSlot = (kPer + kSlots - 1) / kSlots;
  static_assert(kPer >= 1, "every wave fetches");
  const int rows_per_block = (WAVES >> a.log_heads) * kRowsPerWave;
  // Workgroups are handed to the 8 XCDs round-robin by their linear id.  Remap so that the
  // workgroups of one (document, layer, KV head), which read the same K/V, land on ONE XCD and
  // share its L2; within a unit the row blocks with the longest causal range come first.
  const int logical = a.per_xcd > 0 ? (block % kXcds) * a.per_xcd + block / kXcds : block;
  // Causal attention that fills the chip: a workgroup takes the row block with the longest key range still free and
  // then its mirror image (the shortest), so every workgroup does the same number of key tiles.  In smaller launches
  // a row block is a workgroup of its own.
  const int of_slot = a.slots.quotient(logical), of_hg = a.head_groups.quotient(of_slot), of_g = a.kv_heads.quotient(of_hg);
  const int rb_first = a.row_blocks - 1 - (logical - of_slot * a.slots.divisor);
  const int rb_second = a.row_blocks - 1 - rb_first;
  const int passes = (a.paired && rb_second != rb_first) ? 2 : 1;
  const int hg = of_slot - of_hg * a.head_groups.divisor;
  const int g = of_hg - of_g * a.kv_heads.divisor;
  const int bl = of_g;
  const int b = a.layers.quotient(bl), l = bl - b * a.layers.divisor;
  const int wu = __builtin_amdgcn_readfirstlane(w);  // the wave's index as a scalar: what depends on it stays scalar
  char* const k_s = ring;
  char* const v_s = k_s + 2 * Y::kTile;
  const int h_of_wave = ((g * a.head_groups.divisor + hg) << a.log_heads) + (wu & ((1 << a.log_heads) - 1));
  const int n_c = a.n_c;
  auto unit = [&](const UnitView& v, int head) { return v.ptr + (b * v.sb + l * v.sl + head * v.sh); };

  // ---- global -> LDS staging of one 64-key tile, without a stop in registers ----
  // buffer_load ... lds: a wave-level instruction moves 64 x 16 B from per-lane global addresses to 1 KB of consecutive
  // LDS.  The swizzle of a row's segments (Lay) is realised by the loading lane, which fetches global segment
  // (its position in the LDS row) ^ swz(row).  The candidates are tiled segment by segment, the cache first, so that every
  // tile lies in one segment and is fetched with one buffer resource.  Rows behind the end of a segment are out of
  // the resource's range and read as zeros; their logits are masked.
  typedef __attribute__((address_space(3))) char* lds_char_ptr;
  auto lds_addr = [](char* p) { return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_char_ptr)p)); };
  const int fill_row0 = kFillRows * wu;  // first tile row this wave fetches
  const uint32_t fill_lds0 = lds_addr(k_s) + fill_row0 / kR * Y::kBlock;
  const int cache_tiles = (n_c + kTileN - 1) / kTileN;
  // One stream of tiles (K or V): the resource of the segment it is in and, per load instruction, the lane's byte offset
  // of its next tile (row and segment; the range check covers this offset only, so no part of it is a scalar).
  struct Stream {
    i32x4 rs;
    uint32_t step;
    uint32_t voff[kPer];
  };
  auto seg_words = [&](const UnitView& v, int rows_) { return buffer_words(unit(v, g), rows_ > 0 ? (rows_ - 1) * v.ss + 2 * D : 0); };
  const i32x4 k_rs_cache = seg_words(a.k_cache, n_c), k_rs_chunk = seg_words(a.k_chunk, a.c);
  const i32x4 v_rs_cache = seg_words(a.v_cache, n_c), v_rs_chunk = seg_words(a.v_chunk, a.c);
  // Positions the stream at the first tile of a segment.  Of the tiles that are read only the last holds rows behind the
  // segment's end.  If that is the first tile, their offsets are set here; else they are the sum of two numbers of at
  // most 2^31, an offset inside and the step, and so at least the resource's size without a wrap.
  auto enter = [&](Stream& s, const i32x4& rs, const UnitView& v, int seg_rows) {
    s.rs = rs;
    s.step = v.tile_step;
    const uint32_t lanex = when_needed(lane);
    const int fill_row = fill_row0 + lanex / T::kSegs, fill_seg16 = ((lanex % T::kSegs) ^ Y::swz(lanex / T::kSegs)) * 16;
#pragma unroll
    for (int x = 0; x < kPer; ++x) {
      const int row = fill_row + kR * x;
      s.voff[x] = row < seg_rows ? static_cast<uint32_t>(row) * static_cast<uint32_t>(v.ss) + static_cast<uint32_t>(fill_seg16) : kOutside;
    }
  };
  // load x of the stream's next tile into the wave's rows of tile buffer BUF (0, 1: K; 2, 3: V)
  auto issue_one = [&](const Stream& s, auto buf, auto x) {
    load_lds_unwatched<decltype(buf)::value * Y::kTile + decltype(x)::value * Y::kBlock>(s.rs, fill_lds0, s.voff[decltype(x)::value], 0);
  };
  using std::integral_constant;
  auto fetch = [&](Stream& s, auto buf) {  // the stream's next tile
    [&]<int... X>(std::integer_sequence<int, X...>) { (issue_one(s, buf, integral_constant<int, X>{}), ...); }(std::make_integer_sequence<int, kPer>{});
  };
  auto advance = [&](Stream& s) {
#pragma unroll
    for (int x = 0; x < kPer; ++x) s.voff[x] += s.step;
  };

  // per-lane LDS read bases (bytes inside a half tile)
  // A operand of S^T: key row `col`, head_dim segment 2 kk + grp
  int k_base[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) k_base[c] = Y::at(col, Y::kStep * c + grp);
  auto read_row_operand = [&](const char* half_tile, int kk) {
    const int c = 2 * kk / Y::kStep;
    return *reinterpret_cast<const uint4*>(half_tile + k_base[c] + (2 * kk - Y::kStep * c) * 16);
  };
  // V^T operand through transpose reads.  The 16-lane group q16 = lane / 16 serves MFMA rows
  // 16 (q16 % 2) .. +15 for contraction lane group q16 / 2; output row c' of tile r is head_dim
  // 16 r + (c' % 16) + D / 2 (c' / 16).  Source lane s16 points at 4 consecutive head_dim values of key
  // row 4 (q16 / 2) + s16 / 4 (+ 8 rd + 16 half): segment 2 r + D / 16 (q16 % 2) + (s16 % 4) / 2.
  const int s16 = lane % 16, q16 = lane / 16;
  int v_base[2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
    v_base[c] = Y::at(4 * (q16 / 2) + s16 / 4, T::kSegs / 2 * (q16 % 2) + Y::kStep * c + (s16 % 4) / 2) + 8 * (s16 % 2);
  // read rd (keys 8 rd .. + 7) of contraction step `half` for output tile r
  auto read_v_operand = [&](const char* half_tile, int half, int r, int rd) {
    const int c = 2 * r / Y::kStep;
    return lds_read_tr16(half_tile + v_base[c] + (16 * half + 8 * rd) / kR * Y::kBlock + (2 * r - Y::kStep * c) * 16);
  };

  // The first step of a row block multiplies p_prev = 0 with the second half of V buffer 1, which nothing has filled
  // yet in the first row block, and rows behind the end of a segment are never multiplied with anything but 0: the V
  // buffers are zeroed once (0 x garbage could be NaN), in front of the first loads into them.
  auto zero_v = [&] {
    for (int at = 16 * tid; at < 2 * Y::kTile; at += 16 * WAVES * 64)
      *reinterpret_cast<uint4*>(v_s + at) = make_uint4(0u, 0u, 0u, 0u);
  };

  for (int pass = 0; pass < passes; ++pass) {
  const int rb = pass == 0 ? rb_first : rb_second;
  // MIXED: a task behind the last one has rows behind the last one
  const int task = rb * WAVES + wu, tile = MIXED ? a.group.quotient(task) : 0;
  const int h = MIXED ? (g - tile) * a.group.divisor + task : h_of_wave;
  const int row0 = MIXED ? tile * kRowsPerWave : rb * rows_per_block + (wu >> a.log_heads) * kRowsPerWave;

  const int rows = a.c;
  const int rows_until = MIXED ? (a.group.quotient(min((rb + 1) * WAVES, a.tasks) - 1) + 1) * kRowsPerWave : (rb + 1) * rows_per_block;
  const int blk_row_last = min(rows, rows_until) - 1;
  const int t_end = cache_tiles + blk_row_last / kTileN + 1;
  // candidates are numbered tile by tile here: chunk state x is candidate chunk0 + x
  const int chunk0 = cache_tiles * kTileN;
  const int wave_limit_min = chunk0 + row0;       // up to it every row sees the chunk's states
  const int chunk_masked = (wave_limit_min + 1) / 32;               // half tiles of the chunk from here on may need a mask
  int next_masked = n_c % kTileN ? n_c / 32 : chunk_masked;         // the next half tile that may need one

  // ---- Q^T operand, kept in registers: q_op[kk] = Q[row0 + col][16 kk + 8 grp ..+7] ----
  bf16x8 q_op[T::kKk];

  // ---- running softmax state: one query per lane ----
  const float c2 = a.c2;  // logits are kept in the log2 domain
  float m_run = -INFINITY, l_run = 0.f;
  float m_sub = 0.f;         // what is subtracted: m_run, or 0 for a row that has seen nothing yet (exp2(-inf) = 0)
  float m_high = -INFINITY;  // a logit above it moves m_run
  // Optional by-product: each row's log-sum-exp over the cache states alone, i.e. the running (maximum, sum) pair behind
  // the last cache tile; every row sees every cache state.
  const int snap_i = a.lse_cache != nullptr ? cache_tiles - 1 : -1;
  float m_snap = -INFINITY, l_snap = 0.f;
  f32x16 o_acc[T::kOut];
#pragma unroll
  for (int r = 0; r < T::kOut; ++r)
#pragma unroll
    for (int i = 0; i < 16; ++i) o_acc[r][i] = 0.f;

  f32x16 s_cur;            // logits of the half tile whose probabilities are computed next
  uint32_t p_prev[T::kParts][8];  // bf16 probabilities (parts) of the half tile before it, not yet multiplied with V
  Pack8 ka[T::kKk];        // K operand of the next logit product, read one step ahead
  float mx_cur;            // this lane's maximum over s_cur (before masking)
  uint64_t high;           // lanes whose maximum over s_cur (before masking) lies above m_high
#pragma unroll
  for (int y = 0; y < T::kParts; ++y)
#pragma unroll
    for (int x = 0; x < 8; ++x) p_prev[y][x] = 0u;
  // K operand from a half tile; what is read past the last tile feeds logits that are never used
  auto read_k_ops = [&](const char* k_t) {
#pragma unroll
    for (int kk = 0; kk < T::kKk; ++kk) ka[kk].u = read_row_operand(k_t, kk);
  };

  // One half step: finish the softmax of half tile hc (logits in s_cur) while the logits of the next half tile and the
  // product of the previous one's probabilities with V run on the matrix pipe.  Past either end the neighbour's
  // product is formed and not used; p_prev is zero before the first step.  v_t: the previous half tile of V.
  // issue_k(slot) / issue_v(slot) put the loads of the tile being fetched between the MFMAs.
  auto half_step = [&](int hc, const char* v_t, auto&& issue_k, auto&& issue_v, auto&& before_tail) {
    if (__builtin_expect(hc >= next_masked, 0)) {  // wave-uniform: the causal edge and the ends of the segments only
      const uint32_t lanex = when_needed(lane);
      const int limit_lane = chunk0 + min(row0 + static_cast<int>(lanex % 32), rows - 1);
      const int lim_rel = (hc < 2 * cache_tiles ? n_c - 1 : limit_lane) - 32 * hc - 4 * static_cast<int>(lanex / 32);
      if (hc + 1 >= 2 * cache_tiles) next_masked = chunk_masked;
#pragma unroll
      for (int x = 0; x < 16; ++x) s_cur[x] = minus_inf_if_negative(lim_rel - (8 * (x / 4) + (x % 4)), s_cur[x]);
      mx_cur = s_cur[0];
#pragma unroll
      for (int x = 1; x < 16; ++x) mx_cur = fmaxf(mx_cur, s_cur[x]);
      high = __ballot(mx_cur > m_high);
    }
    // Running maximum, kept lazily: softmax is invariant to the subtracted value, so m_run only has
    // to stay within kMaxSlack (log2 units) of the true row maximum to keep exp2 in range.  The vote on the
    // lanes' maxima was taken at the end of the previous step.
    if (__builtin_expect(high != 0, 0)) {  // wave-uniform and rare after the first tiles
      const float mx = fmaxf(mx_cur, __shfl_xor(mx_cur, 32, 64));
      const float m_new = fmaxf(m_run, mx * c2);
      // 0 on a row's first visible tile (m_run = -inf); 1 for a row that has seen nothing yet
      const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
      // the last P.V MFMAs of the previous step may still be in flight and the compiler cannot see them
      if constexpr (T::kOut == 4)
        wait_for_pinned_mfmas(o_acc[0], o_acc[1], o_acc[2], o_acc[3]);
      else
        wait_for_pinned_mfmas(o_acc[0], o_acc[1]);
#pragma unroll
      for (int r = 0; r < T::kOut; ++r)
#pragma unroll
        for (int x = 0; x < 16; ++x) o_acc[r][x] *= alpha;
      // the probabilities still waiting for their product with V were taken against the old maximum
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const uint32_t pw = p_prev[0][x];
        const float lo = __uint_as_float(pw << 16), hi = __uint_as_float(pw & 0xffff0000u);
        if constexpr (T::kParts == 2) {
          const uint32_t rw = p_prev[1][x];
          split_bf16x2((lo + __uint_as_float(rw << 16)) * alpha, (hi + __uint_as_float(rw & 0xffff0000u)) * alpha,
                       p_prev[0][x], p_prev[1][x]);
        } else {
          p_prev[0][x] = pack_bf16x2(lo * alpha, hi * alpha);
        }
      }
      m_run = m_new;
      m_sub = m_new == -INFINITY ? 0.f : m_new;
      m_high = (m_new + kMaxSlack) * a.inv_c2;
    }
    __builtin_amdgcn_sched_barrier(0);

    // O^T += V^T . P^T: contraction step `half` covers keys 16 half .. +15 of the half tile in the slot
    // order the S^T accumulators have: slot x of lane group grp is key 8 (x / 4) + 4 grp + (x % 4) of
    // the step, so slots 0..3 / 4..7 are two transpose reads.
    // The V^T operands of the second contraction step are read once half of the K operands are
    // spent (the empty asm with a memory clobber keeps the reads from being hoisted above it):
    // all sixteen up front would not fit the register budget.
    Pack8 va[2][T::kOut];
    auto read_v_ops = [&](int half) {
#pragma unroll
      for (int r = 0; r < T::kOut; ++r)
#pragma unroll
        for (int rd = 0; rd < 2; ++rd)
          va[half][r].h[rd] = read_v_operand(v_t, half, r, rd);
    };
    read_v_ops(0);
    __builtin_amdgcn_s_waitcnt(0xC07F | ((2 * T::kOut) << 8));  // the K operands are here: one wait for all of them
    // kKk MFMAs of S^T, then 2 kOut kParts of O^T: sixteen (head_dim 64: twelve).  The exponential of logit x of half
    // tile i is issued right before MFMA x + 1 (head_dim 64: two each before the first kPairs of them).
    float p[16];
    float mx_nxt = 0.f;
    f32x16 s_nxt = mfma_pinned_first(ka[0].v, q_op[0]);
    constexpr int kPairs = D == 64 ? 5 : 0;
    auto exps_then_mfma = [&](int slot, f32x16& acc, const bf16x8& a, const bf16x8& bb) {
      const int x = slot < kPairs ? 2 * slot : slot + kPairs;
      if (slot < kPairs)
        exp2x2_then_mfma(fmaf(s_cur[x], c2, -m_sub), fmaf(s_cur[x + 1], c2, -m_sub), p[x], p[x + 1], acc, a, bb);
      else
        p[x] = exp2_then_mfma(fmaf(s_cur[x], c2, -m_sub), acc, a, bb);
    };
#pragma unroll
    for (int kk = 1; kk < T::kKk; ++kk) {
      exps_then_mfma(kk - 1, s_nxt, ka[kk].v, q_op[kk]);
      if (kk & 1) issue_k(kk / 2);
      if (kk == T::kKk / 2) {
        no_memory_motion();
        read_v_ops(1);
      }
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int y = 0; y < T::kParts; ++y) {
        Pack8 pb;
#pragma unroll
        for (int x = 0; x < 4; ++x) pb.w[x] = p_prev[y][4 * half + x];
        if (y == 0 && half == 0) __builtin_amdgcn_s_waitcnt(0xC07F | ((2 * T::kOut) << 8));
        if (y == 0 && half == 1) __builtin_amdgcn_s_waitcnt(0xC07F);
#pragma unroll
        for (int r = 0; r < T::kOut; ++r) {
          const int slot = T::kOut * (T::kParts * half + y) + r;  // of the second product: 0 .. 7
          exps_then_mfma(T::kKk - 1 + slot, o_acc[r], va[half][r].v, pb.v);
          if (slot & 1) issue_v(slot / 2);
          // The lane's maximum of the next half tile's logits, one v_max3 per MFMA slot.  s_nxt was
          // completed by the last MFMA of the first product; three further MFMAs have been issued since.
          const int m3 = slot - 2;  // 0 .. 5
          if (m3 == 0) mx_nxt = max3_pinned(s_nxt[0], s_nxt[1], s_nxt[2]);
          if (m3 > 0) mx_nxt = max3_pinned(mx_nxt, s_nxt[2 * m3 + 1], s_nxt[2 * m3 + 2]);
        }
      }
    }
    before_tail();
    if constexpr (kPairs == 0) p[15] = exp2_pinned(fmaf(s_cur[15], c2, -m_sub));
    mx_nxt = max3_pinned(mx_nxt, s_nxt[13], s_nxt[14]);
    mx_nxt = fmaxf(mx_nxt, s_nxt[15]);
    high = __ballot(mx_nxt > m_high);
    uint32_t p_cur[T::kParts][8];
    if constexpr (T::kParts == 2) {
      float psum[2] = {p[0], p[1]};
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        split_bf16x2(p[2 * x], p[2 * x + 1], p_cur[0][x], p_cur[1][x]);
        if (x > 0) {
          psum[0] += p[2 * x];
          psum[1] += p[2 * x + 1];
        }
      }
      l_run += psum[0] + psum[1];
    } else {
      // the row sum is taken over the bf16-rounded probabilities, the values P.V uses: one v_dot2
      // with (1, 1) adds a pair
      float psum = 0.f;
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        p_cur[0][x] = pack_bf16x2(p[2 * x], p[2 * x + 1]);
        psum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p_cur[0][x]),
                                               __builtin_bit_cast(bf16x2, 0x3f803f80u), psum, false);
      }
      l_run += psum;
    }
    // keep the probabilities in this block: without a use here the optimiser sinks the exponentials
    // to their first use in the next step, behind the MFMAs they are meant to overlap with
#pragma unroll
    for (int y = 0; y < T::kParts; ++y) keep_values_here(p_cur[y], l_run);
    __builtin_amdgcn_sched_barrier(0);
    s_cur = s_nxt;
    mx_cur = mx_nxt;
#pragma unroll
    for (int y = 0; y < T::kParts; ++y)
#pragma unroll
      for (int x = 0; x < 8; ++x) p_prev[y][x] = p_cur[y][x];
  };

  // ---- first requests: K 0, the query rows | V 0, K 1 (the first two are waited for first) ----
  Stream sk, sv;
  auto k_to_chunk = [&] { enter(sk, k_rs_chunk, a.k_chunk, a.c); };  // in front of tile cache_tiles
  auto v_to_chunk = [&] { enter(sv, v_rs_chunk, a.v_chunk, a.c); };
  if (cache_tiles > 0) {
    enter(sk, k_rs_cache, a.k_cache, n_c);
    enter(sv, v_rs_cache, a.v_cache, n_c);
  } else {
    k_to_chunk();
    v_to_chunk();
  }
  fetch(sk, integral_constant<int, 0>{});
  advance(sk);
  // The wave's 32 query rows come in through LDS as well: whole rows, kR per load instruction, laid out like half a
  // key tile, from where the B operand is read like a key operand.  Loading them straight
  // into the operand layout would put 64 scattered 16-byte pieces into every load instruction.
  char* const q_t = q_stage + wu * Y::kHalf;
  {
    const int q_ss2 = a.q.ss;
    const i32x4 q_rs = buffer_words(unit(a.q, h), (rows - 1) * q_ss2 + 2 * D);
    const uint32_t q_lds = lds_addr(q_t);
    const uint32_t lanex = formed_here(lane);
    const int r_in = lanex / T::kSegs, seg16 = ((lanex % T::kSegs) ^ Y::swz(lanex / T::kSegs)) * 16;
#pragma unroll
    for (int i = 0; i < 32 / kR; ++i) {
      const int row = min(row0 + kR * i + r_in, rows - 1);  // rows past the end repeat the last one; never stored
      load_lds_unwatched<0>(q_rs, q_lds + i * Y::kBlock, max(row, 0) * q_ss2 + seg16, 0);
    }
  }
  if (pass == 0) {
    zero_v();
    lds_writes_and_barrier();
  }
  fetch(sv, integral_constant<int, 2>{});
  advance(sv);
  if (cache_tiles == 1) k_to_chunk();
  fetch(sk, integral_constant<int, 1>{});
  advance(sk);
  wait_loads_and_barrier<2 * kPer, true>();  // K 0 and the query rows have landed
  // Position shift: the query rows arrive without rotary embedding and are rotated here, in the staging
  // region, to position a.q_rope_pos0 + row, before the operands are read (only a few registers are live at
  // this point; rotating the operands in registers pushed the whole kernel over its register budget).
  // Element i of a row pairs with element i + D / 2: 16-byte segment sg with segment sg + D / 16.  A lane takes
  // one (row, sg) of the wave's 32 x D / 16 per round; a wave touches only its row tile's rows.
  if (ROTATE_Q) {
    constexpr int kPairs = T::kSegs / 2, kRoundRows = 64 / kPairs;
#pragma unroll 1
    for (int round = 0; round < 32 / kRoundRows; ++round) {
      const int r = kRoundRows * round + lane / kPairs, sg = lane % kPairs;
      uint4* lo_p = reinterpret_cast<uint4*>(q_t + Y::at(r, sg));
      uint4* hi_p = reinterpret_cast<uint4*>(q_t + Y::at(r, sg + kPairs));
      Pack8 lo, hi;
      lo.u = *lo_p;
      hi.u = *hi_p;
      const int pos = a.q_rope_pos0 + max(min(row0 + r, rows - 1), 0);
#pragma unroll
      for (int wd = 0; wd < 4; ++wd) {
        const int i0 = 8 * sg + 2 * wd;
        float s0, c0, s1, c1;
        rope_sincos_bf16(pos, i0, D, a.rope_log2_base, s0, c0);
        rope_sincos_bf16(pos, i0 + 1, D, a.rope_log2_base, s1, c1);
        rope_rotate_words(lo.w[wd], hi.w[wd], c0, s0, c1, s1, lo.w[wd], hi.w[wd]);
      }
      *lo_p = lo.u;
      *hi_p = hi.u;
    }
  }
#pragma unroll
  for (int kk = 0; kk < T::kKk; ++kk) {
    Pack8 p;
    p.u = read_row_operand(q_t, kk);
    q_op[kk] = p.v;
  }
  read_k_ops(k_s);
#pragma unroll
  for (int i = 0; i < 16; ++i) s_cur[i] = 0.f;
#pragma unroll
  for (int kk = 0; kk < T::kKk; ++kk)  // logits of the first half tile
    s_cur = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk].v, q_op[kk], s_cur, 0, 0, 0);
  mx_cur = s_cur[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) mx_cur = fmaxf(mx_cur, s_cur[i]);
  high = ~uint64_t{0};
  read_k_ops(k_s + Y::kHalf);

  // One 64-key tile.  `parity` is the tile's buffer (tile i lives in buffer
  // i % 2), so every LDS address is a per-lane register plus an immediate offset, and nothing branches but for the rare
  // cases.  It always fetches; what it fetches past the block's range is not read.
  const bool early = WAVES == 8 && wu >= 4;
  auto no_issue = [](int) {};
  auto issue_slot = [&](const Stream& s, auto buf, int slot) {
    [&]<int... X>(std::integer_sequence<int, X...>) {
      ((X / kPerSlot == slot ? issue_one(s, buf, integral_constant<int, X>{}) : (void)0), ...);
    }(std::make_integer_sequence<int, kPer>{});
  };
  auto rare_events = [&](int i) {
    if (__builtin_expect(i + 2 == cache_tiles, 0)) k_to_chunk();
    if (__builtin_expect(i + 1 == cache_tiles, 0)) v_to_chunk();
  };
  auto note_cache = [&](int i) {
    if (__builtin_expect(i == snap_i, 0)) {
      m_snap = m_run;
      l_snap = l_run;
    }
  };
  auto tile_step = [&](auto parity, int i) {
    constexpr int P = decltype(parity)::value;
    // P.V of the second half of tile i - 1 (before the first tile: p_prev = 0 times the zeros written above,
    // or times stale finite data in later row blocks)
    half_step(2 * i, v_s + (1 - P) * Y::kTile + Y::kHalf, no_issue, no_issue, [&] { if (early) wait_loads_and_barrier<0, false>(); });
    // Every wave has read the second half of K tile i and the last of V tile i - 1: their buffers
    // take K tile i + 2 and V tile i + 1, which are first read after the next barrier.
    if (!early) wait_loads_and_barrier<0, false>();
    read_k_ops(k_s + (1 - P) * Y::kTile);  // K tile i + 1, first half
    rare_events(i);
    constexpr integral_constant<int, P> kbuf{};
    constexpr integral_constant<int, 3 - P> vbuf{};
    half_step(2 * i + 1, v_s + P * Y::kTile, [&](int slot) { issue_slot(sk, kbuf, slot); },
              [&](int slot) { issue_slot(sv, vbuf, slot); }, [] {});
    advance(sk);
    advance(sv);
    note_cache(i);
    read_k_ops(k_s + (1 - P) * Y::kTile + Y::kHalf);  // K tile i + 1, second half
  };
  for (int i = 0; i < t_end; i += 2) {
    tile_step(integral_constant<int, 0>{}, i);
    if (i + 1 < t_end) tile_step(integral_constant<int, 1>{}, i + 1);
  }
  {  // the product of the last half tile
    const char* v_t = v_s + ((t_end - 1) & 1) * Y::kTile + Y::kHalf;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      Pack8 va[T::kOut];
#pragma unroll
      for (int r = 0; r < T::kOut; ++r)
#pragma unroll
        for (int rd = 0; rd < 2; ++rd)
          va[r].h[rd] = read_v_operand(v_t, half, r, rd);
#pragma unroll
      for (int y = 0; y < T::kParts; ++y) {
        Pack8 pb;
#pragma unroll
        for (int x = 0; x < 4; ++x) pb.w[x] = p_prev[y][4 * half + x];
#pragma unroll
        for (int r = 0; r < T::kOut; ++r) o_acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[r].v, pb.v, o_acc[r], 0, 0, 0);
      }
    }
  }
  barrier_after_lds_fill();  // the buffers are free for the output tiles and for the next row block

  const float l_snap_tot = l_snap + __shfl_xor(l_snap, 32, 64);
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const int64_t row_id0 = (static_cast<int64_t>(bl) * a.q_heads + h) * rows;  // of the lse outputs
  // The output tile leaves through LDS: a lane holds 4-element pieces of ONE query row (256 bytes
  // between neighbouring lanes), so direct stores put 64 scattered 8-byte pieces into every store
  // instruction and keep the compute unit's address path busy for microseconds per row block.  Rows past the end are
  // sent out of the output resource's range and dropped.
  const int out_ss = a.out.ss;
  const __amdgpu_buffer_rsrc_t out_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(unit(a.out, h)), 0,
                                                                          (rows - 1) * out_ss + 2 * D, kBufferFlags);
  const uint32_t lanex = formed_here(lane), colx = SAVE_REGISTERS ? lanex % 32 : formed_here(col), grpx = SAVE_REGISTERS ? lanex / 32 : grp;
  // Each wave parks its 32 x D tile in its own part of the tile buffers (free after the barrier above; 16-byte
  // segments XOR-swizzled by the row: column-wise writes spread over the banks) and stores it back as whole rows.  A
  // lane and its partner l ^ 32 hold the two halves of every segment: a swap gives each of them whole segments.
  char* const o_tile = ring + wu * (32 * kRowBytes);
  char* const o_s = o_tile + colx * kRowBytes;
  const int c_swz = colx % T::kSegs;
  const float inv = 1.f / l_tot;
  float lse = (m_run + log2f(l_tot)) * kLn2;
  float zero = 0.f;  // NaN where an output of the lane is not finite
#pragma unroll
  for (int r = 0; r < T::kOut; ++r)
#pragma unroll
    for (int ip = 0; ip < 2; ++ip) {
      // registers 4 i4 .. + 3, i4 = 2 ip + x, are rows c' = 8 i4 + 4 grp + 0..3 -> head_dim 16 r + (c' % 16) + D / 2 (c' / 16)
      uint32_t wd[2][2];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
        {
          const float lo = o_acc[r][8 * ip + 4 * x + 2 * y] * inv, hi = o_acc[r][8 * ip + 4 * x + 2 * y + 1] * inv;
          if constexpr (D == 64) zero = fmaf(hi, 0.f, fmaf(lo, 0.f, zero));
          wd[x][y] = pack_bf16x2(lo, hi);
        }
      uint4 piece;  // segment 2 r + grp + D / 16 ip
      swap_halves(wd[0][0], wd[1][0], piece.x, piece.z);
      swap_halves(wd[0][1], wd[1][1], piece.y, piece.w);
      *reinterpret_cast<uint4*>(o_s + ((2 * r + T::kSegs / 2 * ip + grpx) ^ c_swz) * 16) = piece;
    }
  if constexpr (D == 64) {  // rows that are not finite once more, see attn_row.h; the query rows are still in q_t
    const uint64_t lanes = __ballot(zero != 0.f);
    uint32_t again = static_cast<uint32_t>(lanes | (lanes >> 32));
    if (__builtin_expect(again != 0, 0)) {  // wave-uniform
      auto row_of = [&](const UnitView& cache, const UnitView& chunk) {
        const char *const in_cache = unit(cache, g), *const in_chunk = unit(chunk, g);
        const int64_t ss_cache = cache.ss, ss_chunk = chunk.ss;
        return [=](int j) {
          return reinterpret_cast<const uint16_t*>(j < n_c ? in_cache + j * ss_cache : in_chunk + (j - n_c) * ss_chunk);
        };
      };
      for (; again != 0; again &= again - 1) {
        const int r = __builtin_ctz(again), t = row0 + r;
        if (t >= rows) break;
        float lse_r;
        const Floats8 o = attn_row_64(bf16x8_to_f32(*reinterpret_cast<const uint4*>(q_t + Y::at(r, lanex % 8))), n_c + t, a.scale,
                                      row_of(a.k_cache, a.k_chunk), row_of(a.v_cache, a.v_chunk), lse_r);
        if (lanex < 8)
          *reinterpret_cast<uint4*>(o_tile + r * kRowBytes + (lanex ^ (r % T::kSegs)) * 16) =
              make_uint4(pack_bf16x2(o.x[0], o.x[1]), pack_bf16x2(o.x[2], o.x[3]), pack_bf16x2(o.x[4], o.x[5]),
                         pack_bf16x2(o.x[6], o.x[7]));
        if (static_cast<int>(colx) == r && !(fabsf(lse) < INFINITY)) lse = lse_r;
      }
      no_memory_motion();
    }
  }
  const int t = row0 + static_cast<int>(SAVE_REGISTERS ? colx : col);
  if (grpx == 0 && t < rows) {
    if (a.lse_cache != nullptr) a.lse_cache[row_id0 + t] = (m_snap + log2f(l_snap_tot)) * kLn2;
    if (a.lse != nullptr) a.lse[row_id0 + t] = lse;
  }
  const char* const o_r = o_tile + lanex * 16;  // row lanex / kSegs of a kR-row group
  const int r_in = lanex / T::kSegs, pos = lanex % T::kSegs;
  static_assert((kR & (kR - 1)) == 0 && kR <= T::kSegs, "row kR i + r_in modulo kSegs is (kR i modulo kSegs) ^ r_in");
  const int seg16 = (pos ^ r_in) * 16, rows_left = rows - row0 - r_in;
  uint32_t at = static_cast<uint32_t>(row0 + r_in) * static_cast<uint32_t>(out_ss);
#pragma unroll
  for (int i = 0; i < 32 / kR; ++i, at += kR * static_cast<uint32_t>(out_ss)) {
    const u32x4 piece = *reinterpret_cast<const u32x4*>(o_r + kR * i * kRowBytes);
    const uint32_t row_at = kR * i < rows_left ? at : kOutside;
    __builtin_amdgcn_raw_buffer_store_b128(piece, out_rs, row_at + (seg16 ^ (kR * i % T::kSegs * 16)), 0, 0);
  }
  __syncthreads();  // the parked tiles have been read back: the next row block may fill the buffers
  }  // pass
}

// Eight waves, launches that fill the chip: two 32-row tiles of the four heads of a KV group (or the equivalent
// split for smaller groups) share every K/V tile, which halves the fetch traffic per MFMA
// against four waves; one workgroup per CU, two waves per SIMD.
// Four waves, smaller launches: half of the rows per workgroup and one wave per SIMD, which has the matrix pipe to itself
// (attn_launch has the line between the two).  A row's sums run over the same tiles in the same order in either: its
// bits do not depend on the size of the launch.  (Splitting the keys of a row between two pairs of waves as well gave
// 19.8 instead of 24.4 us at 32/8 heads, 512 rows over 768 + 512 states; with it a row's bits would follow the launch.)
// PER_SIMD: waves per SIMD that the registers are left for.  Three at head_dim 64 with four waves a workgroup (157 registers),
// three workgroups to a compute unit: smaller pieces, where the larger ones leave the last turn nearly empty.
template <int D, int WAVES, bool MIXED, int PER_SIMD>
__global__ __launch_bounds__(WAVES * 64, PER_SIMD) void attn_pipe_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char ring[attn_ring_bytes<D>()];
  extern __shared__ __attribute__((aligned(1024))) char q_stage[];
  attn_pipe_body<D, WAVES, false, (PER_SIMD > 2), MIXED>(a, blockIdx.x, ring, q_stage);
}
// The same kernel for query rows that arrive without rotary embedding (position shift): they are rotated
// in the LDS staging region before the operands are read.  An instance of its own, so that the kernel
// above does not carry the extra prologue.
template <int D, int WAVES, bool MIXED, int PER_SIMD>
__global__ __launch_bounds__(WAVES * 64, PER_SIMD) void attn_pipe_kernel_rotq(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char ring[attn_ring_bytes<D>()];
  extern __shared__ __attribute__((aligned(1024))) char q_stage[];
  attn_pipe_body<D, WAVES, true, true, MIXED>(a, blockIdx.x, ring, q_stage);
}

// Chunk attention and instruction score of a step in one launch: neither reads what the other writes, and a small step
// leaves compute units idle in both.  The workgroups have the score's eight waves; those of the attention use four.
// What bounds it: the attention's chain, behind which the score disappears.  One layer of 32/8 heads, 512 rows and 64
// instruction rows over 768 + 512 states: 22.4 + 9.2 us in two launches, 23.4 in one.
// The eviction by those scores can be part of the launch too: the workgroup that is the last of its unit's strips to have
// written its column selects and moves the unit's rows (into the other buffer, which nothing here reads).  No workgroup waits
// for another one.  A document of such a layer, 7941 tokens, 524 -> 385 us; 8/4 heads, 43 rows and 86 instruction rows over 463 +
// 430 states, a step 24.3 -> 17.7.
constexpr int kTailRows = 8;  // rows of a thread in flight: one workgroup moves all rows of a unit
template <int TPW>
using TailLds = SelectLds<TPW * kStripWaves * kStripKeys / kStripThreads + 1, kStripThreads, 11>;
template <int D, bool ROTATE_Q, int ROW_TILES, int TPW>
__global__ __launch_bounds__(kStripThreads, 1) void attn_score_kernel(AttnArgs a, int score_blocks, StripArgs s, StepTail t) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  __shared__ int last;
  const int block = blockIdx.x;
  if (block >= score_blocks) {
    if (threadIdx.x >= kThreads) return;  // an ended wave counts at no barrier
    attn_pipe_body<D, kWaves, ROTATE_Q, true>(a, block - score_blocks, smem, smem + attn_ring_bytes<D>());
    return;
  }
  constexpr int kItems = TPW * kStripWaves * kStripKeys / kStripThreads + 1;
  TailLds<TPW>& lds = *reinterpret_cast<TailLds<TPW>*>(smem);
  int32_t* const sel = reinterpret_cast<int32_t*>(smem + sizeof(TailLds<TPW>));
  int unit = 0, r0 = 0;
  if (t.then == Then::kGather) {
    unit = block / t.job.parts;
    r0 = (block - unit * t.job.parts) * t.job.part_rows;
  } else {
    unit = strip_score_body<D, ROW_TILES, TPW, ROTATE_Q, true>(s, block, smem);
    if (t.then == Then::kNothing) return;
    // The wave's part of the column has been written through.  (A fence would write back all that its XCD has not yet,
    // the attention's output among it: 16 layers of 8/4 heads, 176 rows over 153 states, two strips a unit, 33.7 us a step with
    // fences, 21.4 without.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (s.strips > 1) {
      if (threadIdx.x == 0) {
        last = __hip_atomic_fetch_add(t.tickets + unit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == s.strips - 1;
        if (last) __hip_atomic_store(t.tickets + unit, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      if (!last) return;
    }
  }
  const int r1 = min(r0 + t.job.part_rows, t.job.rows);
  if (t.job.sums > 1)
    evict_rows<kItems, kStripThreads, 11, Scores::kSumShared, kTailRows>(t.job, unit, unit_scores(t.job, unit), r0, r1, lds, sel);
  else
    evict_rows<kItems, kStripThreads, 11, Scores::kOneHead, kTailRows>(t.job, unit, unit_scores(t.job, unit), r0, r1, lds, sel);
}
__global__ __launch_bounds__(256) void clear_tickets_kernel(int32_t* tickets, int count) {
  const int x = blockIdx.x * 256 + threadIdx.x;
  if (x < count) tickets[x] = 0;
}

// Brings the per-range (maximum, sum) pairs of a row, part[s * rows_total + row], to one normaliser,
// left in part[row] as (log-sum-exp in the log2 domain, 1).  Done once per row here rather than by every workgroup of the column-sum launch
// (one per 256 keys), each of which walked the ranges with dependent loads in front of every chunk.
__global__ __launch_bounds__(256) void merge_partials_kernel(float2* part, int key_splits, int64_t rows_total) {
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (row >= rows_total) return;
  float2 ps[kMaxKeySplits];
#pragma unroll
  for (int s = 0; s < kMaxKeySplits; ++s)  // independent loads; an absent range counts as (-inf, 0)
    ps[s] = s < key_splits ? part[s * rows_total + row] : make_float2(-INFINITY, 0.f);
  float m = -INFINITY;
#pragma unroll
  for (int s = 0; s < kMaxKeySplits; ++s) m = fmaxf(m, ps[s].x);
  float lsum = 0.f;
#pragma unroll
  for (int s = 0; s < kMaxKeySplits; ++s)
    if (s < key_splits) lsum += ps[s].y * exp2f(ps[s].x - m);
  part[row] = make_float2(m + log2f(lsum), 1.f);
}

// Instruction score (Eq. (1), summed form) in ONE launch for KV groups whose query rows
// (instruction rows x heads of the group, flattened) fit one LDS chunk: a workgroup owns one
// (document, layer, KV head).  All its query rows sit in LDS; wave (kw, qh) walks key tiles
// kw, kw + KW, ... (32 keys, in registers as the A operand) against q-tiles of its share qh:
//   pass 1  per-lane online (maximum, sum) over the wave's keys  -> merged over waves in LDS into
//           the row normaliser (log2 domain);
//   pass 2  the same products again, exp2(s - normaliser) summed down the query rows per key.
// Partial column sums of the q shares meet in LDS and are added in a fixed order: no atomics.
// With KREG > 0 a wave keeps its (at most KREG) key tiles in registers from the first pass to the
// second: K is read from memory once, and all its loads are in flight together at the start.
template <int D, int QT_TOTAL, int Q_SPLIT, int WAVES, int KREG>
__global__ __launch_bounds__(WAVES * 64) void instr_fused_kernel(Dims dm, View q, int rows, Segments ks,
                                                                 float* score) {
  typedef Geo<D> T;
  constexpr int kPitchK = T::kPitchK;
  constexpr int KW = WAVES / Q_SPLIT;         // waves that share the key tiles
  constexpr int QT_PER = QT_TOTAL / Q_SPLIT;  // q-tiles per wave
  constexpr int QROWS = QT_TOTAL * 32;
  extern __shared__ __attribute__((aligned(16))) char fused_smem[];
  uint16_t* q_s = reinterpret_cast<uint16_t*>(fused_smem);              // [QROWS][kPitchK]
  float2* stats_s = reinterpret_cast<float2*>(q_s + QROWS * kPitchK);   // [KW][QROWS]
  float* lse_s = reinterpret_cast<float*>(stats_s + KW * QROWS);        // [QROWS]
  float* part_s = lse_s + QROWS;                                        // [Q_SPLIT][32 * tiles]

  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64;
  const int col = lane % 32, grp = lane / 32;
  const int kw = w / Q_SPLIT, qh = w % Q_SPLIT;
  const int g = blockIdx.x % dm.Hkv, bl = blockIdx.x / dm.Hkv, b = bl / dm.L, l = bl % dm.L;
  const int n_c = ks.n_c, n = n_c + ks.c;
  const int tiles = (n + 31) / 32;
  const int total_rows = dm.G * rows;  // <= QROWS (the launcher guarantees it)
  const float c2 = dm.scale * kLog2e;

  const uint16_t* k_cache_u = unit_ptr(ks.cache, b, l, g) + 8 * grp;
  const uint16_t* k_chunk_u = unit_ptr(ks.chunk, b, l, g) + 8 * grp;
  // the strides are read here, once: a per-lane choice between the two struct fields inside the loader
  // would compile to a per-lane LOAD of the chosen field from the argument block, in front of every tile
  const int64_t k_ss_cache = ks.cache.ss, k_ss_chunk = ks.chunk.ss;
  auto load_keys = [&](int kt, bf16x8 (&k_op)[T::kKk]) {
    const int j = min(32 * kt + col, n - 1);
    const bool in_cache = j < n_c;
    const int64_t off = in_cache ? j * k_ss_cache : (j - n_c) * k_ss_chunk;
    const uint16_t* kp = (in_cache ? k_cache_u : k_chunk_u) + off;
#pragma unroll
    for (int kk = 0; kk < T::kKk; ++kk) {
      Pack8 p;
      p.u = *reinterpret_cast<const uint4*>(kp + 16 * kk);
      k_op[kk] = p.v;
    }
  };
  auto logits = [&](const bf16x8 (&k_op)[T::kKk], int qt) {  // S^T tile: 32 keys x the 32 rows of q-tile qt
    Pack8 qb[T::kKk];
    const uint16_t* qrow = &q_s[(32 * qt + col) * kPitchK + 8 * grp];
#pragma unroll
    for (int kk = 0; kk < T::kKk; ++kk) qb[kk].u = *reinterpret_cast<const uint4*>(qrow + 16 * kk);
    f32x16 s_t;
#pragma unroll
    for (int i = 0; i < 16; ++i) s_t[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < T::kKk; ++kk) s_t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_op[kk], qb[kk].v, s_t, 0, 0, 0);
    return s_t;
  };

  // The query rows go through LDS.  They are requested first and waited for BEFORE the bulk of the key
  // loads is issued: every workgroup of the launch starts at the same moment, and behind 80+ MB of key
  // requests the query rows of the slowest wave (all of them are needed before the first product) arrive
  // when the whole burst is nearly through.  Loads return in order and the compiler counts them, so the
  // first pass then starts on a wave's first key tile while its later ones are still arriving.
  constexpr int kQStep = WAVES * 64 / T::kSegs;  // rows between a thread's loads: kSegs threads per row, 16 bytes each
  static_assert(QROWS % kQStep == 0, "whole rounds of staging loads");
  constexpr int kQLoads = QROWS / kQStep;
  const int st_row = tid / T::kSegs, st_seg = tid % T::kSegs;
  i32x4 q_in[kQLoads];
#pragma unroll
  for (int x = 0; x < kQLoads; ++x) {
    const int f = min(st_row + x * kQStep, total_rows - 1);  // padding rows repeat the last row; never summed
    const int hh = f / rows, t = f % rows;
    q_in[x] = *reinterpret_cast<const i32x4*>(unit_ptr(q, b, l, g * dm.G + hh) + static_cast<int64_t>(t) * q.ss +
                                              8 * st_seg);
  }
  __builtin_amdgcn_sched_barrier(0);  // keep the issue order
  bf16x8 k_res[KREG > 0 ? KREG : 1][T::kKk];
  if constexpr (KREG > 0) load_keys(min(kw, tiles - 1), k_res[0]);  // the launcher guarantees tiles <= KW * KREG
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int x = 0; x < kQLoads; ++x)
    *reinterpret_cast<i32x4*>(&q_s[(st_row + x * kQStep) * kPitchK + 8 * st_seg]) = q_in[x];
  __syncthreads();

  // With resident key tiles the first pass requests tile i + 1 when it starts on tile i: a compute unit
  // can only keep so many requests in flight, so issuing all of a wave's key loads up front would hold
  // the wave (and with it the barrier above) until most of the keys have arrived.
  auto for_my_tiles = [&](auto first_pass, auto&& tile_fn) {
    if constexpr (KREG > 0) {
#pragma unroll
      for (int i = 0; i < KREG; ++i) {
        if constexpr (decltype(first_pass)::value) {
          __builtin_amdgcn_sched_barrier(0);
          if (i + 1 < KREG) load_keys(min(kw + KW * (i + 1), tiles - 1), k_res[i + 1]);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (kw + KW * i < tiles) tile_fn(k_res[i], kw + KW * i);  // wave-uniform
      }
    } else {
      for (int kt = kw; kt < tiles; kt += KW) {
        bf16x8 k_op[T::kKk];
        load_keys(kt, k_op);
        tile_fn(k_op, kt);
      }
    }
  };

  // ---- pass 1: row normalisers ----
  float m_run[QT_PER], l_run[QT_PER];
#pragma unroll
  for (int x = 0; x < QT_PER; ++x) {
    m_run[x] = -INFINITY;
    l_run[x] = 0.f;
  }
  for_my_tiles(std::true_type{}, [&](const bf16x8 (&k_op)[T::kKk], int kt) {
    const int valid = n - 32 * kt;  // keys of the tile that exist (wave-uniform)
#pragma unroll
    for (int x = 0; x < QT_PER; ++x) {
      const int qt = qh * QT_PER + x;
      if (32 * qt >= total_rows) continue;  // wave-uniform
      f32x16 s_t = logits(k_op, qt);
      if (valid < 32) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i / 4) + 4 * grp + (i % 4) >= valid) s_t[i] = -INFINITY;
      }
      float mx = s_t[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s_t[i]);
      const float m_new = fmaxf(m_run[x], mx * c2);  // -inf only while the lane has seen no key at all
      const float alpha = (m_new == m_run[x]) ? 1.f : __builtin_amdgcn_exp2f(m_run[x] - m_new);
      const float m_sub = m_new == -INFINITY ? 0.f : m_new;
      float psum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) psum += __builtin_amdgcn_exp2f(fmaf(s_t[i], c2, -m_sub));
      l_run[x] = fmaf(l_run[x], alpha, psum);
      m_run[x] = m_new;
    }
  });
#pragma unroll
  for (int x = 0; x < QT_PER; ++x) {  // the two lane halves saw different keys of every tile
    const float m_o = __shfl_xor(m_run[x], 32, 64), l_o = __shfl_xor(l_run[x], 32, 64);
    const float mm = fmaxf(m_run[x], m_o);
    const float lt = l_run[x] * (m_run[x] == mm ? 1.f : __builtin_amdgcn_exp2f(m_run[x] - mm)) +
                     l_o * (m_o == mm ? 1.f : __builtin_amdgcn_exp2f(m_o - mm));
    if (grp == 0) stats_s[kw * QROWS + 32 * (qh * QT_PER + x) + col] = make_float2(mm, lt);
  }
  __syncthreads();
  if (tid < QROWS) {
    float v = INFINITY;  // padding rows contribute exp2(-inf) = 0
    if (tid < total_rows) {
      float mm = -INFINITY;
#pragma unroll
      for (int x = 0; x < KW; ++x) mm = fmaxf(mm, stats_s[x * QROWS + tid].x);
      float lsum = 0.f;
#pragma unroll
      for (int x = 0; x < KW; ++x) {
        const float2 ps = stats_s[x * QROWS + tid];
        lsum += ps.y * (ps.x == mm ? 1.f : exp2f(ps.x - mm));
      }
      v = mm + log2f(lsum);
    }
    lse_s[tid] = v;
  }
  __syncthreads();

  // ---- pass 2: column sums of exp2(s - normaliser) ----
  float lse2[QT_PER];
#pragma unroll
  for (int x = 0; x < QT_PER; ++x) lse2[x] = lse_s[32 * (qh * QT_PER + x) + col];
  for_my_tiles(std::false_type{}, [&](const bf16x8 (&k_op)[T::kKk], int kt) {
    float acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int x = 0; x < QT_PER; ++x) {
      const int qt = qh * QT_PER + x;
      if (32 * qt >= total_rows) continue;  // wave-uniform
      const f32x16 s_t = logits(k_op, qt);
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] += __builtin_amdgcn_exp2f(fmaf(s_t[i], c2, -lse2[x]));
    }
    const float tot = reduce16_over32(acc, col);  // value index col / 2 -> key 8 (i / 4) + 4 grp + (i % 4)
    const int i = col >> 1;
    if ((col & 1) == 0) part_s[qh * 32 * tiles + 32 * kt + 8 * (i / 4) + 4 * grp + (i % 4)] = tot;
  });
  __syncthreads();
  float* dst = score + (static_cast<int64_t>(bl) * dm.Hkv + g) * n;
  for (int j = tid; j < n; j += WAVES * 64) {
    float v = part_s[j];
#pragma unroll
    for (int x = 1; x < Q_SPLIT; ++x) v += part_s[x * 32 * tiles + j];
    dst[j] = v;
  }
}

constexpr size_t kFusedLdsBudget = 150 * 1024;  // of the CU's 160 KB
template <int D>
constexpr int fused_key_tiles_in_regs() { return 5 * 128 / D; }  // 160 of a wave's 256 registers

template <int D, int QT_TOTAL, int Q_SPLIT, int WAVES>
size_t instr_fused_lds_bytes(int n) {
  constexpr int QROWS = QT_TOTAL * 32;
  const int tiles = (n + 31) / 32;
  return static_cast<size_t>(QROWS) * Geo<D>::kPitchK * 2 + static_cast<size_t>(WAVES / Q_SPLIT) * QROWS * 8 + QROWS * 4 +
         static_cast<size_t>(Q_SPLIT) * 32 * tiles * 4;
}

template <int D, int QT_TOTAL, int Q_SPLIT, int WAVES, int KREG>
hipError_t instr_fused_launch(const Dims& dm, View q, int rows, Segments ks, float* score, hipStream_t st) {
  const size_t lds = instr_fused_lds_bytes<D, QT_TOTAL, Q_SPLIT, WAVES>(ks.n_c + ks.c);
  auto kern = instr_fused_kernel<D, QT_TOTAL, Q_SPLIT, WAVES, KREG>;
  static LdsLimit limit;
  const hipError_t e = raise_lds_limit(limit, reinterpret_cast<const void*>(kern), static_cast<int>(kFusedLdsBudget));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(dm.B * dm.L * dm.Hkv), dim3(WAVES * 64), lds, st, dm, q, rows, ks, score);
  return hipGetLastError();
}


bool fits_i32(const View& v, int rows) {
  return v.ss > 0 && v.ss * static_cast<int64_t>(rows > 0 ? rows : 1) < (int64_t{1} << 31);
}

// What the kernel needs to know of a launch, and its workgroups.
template <int D, int WAVES, bool MIXED = false>
AttnArgs attn_args(const Dims& dm, View q, Segments ks, Segments vs, bool paired, View out, float* lse,
                   float* lse_cache, int q_rope_pos0, float rope_base, int* blocks) {
  const TaskShape ts = task_shape(dm.G, WAVES);
  const int rows_per_block = ts.tiles_per_block * kRowsPerWave, rows = ks.c;
  AttnArgs a;
  a.q = unit_view(q, rows, D);
  a.out = unit_view(out, rows, D);
  a.k_cache = unit_view(ks.cache, ks.n_c, D);
  a.k_chunk = unit_view(ks.chunk, ks.c, D);
  a.v_cache = unit_view(vs.cache, vs.n_c, D);
  a.v_chunk = unit_view(vs.chunk, vs.c, D);
  a.n_c = ks.n_c;
  a.c = ks.c;
  a.q_heads = dm.Hq;
  a.log_heads = ts.heads_per_block == 4 ? 2 : ts.heads_per_block - 1;
  a.row_blocks = (rows + rows_per_block - 1) / rows_per_block;
  a.tasks = dm.G * ((rows + kRowsPerWave - 1) / kRowsPerWave);
  a.group = fast_div(dm.G);
  if (MIXED) a.row_blocks = (a.tasks + WAVES - 1) / WAVES;
  a.paired = paired;
  const int slots = paired ? (a.row_blocks + 1) / 2 : a.row_blocks;
  a.slots = fast_div(slots);
  a.head_groups = fast_div(MIXED ? 1 : dm.G / ts.heads_per_block);
  a.kv_heads = fast_div(dm.Hkv);
  a.layers = fast_div(dm.L);
  const int grid = slots * a.head_groups.divisor * dm.Hkv * dm.B * dm.L;
  a.per_xcd = grid % kXcds == 0 ? grid / kXcds : 0;
  a.scale = dm.scale;
  a.c2 = dm.scale * kLog2e;
  a.inv_c2 = 1.f / a.c2;
  a.lse = lse;
  a.lse_cache = lse_cache;
  a.q_rope_pos0 = q_rope_pos0;
  a.rope_log2_base = q_rope_pos0 >= 0 ? log2f(rope_base) : 0.f;
  *blocks = grid;
  return a;
}

template <int D, int WAVES, bool MIXED, int PER_SIMD = D == 128 || WAVES < 8 ? 1 : 2>
hipError_t attn_pipe_launch(const Dims& dm, View q, Segments ks, Segments vs, bool paired, View out, float* lse,
                            float* lse_cache, hipStream_t st, int q_rope_pos0, float rope_base) {
  int grid = 0;
  const AttnArgs a = attn_args<D, WAVES, MIXED>(dm, q, ks, vs, paired, out, lse, lse_cache, q_rope_pos0, rope_base, &grid);
  constexpr int kDynBytes = attn_stage_bytes<D, WAVES>();  // next to the static ring
  static LdsLimit limit, limit_rotq;
  const auto kern = q_rope_pos0 >= 0 ? attn_pipe_kernel_rotq<D, WAVES, MIXED, PER_SIMD> : attn_pipe_kernel<D, WAVES, MIXED, PER_SIMD>;
  const hipError_t e = raise_lds_limit(q_rope_pos0 >= 0 ? limit_rotq : limit, reinterpret_cast<const void*>(kern), kDynBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(WAVES * 64), kDynBytes, st, a);
  return hipGetLastError();
}

// Workgroups of a launch with one row block each.
int64_t attn_workgroups(const Dims& dm, int rows, int waves) {
  const TaskShape ts = task_shape(dm.G, waves);
  const int block_rows = ts.tiles_per_block * kRowsPerWave;
  return static_cast<int64_t>((rows + block_rows - 1) / block_rows) * (dm.G / ts.heads_per_block) * dm.Hkv * dm.B * dm.L;
}

// The same for eight waves whose heads are mixed.
int64_t attn_workgroups_mixed(const Dims& dm, int rows) {
  constexpr int kWide = 8;
  return (static_cast<int64_t>(dm.G) * ((rows + kRowsPerWave - 1) / kRowsPerWave) + kWide - 1) / kWide * dm.Hkv * dm.B * dm.L;
}

bool attn_segments_fit(const Segments& ks, const Segments& vs) {
  return fits_i32(ks.cache, ks.n_c) && fits_i32(ks.chunk, ks.c) && fits_i32(vs.cache, vs.n_c) && fits_i32(vs.chunk, vs.c);
}

template <int D, bool ROTATE_Q, int ROW_TILES, int TPW>
hipError_t attn_score_launch(const Dims& dm, View q, Segments ks, Segments vs, View out, int q_rope_pos0, float rope_base,
                             View q_instr, int instr_rows, float* part, const Eviction* evict, int32_t* tickets, hipStream_t st) {
  int blocks = 0;
  const AttnArgs a = attn_args<D, kWaves>(dm, q, ks, vs, false, out, nullptr, nullptr, q_rope_pos0, rope_base, &blocks);
  const StripArgs s = strip_args(dm, q_instr, instr_rows, ks, 32 * ROW_TILES, part);
  constexpr int kLdsBytes = std::max(attn_ring_bytes<D>() + attn_stage_bytes<D, kWaves>(), strip_lds_bytes<D, ROW_TILES>());
  static_assert(sizeof(TailLds<TPW>) + TPW * kStripWaves * kStripKeys * sizeof(int32_t) <= kLdsBytes);
  const int units = dm.B * dm.L * dm.Hkv;
  StepTail t;
  t.then = Then::kNothing;
  if (evict != nullptr) {
    Eviction e = *evict;
    e.score = ScoreSums{part, s.strips};
    t.job = evict_job(sizeof(uint16_t), dm, e);
    t.tickets = tickets;
    t.then = gather_only(e) ? Then::kGather : Then::kEvict;
    if (t.then == Then::kGather) cut_in_parts(t.job, 32, (compute_units() - blocks) / units);
  }
  const auto kern = attn_score_kernel<D, ROTATE_Q, ROW_TILES, TPW>;
  static LdsLimit limit;
  const hipError_t e = raise_lds_limit(limit, reinterpret_cast<const void*>(kern), kLdsBytes);
  if (e != hipSuccess) return e;
  const int score_blocks = units * (t.then == Then::kGather ? t.job.parts : s.strips);
  hipLaunchKernelGGL(kern, dim3(blocks + score_blocks), dim3(kStripThreads), kLdsBytes, st, a, score_blocks, s, t);
  return hipGetLastError();
}

template <int D>
hipError_t attn_launch(const Dims& dm, View q, Segments ks, Segments vs, View out, float* lse, float* lse_cache,
                       hipStream_t st, int q_rope_pos0, float rope_base) {
  if (out.ptr == nullptr || (lse_cache != nullptr && ks.n_c < 1)) return hipErrorInvalidValue;
  if (!attn_segments_fit(ks, vs)) return hipErrorInvalidValue;
  // The smallest piece of work per workgroup whose workgroups still fit the chip side by side: a launch that leaves
  // compute units idle lasts as long as its longest workgroup.  Measured in us, 32/8 heads, 512 rows over 768 + 512
  // states, head_dim 128 (row blocks in pairs | one row block | four waves, one row block):
  //   1 layer    54.6 | 34.4 | 24.4       4 layers   56.1 | 42.0 | 47.2
  //   2 layers   55.0 | 35.8 | 26.2       5 layers   56.9 | 66.8 | 61.4
  //   3 layers   56.1 | 38.4 | 42.0       8 layers   72.9 | 83.0 | 90.3
  // The best of a line is the last whose workgroups (128, 256, 192, 256 | 160, 256) are no more than the 256 compute
  // units; head_dim 64 and the other group sizes follow the same line (head_dim 64, one layer: 36.7 | 22.9 | 17.2).
  const auto workgroups = [&](int waves) { return attn_workgroups(dm, ks.c, waves); };
  const int cus = compute_units();
  if (workgroups(4) <= cus)
    return attn_pipe_launch<D, 4, false>(dm, q, ks, vs, false, out, lse, lse_cache, st, q_rope_pos0, rope_base);
  const bool mixed = attn_workgroups_mixed(dm, ks.c) < workgroups(8);
  const int64_t blocks = mixed ? attn_workgroups_mixed(dm, ks.c) : workgroups(8);
  // Beyond that pairs keep the causal work even, and singles leave less of the chip idle in the last turn.  Turns are counted in
  // blocks.  Pairs are formed within a head group; where a block is left over there pairs end unevenly, which counts as a turn
  // unless all of them fit the chip side by side and leave little of it idle.  us in pairs | single, 512 rows over 768 states of 32/8
  // heads: 5 layers 70.7 | 72.4, 9 123 | 104, 10 121 | 107, 12 124 | 118, 15 138 | 143, 17 186 | 166, 20 195 | 191, 24 221 | 240, 32
  // 297 | 310, 33 329 | 319; 700 rows over 200 states, 12 layers 123 | 104; 32/32 heads, 1024 rows over 1024 states, 5 layers 180 | 165.  An odd
  // number of row blocks: 64/8 heads, 300 rows over 700 states, 6 layers 92.0 | 76.7 (288 workgroups | 480), 17 layers 181 | 175; all side by
  // side, 48/4 heads, 598 rows over 491 states, 3 layers 50.1 | 58.5 (180 | 348), 8/2 heads, 312 rows over 369 states, 32 layers
  // 37.8 | 41.5 (192 | 320), but 32/8 heads, 1063 rows over 583 states, 2 layers 63.2 | 53.0 (144 | 272) and 32/4 heads, 263 rows over 188
  // states, 8 layers 30.7 | 28.9 (160 | 288).  Over 216 shapes the choice is 0.2 % from the better one on average, at most 8 %.
  const auto turns = [](int64_t work, int64_t places) { return (work + places - 1) / places; };
  const int64_t head_groups = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv * (mixed ? 1 : dm.G / task_shape(dm.G, 8).heads_per_block);
  const int64_t pairs = (blocks / head_groups + 1) / 2 * head_groups;  // with the blocks that are left over
  const bool side_by_side = pairs <= cus && 8 * pairs > 5 * cus;
  const int64_t pairs_turns = blocks / head_groups % 2 == 0 ? 2 * turns(pairs, cus) : side_by_side ? 2 : turns(blocks, cus) + 1;
  auto launch = mixed ? attn_pipe_launch<D, 8, true> : attn_pipe_launch<D, 8, false>;
  bool paired = blocks > cus && pairs_turns <= turns(blocks, cus);
  if constexpr (D == 64) {
    // Workgroups of four waves that leave the registers for three of them on a compute unit, one block (of half the size) each: taken
    // in place of single blocks of eight waves (faster at 23 of 23 shapes: 16/8 heads, 641 rows over 231 states, 48 layers, pairs | single
    // | three to a compute unit 199 | 208 | 166; 567 over 311, 11 layers 43.2 | 48.0 | 35.7), and where the pairs' last turn wastes more of
    // the chip.  us, pairs | three to a compute unit, 512 rows over 768 states of 32/8
    // heads: 5 layers 52.5 | 49.4, 8 62.1 | 64, 9 109.9 | 71.9, 10 109 | 82, 12 109.7 | 94.3, 16 121 | 124, 32 235 | 235; 28/4
    // heads, 300 rows over 1000 states, 16 layers 135 | 97 (in 256 rows of a head at a time); 8/8 heads, 700 rows over 900 states,
    // 40 layers 213 | 154.
    const double of_pairs = static_cast<double>(blocks) / (pairs_turns * cus);
    const double of_three = static_cast<double>(workgroups(4)) / (turns(workgroups(4), 3 * cus) * 3 * cus);
    if (blocks > cus && (!paired || of_three > of_pairs + 0.05)) {
      launch = attn_pipe_launch<64, 4, false, 3>;
      paired = false;
    }
  }
  return launch(dm, q, ks, vs, paired, out, lse, lse_cache, st, q_rope_pos0, rope_base);
}

// Partial (maximum, sum) pairs of every query row over `key_splits` ranges of the keys.
template <int D>
hipError_t lse_launch(const Dims& dm, View q, int rows, Segments ks, int key_splits, float2* part, hipStream_t st) {
  if (!fits_i32(ks.cache, ks.n_c) || !fits_i32(ks.chunk, ks.c)) return hipErrorInvalidValue;
  const TaskShape ts = task_shape(dm.G, kWaves);
  const int rows_per_block = ts.tiles_per_block * kRowsPerWave;
  const int row_blocks = (rows + rows_per_block - 1) / rows_per_block;
  const dim3 grid(row_blocks * (dm.G / ts.heads_per_block) * dm.Hkv * dm.B * dm.L * key_splits);
  hipLaunchKernelGGL(lse_mfma_kernel<D>, grid, dim3(kThreads), 0, st, dm, q, rows, ks, key_splits, part);
  return hipGetLastError();
}

template <int D>
hipError_t instr_score_launch(const Dims& dm, View q, int rows, Segments ks, float* workspace, size_t workspace_floats,
                              float* score, hipStream_t st, ScoreSums* sums) {
  const int n = ks.n_c + ks.c;
  // a short text over a candidate set that a workgroup's registers can hold one row strip of: one product
  // per (row, key)
  if (instr_strip_supported(dm, q, rows, ks))
    return launch_instr_strip(dm, q, rows, ks, workspace, workspace_floats, score, st, sums);
  // otherwise two passes over the keys; few query rows per KV group: one fused launch
  const int total_rows = dm.G * rows;
  const int tiles32 = (n + 31) / 32;
  if (total_rows <= 128 && instr_fused_lds_bytes<D, 4, 1, 8>(n) <= kFusedLdsBudget)
    return instr_fused_launch<D, 4, 1, 8, 0>(dm, q, rows, ks, score, st);
  if (total_rows <= 256 && tiles32 <= 8 * fused_key_tiles_in_regs<D>() && instr_fused_lds_bytes<D, 8, 1, 8>(n) <= kFusedLdsBudget)
    return instr_fused_launch<D, 8, 1, 8, fused_key_tiles_in_regs<D>()>(dm, q, rows, ks, score, st);
  if (total_rows <= 256 && instr_fused_lds_bytes<D, 8, 2, 16>(n) <= kFusedLdsBudget)
    return instr_fused_launch<D, 8, 2, 16, 0>(dm, q, rows, ks, score, st);
  const int tiles = (n + kTileN - 1) / kTileN;
  int splits = (tiles + 3) / 4;  // about four key tiles per workgroup
  splits = splits < 1 ? 1 : (splits > kMaxKeySplits ? kMaxKeySplits : splits);
  const int64_t rows_total = static_cast<int64_t>(dm.B) * dm.L * dm.Hq * rows;
  if (static_cast<size_t>(2) * splits * rows_total > workspace_floats) return hipErrorInvalidValue;
  float2* part = reinterpret_cast<float2*>(workspace);
  hipError_t e = lse_launch<D>(dm, q, rows, ks, splits, part, st);
  if (e != hipSuccess) return e;
  if (splits > 1) {  // one normaliser per row, in place of the first range's pairs
    hipLaunchKernelGGL(merge_partials_kernel, dim3(static_cast<unsigned>((rows_total + 255) / 256)), dim3(256), 0, st, part,
                       splits, rows_total);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return launch_colsum_mfma(dm, q, rows, ks, /*causal=*/0, workspace, 2, 1.f, score, st);
}

}  // namespace

bool mfma_path_supported(int dtype, const Dims& dm) { return dtype == CITRUS_BF16 && (dm.D == 64 || dm.D == 128); }

hipError_t launch_attn_mfma(const Dims& dm, View q, Segments ks, Segments vs, View out, float* lse, float* lse_cache,
                            hipStream_t st, int q_rope_pos0, float rope_base) {
  const auto launch = dm.D == 64 ? attn_launch<64> : attn_launch<128>;
  return launch(dm, q, ks, vs, out, lse, lse_cache, st, q_rope_pos0, rope_base);
}

// Taken where the attention's workgroups of four waves fit the chip side by side, whatever the score's 32-row strips add to them up to half
// as many again: those come first, and the shorter blocks of the attention follow them.  us a step, apart | one launch (attention's |
// score's workgroups): 32/8 heads, 512 rows over 768 states, 2 layers 47.0 | 39.5 (256 | 128); 64/8 heads, head_dim 64, 274 rows over
// 195 states 25.0 | 16.4 (144 | 144); 8/4 heads, head_dim 64, 98 rows over 65 states, 16 layers 20.6 | 12.6 (256 | 128).  Over 140 shapes of
// the range (1 to 40 layers, chunks of 32 to 1000, up to 256 | 384) one launch with the eviction in it is 0.97 to 1.64 times as fast; the
// slowest is 14/2 heads, 16 layers, 59 rows over 84 states 20.4 | 21.1 (224 | 256).  Further out it is not always: 7/1 heads, 53 rows
// over 61 states, 16 layers 19.1 | 21.4 (112 | 480).
bool attn_score_in_one_launch(const Dims& dm, const Segments& ks, const Segments& vs, const View& q_instr, int instr_rows) {
  const int64_t strips = (static_cast<int64_t>(dm.G) * instr_rows + 31) / 32;
  return attn_workgroups(dm, ks.c, kWaves) <= compute_units() && 2 * strips * dm.Hkv * dm.B * dm.L <= 3 * compute_units() && attn_segments_fit(ks, vs) &&
         instr_strip_supported(dm, q_instr, instr_rows, ks);
}

static int strips_of(const Dims& dm, int instr_rows, int n) {
  const int per_strip = instr_strip_rows(dm, instr_rows, n);
  return (dm.G * instr_rows + per_strip - 1) / per_strip;
}
bool step_needs_tickets(const Dims& dm, int instr_rows, int n, const Eviction& e) {
  return strips_of(dm, instr_rows, n) > 1 && !gather_only(e);
}
hipError_t launch_clear_tickets(const Dims& dm, int32_t* tickets, hipStream_t st) {
  const int units = dm.B * dm.L * dm.Hkv;
  hipLaunchKernelGGL(clear_tickets_kernel, dim3((units + 255) / 256), dim3(256), 0, st, tickets, units);
  return hipGetLastError();
}

// The strips are those of the launch of the score alone, in number and in height: its rule has checked that their columns fit the
// scratch, and a score's bits are the same.
hipError_t launch_attn_score_mfma(const Dims& dm, View q, Segments ks, Segments vs, View out, int q_rope_pos0, float rope_base,
                                  View q_instr, int instr_rows, float* workspace, size_t workspace_floats, float* score,
                                  hipStream_t st, ScoreSums* sums, const Eviction* evict, int32_t* tickets) {
  const int n = ks.n_c + ks.c, strips = strips_of(dm, instr_rows, n);
  if (strips > 1 && static_cast<size_t>(dm.B) * dm.L * dm.Hkv * strips * n > workspace_floats) return hipErrorInvalidValue;
  const auto choose = [&](auto head_dim, auto rotate) {
    constexpr int D = decltype(head_dim)::value;
    constexpr bool R = decltype(rotate)::value;
    if (instr_strip_rows(dm, instr_rows, n) == 64) return attn_score_launch<D, R, 2, 5>;
    return n <= kStripMaxKeysShort ? attn_score_launch<D, R, 1, 5> : attn_score_launch<D, R, 1, 10>;
  };
  const std::integral_constant<int, 64> d64;
  const std::integral_constant<int, 128> d128;
  auto launch = dm.D == 128 ? choose(d128, std::false_type()) : choose(d64, std::false_type());
  if (q_rope_pos0 >= 0) launch = dm.D == 128 ? choose(d128, std::true_type()) : choose(d64, std::true_type());
  float* const part = strips == 1 ? score : workspace;  // one strip: its column is the score
  const hipError_t e = launch(dm, q, ks, vs, out, q_rope_pos0, rope_base, q_instr, instr_rows, part, evict, tickets, st);
  return e != hipSuccess || evict != nullptr ? e : finish_strip_scores(dm, part, strips, n, score, st, sums);
}

// Instruction score in two launches: partial log-sum-exp over ranges of key tiles (enough
// workgroups to fill the chip although there are few instruction rows), then the column sums.
size_t instr_score_mfma_workspace_floats(const Dims& dm, int rows, int n) {
  const size_t two_launch = static_cast<size_t>(2) * kMaxKeySplits * dm.B * dm.L * dm.Hq * rows;
  const size_t strips = instr_strip_workspace_floats(dm, rows, n);
  return two_launch > strips ? two_launch : strips;
}

hipError_t launch_instr_score_mfma(const Dims& dm, View q, int rows, Segments ks, float* workspace,
                                   size_t workspace_floats, float* score, hipStream_t st, ScoreSums* sums) {
  const auto launch = dm.D == 64 ? instr_score_launch<64> : instr_score_launch<128>;
  return launch(dm, q, rows, ks, workspace, workspace_floats, score, st, sums);
}

}  // namespace citrus
