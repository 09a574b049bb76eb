// One workgroup of the single-product instruction score (see instr_strip.hip, which launches it).
#pragma once

#include "mfma_common.h"

namespace citrus {
namespace {

constexpr int kStripKeys = 32;   // keys per tile
constexpr int kStripWaves = 8;
constexpr int kStripThreads = kStripWaves * 64;
constexpr int kStripMaxKeysShort = kStripWaves * 5 * kStripKeys;  // 1280: five key tiles per wave
constexpr int kStripMaxKeysLong = kStripWaves * 10 * kStripKeys;  // 2560: 32-row strips, ten key tiles per wave

// What a workgroup of the score works on, prepared on the host.
struct StripArgs {
  View q;
  Segments ks;
  int Hkv, L, G, rows;          // rows of a head
  int strips;                   // of a unit, one per workgroup
  FastDiv per_unit, kv_heads, layers, head_rows;  // workgroup -> (strip, KV head, layer); flattened row -> head
  int per_xcd;                  // workgroups per XCD, 0: not a whole number
  float c2;                     // softmax scale, log2 domain
  float* part;                  // [units][strips][n]
};

inline StripArgs strip_args(const Dims& dm, const View& q, int rows, const Segments& ks, int strip_rows, float* part) {
  StripArgs a;
  a.q = q;
  a.ks = ks;
  a.Hkv = dm.Hkv;
  a.L = dm.L;
  a.G = dm.G;
  a.rows = rows;
  a.strips = (dm.G * rows + strip_rows - 1) / strip_rows;
  a.per_unit = fast_div(a.strips);
  a.kv_heads = fast_div(dm.Hkv);
  a.layers = fast_div(dm.L);
  a.head_rows = fast_div(rows);
  const int groups = dm.B * dm.L * dm.Hkv * a.strips;
  a.per_xcd = groups % kXcds == 0 ? groups / kXcds : 0;
  a.c2 = dm.scale * kLog2e;
  a.part = part;
  return a;
}

// Key tiles of 32 rows in LDS: rows unpadded, segments XOR-swizzled (Geo), a wave-level load fills kR rows.
template <int D>
struct StripGeo {
  static constexpr int kRowBytes = Geo<D>::kRowBytes, kSegs = Geo<D>::kSegs, kR = Geo<D>::kRowsPerLoad, kKk = Geo<D>::kKk;
  static constexpr int kTile = kStripKeys * kRowBytes;
  static constexpr int kLoads = kStripKeys / kR;  // load instructions of a tile
};

// The 16-byte operands of 32 tile rows, read from LDS.  Written as asm: while LDS-direct loads are in flight
// the compiler drains the vector-memory counter in front of every LDS read it can see (it cannot tell that they fill
// another buffer).  The block waits for its own reads.
__device__ inline void lds_read_four(bf16x8* a, const uint32_t (&addr)[4]) {
  i32x4 r0, r1, r2, r3;
  asm volatile(
      "ds_read_b128 %0, %4\n\t"
      "ds_read_b128 %1, %5\n\t"
      "ds_read_b128 %2, %6\n\t"
      "ds_read_b128 %3, %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3)
      : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3])
      : "memory");
  a[0] = __builtin_bit_cast(bf16x8, r0); a[1] = __builtin_bit_cast(bf16x8, r1);
  a[2] = __builtin_bit_cast(bf16x8, r2); a[3] = __builtin_bit_cast(bf16x8, r3);
}

// LDS-direct loads complete in order and are counted by the issuing wave's vector-memory counter.  The
// waits are the compiler's own builtin so that its counter bookkeeping knows about them; the empty asm
// with a memory clobber keeps the LDS reads of the tile behind the wait.
// s_waitcnt immediate on gfx9: vmcnt[3:0] = bits 3:0, expcnt = bits 6:4, lgkmcnt = bits 11:8, vmcnt[5:4] = bits 15:14.
template <int LEFT>
__device__ inline void wait_all_but_newest() {
  static_assert(LEFT < 16);
  __builtin_amdgcn_s_waitcnt(0x0F70 | LEFT);
  asm volatile("" ::: "memory");
}

// 2^(reference - maximum).  A part without a key has the reference -inf and counts 0 times its sum of 0; so has a part whose
// logits are NaN (a maximum passes over them), and its NaN has to reach the row's sum.  A row without any finite logit
// has the maximum -inf and a sum of 0 or NaN: its weights come out NaN, as a softmax gives.
__device__ inline float against_max(float reference, float maximum) {
  return reference == maximum ? 1.f : __builtin_amdgcn_exp2f(reference - maximum);
}

template <int D, int ROW_TILES>
constexpr int strip_lds_bytes() {
  typedef StripGeo<D> T;
  return ROW_TILES * T::kTile + kStripWaves * 2 * T::kTile + kStripWaves * ROW_TILES * 32 * 8;
}

// ROW_TILES: 32-row tiles per strip; TPW: key tiles a wave can hold (n <= 8 * TPW * 32).  smem: strip_lds_bytes.
// Kernels cannot share an instance (the compiler's host pass accepts a body with LDS-direct loads once): KERNEL tells those of
// a translation unit apart.  Returns the unit.
// SHARED: the columns of several strips are read in the same launch: their stores write through to where every XCD finds them.
template <int D, int ROW_TILES, int TPW, int KERNEL = 0, bool SHARED = false>
__device__ __forceinline__ int strip_score_body(const StripArgs& a, int block, char* smem) {
  typedef StripGeo<D> T;
  constexpr int kStripRows = 32 * ROW_TILES;
  // query operands stay in registers where the weights leave room
  constexpr bool kKeepQ = ROW_TILES * TPW * 16 + ROW_TILES * T::kKk * 4 <= 128;
  char* const q_s = smem;                       // [ROW_TILES] tiles
  char* const k_s = smem + ROW_TILES * T::kTile;  // [waves][2] tiles
  float2* const stats_s = reinterpret_cast<float2*>(k_s + kStripWaves * 2 * T::kTile);  // [waves][ROW_TILES][32]

  const int tid = threadIdx.x, lane = tid % 64;
  const int wu = __builtin_amdgcn_readfirstlane(tid / 64);
  const int col = lane % 32, grp = lane / 32;
  // Workgroups go to the 8 XCDs round-robin by their linear id.  Remap so that the strips of one
  // (document, layer, KV head), which stream the same keys, are neighbours on ONE XCD and share its L2.
  const int logical = a.per_xcd > 0 ? (block % kXcds) * a.per_xcd + block / kXcds : block;
  const int unit = a.per_unit.quotient(logical), strip = logical - unit * a.strips;
  const int bl = a.kv_heads.quotient(unit), g = unit - bl * a.Hkv;
  const int b = a.layers.quotient(bl), l = bl - b * a.L;
  const int n_c = a.ks.n_c, n = n_c + a.ks.c;
  const int tiles = (n + kStripKeys - 1) / kStripKeys;
  const int total_rows = a.G * a.rows;  // instruction rows of the KV group, flattened (head, row)

  // ---- global -> LDS staging of one 32-key tile by ONE wave ----
  const int k_ss_cache = static_cast<int>(a.ks.cache.ss), k_ss_chunk = static_cast<int>(a.ks.chunk.ss);
  auto seg_bytes = [](int rows_, int ss_) { return rows_ > 0 ? ((rows_ - 1) * ss_ + D) * 2 : 0; };
  const __amdgpu_buffer_rsrc_t k_rs_cache = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(unit_ptr(a.ks.cache, b, l, g)), 0, seg_bytes(n_c, k_ss_cache), kBufferFlags);
  const __amdgpu_buffer_rsrc_t k_rs_chunk = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(unit_ptr(a.ks.chunk, b, l, g)), 0, seg_bytes(a.ks.c, k_ss_chunk), kBufferFlags);
  typedef __attribute__((address_space(3))) void* lds_void_ptr;
  typedef __attribute__((address_space(3))) char* lds_char_ptr;
  char* const wave_lds = k_s + wu * 2 * T::kTile;
  const int fill_row = lane / T::kSegs;  // row inside the group of one instruction
  const int fill_seg = ((lane % T::kSegs) ^ Geo<D>::swz(fill_row)) * 16;
  auto fill_tile = [&](int tile, int buf) {
    const int j0 = tile * kStripKeys;
    char* k_t = wave_lds + buf * T::kTile;
    const bool in_cache = j0 + kStripKeys <= n_c;             // wave-uniform: every row is a cache row
    const bool in_chunk = j0 >= n_c && j0 + kStripKeys <= n;  // wave-uniform: every row is a chunk row
    if (in_cache || in_chunk) {  // one resource, scalar row offsets
      const __amdgpu_buffer_rsrc_t rs = in_cache ? k_rs_cache : k_rs_chunk;
      const int ss2 = (in_cache ? k_ss_cache : k_ss_chunk) * 2;
      const int r0 = in_cache ? j0 : j0 - n_c;
      const int row_off = fill_row * ss2;
#pragma unroll
      for (int i = 0; i < T::kLoads; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_ptr)(k_t + T::kR * i * T::kRowBytes), 16,
                                                 row_off + (fill_seg ^ (Geo<D>::swz(T::kR * i) * 16)), (r0 + T::kR * i) * ss2, 0, 0);
    } else {
      // The tile holds the cache / chunk boundary or the end of the candidates (rows past the end re-read
      // the last row: finite values, masked in the logits).  Two separately predicated loads, each with
      // ONE buffer resource: a resource chosen per lane would be loaded in a serialising loop.  Such a
      // tile takes up to twice the load instructions; the wait in the key loop counts a plain newest tile, so
      // behind such a tile it waits for more than it needs, never for less.
#pragma unroll
      for (int i = 0; i < T::kLoads; ++i) {
        const int seg = fill_seg ^ (Geo<D>::swz(T::kR * i) * 16);
        lds_void_ptr kd = (lds_void_ptr)(k_t + T::kR * i * T::kRowBytes);
        const int j = min(j0 + T::kR * i + fill_row, n - 1);
        if (j < n_c) __builtin_amdgcn_raw_ptr_buffer_load_lds(k_rs_cache, kd, 16, j * k_ss_cache * 2 + seg, 0, 0, 0);
        no_memory_motion();
        if (j >= n_c)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(k_rs_chunk, kd, 16, (j - n_c) * k_ss_chunk * 2 + seg, 0, 0, 0);
        no_memory_motion();
      }
    }
  };

  // ---- the strip's instruction rows, then the wave's first two key tiles ----
  // Flattened row fl = strip * kStripRows + r is row fl % rows of head fl / rows of the group; rows past the
  // end repeat the last one and are given weight 0 at the end.
  const __amdgpu_buffer_rsrc_t q_rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(unit_ptr(a.q, b, l, g * a.G)), 0,
      static_cast<int>(((a.G - 1) * a.q.sh + (a.rows - 1) * a.q.ss + D) * 2), kBufferFlags);
  {
    constexpr int kQInstr = kStripRows / T::kR;  // load instructions for the strip
#pragma unroll
    for (int x = 0; x < (kQInstr + kStripWaves - 1) / kStripWaves; ++x) {
      const int i = wu + kStripWaves * x;  // wave-uniform
      if (i < kQInstr) {
        const int r = T::kR * i + fill_row;
        const int fl = min(strip * kStripRows + r, total_rows - 1);
        const int hh = a.head_rows.quotient(fl), t = fl - hh * a.rows;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(q_rs, (lds_void_ptr)(q_s + T::kR * i * T::kRowBytes), 16,
                                                 (hh * static_cast<int>(a.q.sh) + t * static_cast<int>(a.q.ss)) * 2 +
                                                     ((lane % T::kSegs) ^ Geo<D>::swz(r)) * 16,
                                                 0, 0, 0);
      }
    }
  }
  if (wu < tiles) fill_tile(wu, 0);
  if (wu + kStripWaves < tiles) {
    fill_tile(wu + kStripWaves, 1);
    wait_all_but_newest<T::kLoads>();
  } else {
    wait_all_but_newest<0>();
  }
  __builtin_amdgcn_s_barrier();  // every wave's part of the strip has landed (each wave has waited for its own)
  no_memory_motion();

  // Operands of a tile's 32 rows: lane's row col, segment 2 kk + grp, at position segment ^ swz(col) of the row.  The tile
  // begins at a multiple of a row, so the address of segment 2 kk is that of segment 0 with 32 kk exclusive-ored.
  const uint32_t op_off = col * T::kRowBytes + (grp ^ Geo<D>::swz(col)) * 16;
  auto read_half = [&](bf16x8* op, const char* tile, int half) {
    const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_char_ptr)tile)) + op_off;
    uint32_t addr[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) addr[x] = at ^ (32 * (4 * half + x));
    lds_read_four(op, addr);
  };
  auto read_tile = [&](bf16x8 (&op)[T::kKk], const char* tile) {
#pragma unroll
    for (int half = 0; half < T::kKk / 4; ++half) read_half(op + 4 * half, tile, half);
  };
  // Q^T operands: row (32 rt + col) of the strip, head_dim 16 kk + 8 grp .. + 7
  bf16x8 q_op[ROW_TILES][T::kKk];  // used where kKeepQ
  if constexpr (kKeepQ) {
#pragma unroll
    for (int rt = 0; rt < ROW_TILES; ++rt) read_tile(q_op[rt], q_s + rt * T::kTile);
  }

  // ---- the key loop: un-normalised weights of the wave's tiles, kept in registers in f32 ----
  float e[TPW][ROW_TILES][16];  // of key slot x (key 8 (x / 4) + 4 grp + (x % 4) of the tile) and the lane's row
  float ref[TPW][ROW_TILES];    // the reference the weights of a tile were taken against (log2 domain)
  float m_run[ROW_TILES], l_run[ROW_TILES];
#pragma unroll
  for (int rt = 0; rt < ROW_TILES; ++rt) {
    m_run[rt] = -INFINITY;
    l_run[rt] = 0.f;
  }
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int kt = wu + kStripWaves * i;  // wave-uniform
#pragma unroll
    for (int rt = 0; rt < ROW_TILES; ++rt) ref[i][rt] = -INFINITY;
    if (kt >= tiles) continue;
    // tile i + 1 was requested behind it, if there is one
    if (i + 1 < TPW && kt + kStripWaves < tiles)
      wait_all_but_newest<T::kLoads>();
    else
      wait_all_but_newest<0>();
    bf16x8 ka[T::kKk];
    read_tile(ka, wave_lds + (i & 1) * T::kTile);
    if (i + 2 < TPW && kt + 2 * kStripWaves < tiles) fill_tile(kt + 2 * kStripWaves, i & 1);  // the operands are in registers
    const int valid = n - kStripKeys * kt;  // keys of the tile that exist (wave-uniform)
#pragma unroll
    for (int rt = 0; rt < ROW_TILES; ++rt) {
      f32x16 s;
#pragma unroll
      for (int x = 0; x < 16; ++x) s[x] = 0.f;
#pragma unroll
      for (int half = 0; half < T::kKk / 4; ++half) {
        bf16x8 qh[4];
        if constexpr (!kKeepQ) read_half(qh, q_s + rt * T::kTile, half);
#pragma unroll
        for (int x = 0; x < 4; ++x)
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[4 * half + x], kKeepQ ? q_op[rt][4 * half + x] : qh[x], s, 0, 0, 0);
      }
      if (valid < kStripKeys) {
#pragma unroll
        for (int x = 0; x < 16; ++x)
          if (8 * (x / 4) + 4 * grp + (x % 4) >= valid) s[x] = -INFINITY;
      }
      float mx = s[0];
#pragma unroll
      for (int x = 1; x < 16; ++x) mx = __builtin_fmaxf(mx, s[x]);
      mx *= a.c2;
      // Lazy reference, one per row (the two lanes of a row see different keys of the tile and share it): it
      // only has to stay within kMaxSlack of the row's running maximum, so the exchange with the other lane
      // happens in the rare branch alone.
      if (__any(mx > m_run[rt] + kMaxSlack)) {  // wave-uniform; rare after the first tile
        const float mxr = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if (mxr > m_run[rt] + kMaxSlack) {
          l_run[rt] *= __builtin_amdgcn_exp2f(m_run[rt] - mxr);  // 0 when nothing was seen before
          m_run[rt] = mxr;
        }
      }
      const float m_sub = m_run[rt] == -INFINITY ? 0.f : m_run[rt];  // a row whose keys are all masked so far
      ref[i][rt] = m_run[rt];
      float psum[2] = {0.f, 0.f};
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        e[i][rt][x] = __builtin_amdgcn_exp2f(fmaf(s[x], a.c2, -m_sub));
        psum[x % 2] += e[i][rt][x];
      }
      l_run[rt] += psum[0] + psum[1];
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- row normalisers: the (reference, sum) pairs of the eight waves ----
#pragma unroll
  for (int rt = 0; rt < ROW_TILES; ++rt) {
    const float l_row = l_run[rt] + __shfl_xor(l_run[rt], 32, 64);
    if (grp == 0) stats_s[(wu * ROW_TILES + rt) * 32 + col] = make_float2(m_run[rt], l_row);
  }
  __syncthreads();
  float m_row[ROW_TILES], inv_row[ROW_TILES];
#pragma unroll
  for (int rt = 0; rt < ROW_TILES; ++rt) {
    float2 ps[kStripWaves];
#pragma unroll
    for (int x = 0; x < kStripWaves; ++x) ps[x] = stats_s[(x * ROW_TILES + rt) * 32 + col];
    float mm = -INFINITY;
#pragma unroll
    for (int x = 0; x < kStripWaves; ++x) mm = fmaxf(mm, ps[x].x);
    float lsum = 0.f;
#pragma unroll
    for (int x = 0; x < kStripWaves; ++x)  // fixed order: every lane of the row gets the same bits
      lsum += ps[x].y * against_max(ps[x].x, mm);
    m_row[rt] = mm;
    const bool real_row = strip * kStripRows + 32 * rt + col < total_rows;
    inv_row[rt] = real_row ? 1.f / lsum : 0.f;  // padding rows carry no weight
  }

  // ---- column sums of the strip: each weight times its row's factor, added over the rows = lanes ----
  float* const dst = a.part + (static_cast<int64_t>(unit) * a.strips + strip) * n;
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int kt = wu + kStripWaves * i;  // wave-uniform
    if (kt >= tiles) continue;
    float v[16];
#pragma unroll
    for (int rt = 0; rt < ROW_TILES; ++rt) {
      const float f = against_max(ref[i][rt], m_row[rt]) * inv_row[rt];
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const float p = e[i][rt][x] * f;
        v[x] = rt == 0 ? p : v[x] + p;
      }
    }
    const float tot = reduce16_over32(v, col);  // value index col / 2 -> key 8 (x / 4) + 4 grp + (x % 4)
    const int x = col >> 1, j = kStripKeys * kt + 8 * (x / 4) + 4 * grp + (x % 4);
    if ((col & 1) == 0 && j < n) {
      if (SHARED && a.strips > 1)
        __hip_atomic_store(dst + j, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        dst[j] = tot;
    }
  }
  return unit;
}

}  // namespace
}  // namespace citrus
