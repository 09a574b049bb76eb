// Attention kernels of the f32 mode (bf16 has its own for every head dimension), on the f64 matrix instructions.  They
// follow the same definitions as the fast path: softmax attention with the 1/sqrt(d_k) scaling of Eq. (1) (Section 4.1
// step 1), and the summed form of Eq. (1) for the importance scores.
//
// Precision.  The mode promises 1e-5 against an f64 reference: with logits of a few tens an f32 dot product and
// subtraction alone leave a relative error of that order in the probability.  So both products are formed and added in
// f64; probabilities, row sums and what leaves a wave are f32.
//
// Layout of v_mfma_f64_16x16x4_f64 (wave64): A holds row l % 16, contraction slot l / 16; B column l % 16, the same slot;
// C/D register i holds row 4 i + l / 16, column l % 16.  S^T = K.Q^T puts one query per lane, and its register i is
// the B operand (P^T) of step i of O^T = V^T.P^T.  A float4 of a row gives four operands: the contraction over head_dim, and
// the rows of O^T, may run in any order.
//
// What bounds it: these launches are small, and a workgroup's time is its chain of dependent steps (memory 1 us, sixteen
// to thirty-two MFMAs of 58 cycles, exchange through LDS).  So the waves of a workgroup share sixteen query rows and split
// the keys.  Against one wavefront per query row on the vector units, keys one by one: 4 heads, 32 rows over 96 states, 8
// instruction rows, head_dim 64: 15.0 + 5 + 7.6 us in three launches, 8.8 in one (a document of 512 tokens 527 -> 235 us);
// documents of 32/8 heads, head_dim 128, 128 rows over 384 states 1599 -> 431 us, 8/1 heads in 16 layers, 512 rows over 1280
// states 11651 -> 2204 us; decoding 8 layers of 32/8 heads, 1000 states, 4 tokens 512 -> 227 us.  Errors against f64 are the
// same or smaller (outputs 9e-8 to 1.2e-7 instead of 1.2e-7 to 7e-7).
#include <algorithm>

#include "citrus_internal.h"
#include "evict_body.h"
#include "lanes.h"

namespace citrus {
namespace {

typedef __attribute__((ext_vector_type(4))) double f64x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWave = 64;
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kWave;
constexpr int kTile = 16;  // query rows of a workgroup; keys of a wave's tile

__device__ inline const float* row_ptr(const View& v, int b, int l, int h, int s) {
  return static_cast<const float*>(v.ptr) + (b * v.sb + l * v.sl + h * v.sh + static_cast<int64_t>(s) * v.ss);
}
// candidate j -> its row in the cache or the chunk segment (both addresses, then the choice)
__device__ inline const float* cand_ptr(const Segments& sg, int b, int l, int g, int j) {
  const float* const in_cache = row_ptr(sg.cache, b, l, g, j);
  const float* const in_chunk = row_ptr(sg.chunk, b, l, g, j - sg.n_c);
  return j < sg.n_c ? in_cache : in_chunk;
}
__device__ inline f64x4 mfma(double a, double b, const f64x4& c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
// exchange over the four lanes of a column
__device__ inline float column_max(float v) {
  float a, b;
  both_of_rows(v, a, b);
  both_of_halves(fmaxf(a, b), a, b);
  return fmaxf(a, b);
}
__device__ inline float column_sum(float v) {
  float a, b;
  both_of_rows(v, a, b);
  both_of_halves(a + b, a, b);
  return a + b;
}

// The lane's part of sixteen rows as an operand: four elements of its row (l % 16) per 16 of head_dim, from 4 (l / 16).
template <int D>
struct Operand {
  f32x4 x[D / 16];
};
template <int D>
__device__ inline void load_operand(Operand<D>& o, const float* row, int lane) {
#pragma unroll
  for (int x = 0; x < D / 16; ++x) o.x[x] = *reinterpret_cast<const f32x4*>(row + 16 * x + 4 * (lane / 16));
}
// logits of sixteen keys x sixteen queries, unscaled; two chains
template <int D>
__device__ inline f64x4 products(const Operand<D>& k, const Operand<D>& q) {
  f64x4 s[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
  for (int x = 0; x < D / 16; ++x)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      s[c % 2] = mfma(static_cast<double>(k.x[x][c]), static_cast<double>(q.x[x][c]), s[c % 2]);
  return s[0] + s[1];
}

struct AttnF32Args {
  Dims dm;
  View q, out;
  int rows, causal;
  Segments ks, vs;
  float* lse;
  int row_blocks;
};

template <int D, int WAVES>
constexpr int attn_f32_lds_bytes() { return WAVES * kTile * (D + 4) * 4 + 2 * WAVES * kTile * 4; }

// Sixteen query rows, block rb of head h in (document, layer) bl.  out and lse are optional.
template <int D, int WAVES>
__device__ __forceinline__ void attn_f32_body(const AttnF32Args& a, int rb, int h, int bl, char* smem) {
  constexpr int kPitch = D + 4, kCols = D / 64;  // float4 columns of O^T per lane
  float* const o_s = reinterpret_cast<float*>(smem);  // [waves][16][kPitch]
  float* const m_s = o_s + WAVES * kTile * kPitch;    // [waves][16]
  float* const l_s = m_s + WAVES * kTile;
  const int tid = threadIdx.x, lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane % 16, quad = lane / 16;
  const int b = bl / a.dm.L, l = bl % a.dm.L, g = h / a.dm.G;
  const int n_c = a.ks.n_c, n = n_c + a.ks.c;
  const int row0 = rb * kTile, t = min(row0 + col, a.rows - 1);  // rows past the end repeat the last one and are not stored
  const int limit = a.causal ? n_c + t : n - 1;                  // last candidate the lane's row sees
  const int first_limit = a.causal ? n_c + row0 : n - 1;         // ... and every row of the block
  const int last_limit = a.causal ? n_c + min(row0 + kTile, a.rows) - 1 : n - 1;
  const int tiles = last_limit / kTile + 1;
  const bool values = a.out.ptr != nullptr;
  const double scale = static_cast<double>(a.dm.scale);

  Operand<D> q;
  load_operand(q, row_ptr(a.q, b, l, h, t), lane);
  float m = -INFINITY, lsum = 0.f;
  f64x4 acc[kCols][4];  // [hh][c], register i: head_dim 64 hh + 16 i + 4 quad + c
#pragma unroll
  for (int hh = 0; hh < kCols; ++hh)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[hh][c] = f64x4{0, 0, 0, 0};

  for (int kt = w; kt < tiles; kt += WAVES) {
    const int j0 = kt * kTile;
    Operand<D> k;
    load_operand(k, cand_ptr(a.ks, b, l, g, min(j0 + col, n - 1)), lane);
    f32x4 v[4][kCols];  // values of keys j0 + 4 i + quad, head_dim 64 hh + 4 col .. + 3
    if (values) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float* const vp = cand_ptr(a.vs, b, l, g, min(j0 + 4 * i + quad, n - 1));
#pragma unroll
        for (int hh = 0; hh < kCols; ++hh) v[i][hh] = *reinterpret_cast<const f32x4*>(vp + 64 * hh + 4 * col);
      }
    }
    f64x4 s = products(k, q);
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] *= scale;
      if (j0 + 4 * i + quad <= limit) mx = fmaxf(mx, static_cast<float>(s[i]));
    }
    // the running maximum is an f32 value; it only has to be the same number wherever it is subtracted
    const float m_new = fmaxf(m, column_max(mx));
    if (__any(m_new != m)) {  // wave-uniform
      const float corr = m_new == m ? 1.f : expf(m - m_new);
      lsum *= corr;
#pragma unroll
      for (int hh = 0; hh < kCols; ++hh)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[hh][c] *= static_cast<double>(corr);
      m = m_new;
    }
    const double m_sub = m == -INFINITY ? 0.0 : static_cast<double>(m);  // a row that has seen nothing yet
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = j0 + 4 * i + quad <= limit ? expf(static_cast<float>(s[i] - m_sub)) : 0.f;
      lsum += p[i];
    }
    if (!values) continue;
    // A value that is not finite must not reach a row that does not see its key, and a product with probability 0 would
    // carry it there.
    bool finite = true;
    if (j0 + kTile - 1 > first_limit) {  // wave-uniform: some row does not see some key of the tile
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int hh = 0; hh < kCols; ++hh)
#pragma unroll
          for (int c = 0; c < 4; ++c) finite = finite && fabsf(v[i][hh][c]) < INFINITY;
      finite = __all(finite);
    }
    if (__builtin_expect(finite, 1)) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int hh = 0; hh < kCols; ++hh)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[hh][c] = mfma(static_cast<double>(v[i][hh][c]), static_cast<double>(p[i]), acc[hh][c]);
    } else {
      for (int key = 0; key < kTile; ++key) {  // one key after the other, to the rows that see it
        float pk = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float pi = __shfl(p[i], col + 16 * (key % 4), kWave);
          pk = key / 4 == i ? pi : pk;
        }
        if (j0 + key > last_limit) break;
        const float* const vp = cand_ptr(a.vs, b, l, g, j0 + key);
#pragma unroll
        for (int hh = 0; hh < kCols; ++hh)
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (j0 + key <= limit)
                acc[hh][c][i] = fma(static_cast<double>(pk), static_cast<double>(vp[64 * hh + 16 * i + 4 * quad + c]), acc[hh][c][i]);
      }
    }
  }

  lsum = column_sum(lsum);
  if (quad == 0) {
    m_s[w * kTile + col] = m;
    l_s[w * kTile + col] = lsum;
  }
  if (values) {
#pragma unroll
    for (int hh = 0; hh < kCols; ++hh)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4*>(o_s + (w * kTile + col) * kPitch + 64 * hh + 16 * i + 4 * quad) =
            f32x4{static_cast<float>(acc[hh][0][i]), static_cast<float>(acc[hh][1][i]), static_cast<float>(acc[hh][2][i]),
                  static_cast<float>(acc[hh][3][i])};
  }
  __syncthreads();
  // query row r, four elements of its output; the waves' parts in a fixed order
  for (int x = tid; x < kTile * (D / 4); x += WAVES * kWave) {
    const int r = x / (D / 4), e = x % (D / 4) * 4;
    if (row0 + r >= a.rows) break;
    float mw[WAVES], mm = -INFINITY;
#pragma unroll
    for (int y = 0; y < WAVES; ++y) {
      mw[y] = m_s[y * kTile + r];
      mm = fmaxf(mm, mw[y]);
    }
    float sum = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int y = 0; y < WAVES; ++y) {
      // A wave without a key the row sees adds 0 * 0.  So does one whose logits are all -inf, and one whose logits are NaN
      // (which a maximum passes over) adds its NaN: no part is left out.
      const float f = expf(mw[y] - mm);
      sum += l_s[y * kTile + r] * f;
      if (values) o += *reinterpret_cast<const f32x4*>(o_s + (y * kTile + r) * kPitch + e) * f;
    }
    if (values) {
      const float inv = 1.f / sum;
      *reinterpret_cast<f32x4*>(const_cast<float*>(row_ptr(a.out, b, l, h, row0 + r)) + e) = o * inv;
    }
    if (a.lse != nullptr && e == 0) a.lse[(static_cast<int64_t>(bl) * a.dm.Hq + h) * a.rows + row0 + r] = mm + logf(sum);
  }
}

template <int D, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void attn_f32_kernel(AttnF32Args a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  attn_f32_body<D, WAVES>(a, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}
// The same where every wave can have a SIMD to itself, as one that takes more than half of a SIMD's registers has: two workgroups
// of two waves on a compute unit came to lie on two of its four SIMDs.  us, shared | apart: 128 heads, 55 rows over 93 states 33.5 | 24.5.
template <int D, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void attn_f32_apart_kernel(AttnF32Args a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  asm volatile("" ::: "a31");
  attn_f32_body<D, WAVES>(a, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}

// Column sums: score[g, j] = sum over the query rows of the KV group of exp(s - lse).  A workgroup owns two tiles of sixteen
// keys; four waves per tile split the rows (head after head, flattened), whose sums meet in LDS in a fixed order.
constexpr int kColsumKeyTiles = 2, kColsumSplits = kWaves / kColsumKeyTiles;
template <int D>
__global__ __launch_bounds__(kThreads) void colsum_f32_kernel(Dims dm, View q, int rows, Segments ks, int causal,
                                                              const float* lse, float* score) {
  __shared__ float part[kWaves][kTile];
  const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int col = lane % 16, quad = lane / 16;
  const int g = blockIdx.y, b = blockIdx.z / dm.L, l = blockIdx.z % dm.L;
  const int n_c = ks.n_c, n = n_c + ks.c;
  const int j0 = (blockIdx.x * kColsumKeyTiles + w / kColsumSplits) * kTile, split = w % kColsumSplits;
  const int total = dm.G * rows, row_tiles = (total + kTile - 1) / kTile;
  const double scale = static_cast<double>(dm.scale);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (j0 < n) {  // wave-uniform
    Operand<D> k;
    load_operand(k, cand_ptr(ks, b, l, g, min(j0 + col, n - 1)), lane);
    auto row_of = [&](int rt, int& t) {  // flattened row rt * 16 + col: row t of a head; rows past the end repeat the last
      const int r = min(rt * kTile + col, total - 1), hh = r / rows;
      t = r - hh * rows;
      return g * dm.G + hh;
    };
    Operand<D> q_next;
    float lse_next = 0.f;
    int t_next = 0;
    auto request = [&](int rt) {
      const int h = row_of(min(rt, row_tiles - 1), t_next);
      load_operand(q_next, row_ptr(q, b, l, h, t_next), lane);
      lse_next = lse[(static_cast<int64_t>(blockIdx.z) * dm.Hq + h) * rows + t_next];
    };
    request(split);
    for (int rt = split; rt < row_tiles; rt += kColsumSplits) {
      const Operand<D> qo = q_next;
      const double norm = static_cast<double>(lse_next);
      const int t = t_next;
      request(rt + kColsumSplits);
      const f64x4 s = products(k, qo);
      const int limit = rt * kTile + col >= total ? -1 : causal ? n_c + t : n - 1;  // a row past the end sees nothing
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = expf(static_cast<float>(s[i] * scale - norm));
        acc[i] += j0 + 4 * i + quad <= limit ? p : 0.f;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // over the sixteen rows of a tile = lanes of a quad
    acc[i] = row_sum(acc[i]);
    if (col == 0) part[w][4 * i + quad] = acc[i];
  }
  __syncthreads();
  if (threadIdx.x < kColsumKeyTiles * kTile) {
    const int kt = threadIdx.x / kTile, x = threadIdx.x % kTile;
    const int j = (blockIdx.x * kColsumKeyTiles + kt) * kTile + x;
    float v = part[kt * kColsumSplits][x];
#pragma unroll
    for (int y = 1; y < kColsumSplits; ++y) v += part[kt * kColsumSplits + y][x];
    if (j < n) score[(static_cast<int64_t>(blockIdx.z) * dm.Hkv + g) * n + j] = v;
  }
}

// Instruction score of a KV group whose logits fit the registers of a workgroup (512 keys; 64 rows, at head_dim 128 32): products once,
// normalisers through LDS, column sums (to out).  No mask.
struct ScoreF32Args {
  Dims dm;
  View q;
  int rows;
  Segments ks;
  float* score;
};
constexpr int kScoreKeyTiles = 4;  // key tiles of a wave
template <int D>
constexpr int score_row_tiles() { return 256 / D; }
bool score_f32_fits(const Dims& dm, int rows, int n) {
  const int row_tiles = dm.D == 64 ? score_row_tiles<64>() : score_row_tiles<128>();
  return static_cast<int64_t>(dm.G) * rows <= row_tiles * kTile && n <= kScoreKeyTiles * kWaves * kTile;
}
constexpr int kScoreF32LdsBytes = kWaves * score_row_tiles<64>() * kTile * 8;

template <int D>
__device__ __forceinline__ void score_f32_body(const ScoreF32Args& a, int g, int bl, char* smem, float* out) {
  constexpr int kScoreRowTiles = score_row_tiles<D>();
  float2* const stats = reinterpret_cast<float2*>(smem);  // [waves][row tiles][16]: maximum, sum
  const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int col = lane % 16, quad = lane / 16;
  const int b = bl / a.dm.L, l = bl % a.dm.L;
  const int n = a.ks.n_c + a.ks.c;
  const int total = a.dm.G * a.rows, row_tiles = (total + kTile - 1) / kTile;
  const double scale = static_cast<double>(a.dm.scale);
  Operand<D> q[kScoreRowTiles];
#pragma unroll
  for (int rt = 0; rt < kScoreRowTiles; ++rt) {
    if (rt >= row_tiles) break;  // uniform
    const int r = min(rt * kTile + col, total - 1), hh = r / a.rows;
    load_operand(q[rt], row_ptr(a.q, b, l, g * a.dm.G + hh, r - hh * a.rows), lane);
  }
  f64x4 s[kScoreKeyTiles][kScoreRowTiles];
  float m[kScoreRowTiles];
#pragma unroll
  for (int rt = 0; rt < kScoreRowTiles; ++rt) m[rt] = -INFINITY;
#pragma unroll
  for (int i = 0; i < kScoreKeyTiles; ++i) {
    const int j0 = (w + kWaves * i) * kTile;
    if (j0 >= n) break;  // wave-uniform
    Operand<D> k;
    load_operand(k, cand_ptr(a.ks, b, l, g, min(j0 + col, n - 1)), lane);
#pragma unroll
    for (int rt = 0; rt < kScoreRowTiles; ++rt) {
      if (rt >= row_tiles) break;
      s[i][rt] = products(k, q[rt]);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        s[i][rt][x] *= scale;
        if (j0 + 4 * x + quad < n) m[rt] = fmaxf(m[rt], static_cast<float>(s[i][rt][x]));
      }
    }
  }
  auto sum_over_keys = [&](int rt, double base) {  // of exp(s - base) over the wave's keys of the lane's row
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < kScoreKeyTiles; ++i) {
      const int j0 = (w + kWaves * i) * kTile;
      if (j0 >= n) break;
#pragma unroll
      for (int x = 0; x < 4; ++x)
        v += j0 + 4 * x + quad < n ? expf(static_cast<float>(s[i][rt][x] - base)) : 0.f;
    }
    return column_sum(v);
  };
#pragma unroll
  for (int rt = 0; rt < kScoreRowTiles; ++rt) {
    if (rt >= row_tiles) break;
    const float mr = column_max(m[rt]);
    const float lr = sum_over_keys(rt, mr == -INFINITY ? 0.0 : static_cast<double>(mr));
    if (quad == 0) stats[(w * kScoreRowTiles + rt) * kTile + col] = make_float2(mr, lr);
  }
  __syncthreads();
  float acc[kScoreKeyTiles][4];
#pragma unroll
  for (int i = 0; i < kScoreKeyTiles; ++i)
#pragma unroll
    for (int x = 0; x < 4; ++x) acc[i][x] = 0.f;
#pragma unroll
  for (int rt = 0; rt < kScoreRowTiles; ++rt) {
    if (rt >= row_tiles) break;
    float2 ps[kWaves];
    float mm = -INFINITY, lsum = 0.f;
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      ps[x] = stats[(x * kScoreRowTiles + rt) * kTile + col];
      mm = fmaxf(mm, ps[x].x);
    }
#pragma unroll
    for (int x = 0; x < kWaves; ++x) lsum += ps[x].y * expf(ps[x].x - mm);  // a wave's NaN is not left out, as in attn_f32_body
    const double norm = static_cast<double>(mm + logf(lsum));
    const bool real_row = rt * kTile + col < total;
#pragma unroll
    for (int i = 0; i < kScoreKeyTiles; ++i) {
      if ((w + kWaves * i) * kTile >= n) break;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const float p = expf(static_cast<float>(s[i][rt][x] - norm));
        acc[i][x] += real_row ? p : 0.f;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kScoreKeyTiles; ++i) {
    const int j0 = (w + kWaves * i) * kTile;
    if (j0 >= n) break;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const float v = row_sum(acc[i][x]);
      const int j = j0 + 4 * x + quad;
      if (col == 0 && j < n) out[j] = v;
    }
  }
}

template <int D>
__global__ __launch_bounds__(kThreads) void score_f32_kernel(ScoreF32Args a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  score_f32_body<D>(a, blockIdx.x, blockIdx.y, smem,
                    a.score + (static_cast<int64_t>(blockIdx.y) * a.dm.Hkv + blockIdx.x) * (a.ks.n_c + a.ks.c));
}
// A step's attention and instruction score in one launch; neither reads what the other writes.  A unit's scores come from one
// workgroup, which then evicts the unit as well (the rows go to the other buffer, which nothing here reads): behind the
// attention's chain both disappear.  4 heads, 32 rows over 96 states, 8 instruction
// rows, head_dim 64: 13.8 us a step in two launches, 13.0 in one; 12.7 of them the score's workgroup.
constexpr int kTailRows = 8;  // rows of a thread in flight
constexpr int kTailScores = std::max<int>(kScoreF32LdsBytes, sizeof(SelectLds<1, kThreads, 8>) + kThreads * sizeof(int32_t));
template <int D>
__global__ __launch_bounds__(kThreads) void attn_score_f32_kernel(AttnF32Args a, ScoreF32Args s, int score_blocks, StepTail t) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  typedef SelectLds<1, kThreads, 8> Lds;  // 512 candidates
  static_assert(kScoreKeyTiles * kWaves * kTile <= kThreads);
  int block = blockIdx.x;
  if (block < score_blocks) {
    Lds& lds = *reinterpret_cast<Lds*>(smem);
    int32_t* const sel = reinterpret_cast<int32_t*>(smem + sizeof(Lds));
    float* const scores = reinterpret_cast<float*>(smem + kTailScores);  // what the selection reads does not leave the workgroup
    int unit = block, r0 = 0;
    if (t.then == Then::kGather) {
      unit = block / t.job.parts;
      r0 = (block - unit * t.job.parts) * t.job.part_rows;
    } else {
      const int g = block % s.dm.Hkv, bl = block / s.dm.Hkv, n = s.ks.n_c + s.ks.c;
      score_f32_body<D>(s, g, bl, smem, scores);
      __syncthreads();
      if (t.then == Then::kNothing) {
        if (static_cast<int>(threadIdx.x) < n) s.score[static_cast<int64_t>(block) * n + threadIdx.x] = scores[threadIdx.x];
        return;
      }
    }
    evict_rows<1, kThreads, 8, Scores::kOneHead, kTailRows>(t.job, unit, scores, r0, min(r0 + t.job.part_rows, t.job.rows), lds, sel);
  } else {
    block -= score_blocks;
    const int hb = block / a.row_blocks;
    attn_f32_body<D, kWaves>(a, block % a.row_blocks, hb % a.dm.Hq, hb / a.dm.Hq, smem);
  }
}

AttnF32Args attn_f32_args(const Dims& dm, const View& q, int rows, const Segments& ks, const Segments& vs, int causal,
                          const View& out, float* lse) {
  return AttnF32Args{dm, q, out, rows, causal, ks, vs, lse, (rows + kTile - 1) / kTile};
}
// A grid's dimension has less than 2^32 work-items: one of workgroups x heads x layers has more dimensions than one.
dim3 attn_f32_grid(const AttnF32Args& a) { return dim3(a.row_blocks, a.dm.Hq, a.dm.B * a.dm.L); }
int64_t attn_f32_blocks(const Dims& dm, int rows) { return static_cast<int64_t>((rows + kTile - 1) / kTile) * dm.Hq * dm.B * dm.L; }

// Waves of a workgroup, which split the keys of its sixteen rows.  Eight while two workgroups of eight to a compute unit have room
// for all of them: the chain over the keys is the time.  In larger launches the other workgroups fill the chip, and
// waves that have few keys or none, their LDS and the exchange at the end are what is left of it.  us with one | two | four |
// eight waves (and with one wave on the vector units per row), one row per head, workgroups in brackets.  head_dim 64, 6
// states 7.5 | 7.8 | 11.0 | 18.0 (8.9) (1024), 23 | 35 | 49 | 117 (35) (8192); 65 states 15.1 | 14.6 | 11.8 | 15.6 (12.2) (512), 17.5 |
// 16.5 | 18.0 | 28.4 (14.6) (1024), 27.8 | 32.4 | 30.9 | 53.5 (27.8) (2048); 1001 states 134 | 111 | 65 | 71 (97) (512), 244 | 258 |
// 210 | 256 (224) (2048).  head_dim 128, 65 states 22 | 17 | 22 | 23 (18) (512), 40 | 55 | 78 | 79 (48) (2048); 1001 states 200 |
// 113 | 116 | 111 (129) (512), 380 | 446 | 463 | 423 (440) (2048); 3001 states 752 | 651 |
// 659 | 601 (837) (1024); 128 rows over 384 states 547 | 665 | 736 | 721 (8192).
int attn_f32_waves(const Dims& dm, int rows, int n) {
  const int64_t blocks = attn_f32_blocks(dm, rows);
  const int cus = compute_units(), tiles = (n + kTile - 1) / kTile;
  if (blocks < 2 * cus) return kWaves;
  if (dm.D == 64) return tiles <= 2 || blocks >= 16 * cus || (tiles <= 8 && blocks >= 4 * cus) ? 1 : 4;
  return tiles <= 1 || blocks >= 8 * cus ? 1 : tiles > 48 ? kWaves : 2;
}

template <int D, int WAVES, bool APART = false>
hipError_t attn_f32_launch(const AttnF32Args& a, hipStream_t st) {
  constexpr int kLdsBytes = attn_f32_lds_bytes<D, WAVES>();
  auto kern = [] {
    if constexpr (APART)
      return attn_f32_apart_kernel<D, WAVES>;
    else
      return attn_f32_kernel<D, WAVES>;
  }();
  static LdsLimit limit;
  const hipError_t e = raise_lds_limit(limit, reinterpret_cast<const void*>(kern), kLdsBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, attn_f32_grid(a), dim3(WAVES * kWave), kLdsBytes, st, a);
  return hipGetLastError();
}

template <int D>
hipError_t attn_score_f32_launch(const AttnF32Args& a, const ScoreF32Args& s, const Eviction* evict, hipStream_t st) {
  constexpr int kLdsBytes = std::max(attn_f32_lds_bytes<D, kWaves>(), kScoreF32LdsBytes);
  static_assert(kTailScores + kThreads * sizeof(float) <= kLdsBytes);
  static LdsLimit limit;
  const hipError_t e = raise_lds_limit(limit, reinterpret_cast<const void*>(attn_score_f32_kernel<D>), kLdsBytes);
  if (e != hipSuccess) return e;
  const int units = s.dm.B * s.dm.L * s.dm.Hkv, attn_blocks = static_cast<int>(attn_f32_blocks(a.dm, a.rows));
  StepTail t;
  t.then = Then::kNothing;
  if (evict != nullptr) {
    t.job = evict_job(sizeof(float), s.dm, *evict);
    t.then = gather_only(*evict) ? Then::kGather : Then::kEvict;
    if (t.then == Then::kGather) cut_in_parts(t.job, 32, (2 * compute_units() - attn_blocks) / units);
  }
  const int score_blocks = t.then == Then::kGather ? units * t.job.parts : units;
  hipLaunchKernelGGL(attn_score_f32_kernel<D>, dim3(score_blocks + attn_blocks), dim3(kThreads), kLdsBytes, st, a, s, score_blocks, t);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(const Dims& dm, View q, int rows, Segments ks, Segments vs, int causal, View out, float* lse,
                           hipStream_t st) {
  const AttnF32Args a = attn_f32_args(dm, q, rows, ks, vs, causal, out, lse);
  const int waves = attn_f32_waves(dm, rows, ks.n_c + ks.c);
  const bool apart = waves * attn_f32_blocks(dm, rows) <= 4 * compute_units();  // four SIMDs
  auto launch = waves == 8 ? attn_f32_launch<128, 8> : waves == 1 ? attn_f32_launch<128, 1> : apart ? attn_f32_launch<128, 2, true> : attn_f32_launch<128, 2>;
  if (dm.D == 64) launch = waves == 8 ? attn_f32_launch<64, 8> : waves == 4 ? attn_f32_launch<64, 4> : attn_f32_launch<64, 1>;
  return launch(a, st);
}

hipError_t launch_colsum_f32(const Dims& dm, View q, int rows, Segments ks, int causal, const float* lse, float* score,
                             hipStream_t st) {
  const int n = ks.n_c + ks.c, keys = kColsumKeyTiles * kTile;
  const auto kern = dm.D == 64 ? colsum_f32_kernel<64> : colsum_f32_kernel<128>;
  hipLaunchKernelGGL(kern, dim3((n + keys - 1) / keys, dm.Hkv, dm.B * dm.L), dim3(kThreads), 0, st, dm, q, rows, ks, causal,
                     lse, score);
  return hipGetLastError();
}

hipError_t launch_instr_score_f32(const Dims& dm, View q, int rows, Segments ks, float* lse_scratch, float* score, hipStream_t st) {
  if (score_f32_fits(dm, rows, ks.n_c + ks.c)) {
    const ScoreF32Args a{dm, q, rows, ks, score};
    const auto kern = dm.D == 64 ? score_f32_kernel<64> : score_f32_kernel<128>;
    hipLaunchKernelGGL(kern, dim3(dm.Hkv, dm.B * dm.L), dim3(kThreads), kScoreF32LdsBytes, st, a);
    return hipGetLastError();
  }
  // pass 1: row normalisers (log-sum-exp over all candidates, no mask); pass 2: probabilities summed down the rows of each KV group
  const View none{nullptr, 0, 0, 0, 0};
  const hipError_t e = launch_attn_f32(dm, q, rows, ks, ks, /*causal=*/0, none, lse_scratch, st);
  return e != hipSuccess ? e : launch_colsum_f32(dm, q, rows, ks, /*causal=*/0, lse_scratch, score, st);
}

// One workgroup moves a unit's rows: from 128 KB on the launch that shares them out is faster.  us a step apart | one launch,
// bytes kept: 57 KB 16.1 | 15.2, 123 KB 25.8 | 25.3, 227 KB 26.7 | 28.5, 251 KB 30.3 | 32.1.
bool step_f32_in_one_launch(const Dims& dm, const Eviction& e) {
  return gather_only(e) || 2 * static_cast<int64_t>(std::min(e.n, e.k)) * dm.D * static_cast<int>(sizeof(float)) <= 128 << 10;
}

bool attn_score_f32_in_one_launch(const Dims& dm, int rows, int instr_rows, int n) {
  return score_f32_fits(dm, instr_rows, n) && attn_f32_waves(dm, rows, n) == kWaves;  // the score's workgroups have eight
}

hipError_t launch_attn_score_f32(const Dims& dm, View q, Segments ks, Segments vs, View out, View q_instr, int instr_rows,
                                 float* score, const Eviction* evict, hipStream_t st) {
  const AttnF32Args a = attn_f32_args(dm, q, ks.c, ks, vs, /*causal=*/1, out, nullptr);
  const ScoreF32Args s{dm, q_instr, instr_rows, ks, score};
  return dm.D == 64 ? attn_score_f32_launch<64>(a, s, evict, st) : attn_score_f32_launch<128>(a, s, evict, st);
}

}  // namespace citrus
