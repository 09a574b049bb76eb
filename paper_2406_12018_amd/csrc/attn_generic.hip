// Vector-ALU attention kernels of the f32 mode (bf16 runs on the matrix-core kernels for every head
// dimension).  They follow the same definitions as the fast path: softmax attention with the 1/sqrt(d_k) scaling
// of Eq. (1) (Section 4.1 step 1), and the summed form of Eq. (1) for the
// importance scores.
#include "citrus_internal.h"

namespace citrus {
namespace {

constexpr int kWave = 64;
constexpr int kRowsPerBlock = 4;  // one wavefront per query row

// The type the q.k products are accumulated and the maximum / normaliser subtracted in.  The f32
// mode promises 1e-5 against an f64 reference: with logits of a few tens an f32 dot product and subtraction
// alone leave a relative error of that order in the probability.
typedef double Logit;

constexpr int kVec = 4;  // elements per 16-byte load
__device__ inline void load16(const float* p, float* dst) {
  float4 v = *reinterpret_cast<const float4*>(p);
  dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
}
__device__ inline const float* row_ptr(const View& v, int b, int l, int h, int s) {
  return static_cast<const float*>(v.ptr) + (b * v.sb + l * v.sl + h * v.sh + static_cast<int64_t>(s) * v.ss);
}

// candidate j -> its row in the cache or the chunk segment
__device__ inline const float* cand_ptr(const Segments& sg, int b, int l, int g, int j) {
  return j < sg.n_c ? row_ptr(sg.cache, b, l, g, j) : row_ptr(sg.chunk, b, l, g, j - sg.n_c);
}

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// One wavefront per query row; lanes split the keys of a 64-key tile for the
// logits and split head_dim for the output accumulation.
// A launch of the f32 mode has few wavefronts, so a row's chain of dependent loads is its time.  A lane
// requests 256 bytes of its key at once, the value rows come kValueRows at a time, the first of them before
// the logits and the next while one batch is added; the sums keep their order.
// Same bits as one load after the other.  Decoding step, 4 tokens (a workgroup's wavefronts without a row load
// nothing): 8 layers of 32/8 heads, head_dim 128, 1000 states 668 -> 516 us; 2 layers of 8/8 heads, head_dim 64,
// 3000 states 1108 -> 987 us.
constexpr int kValueRows = 16;
template <int D>
__global__ __launch_bounds__(kWave* kRowsPerBlock) void attn_f32_kernel(Dims dm, View q, int rows, Segments ks,
                                                                           Segments vs, int causal, View out,
                                                                           float* lse) {
  __shared__ __attribute__((aligned(16))) Logit q_s[kRowsPerBlock][D];
  __shared__ __attribute__((aligned(16))) float p_s[kRowsPerBlock][kWave];
  const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int h = blockIdx.y, b = blockIdx.z / dm.L, l = blockIdx.z % dm.L, g = h / dm.G;
  const int n = ks.n_c + ks.c;
  const int t_raw = blockIdx.x * kRowsPerBlock + w;
  const bool row_ok = t_raw < rows;
  const int t = row_ok ? t_raw : rows - 1;
  // last visible candidate; a wavefront without a row sees none and loads none
  const int limit = !row_ok ? -1 : causal ? ks.n_c + t : n - 1;
  const int t_blk_last = min(rows - 1, blockIdx.x * kRowsPerBlock + kRowsPerBlock - 1);
  const int blk_limit = causal ? ks.n_c + t_blk_last : n - 1;
  constexpr int E = D / kWave;                   // output dims per lane
  constexpr int kKeyElems = D < 64 ? D : 64;     // elements of a key in flight per lane

  const float* qp = row_ptr(q, b, l, h, t);
  for (int e = lane; e < D; e += kWave) q_s[w][e] = static_cast<Logit>(qp[e]);
  __syncthreads();

  float m = -INFINITY, lsum = 0.f, acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.f;

  // value rows j .. j + kValueRows - 1; those the row does not see repeat the last one it sees and are not added
  auto load_values = [&](int j, float (&v)[kValueRows][E]) {
#pragma unroll
    for (int u = 0; u < kValueRows; ++u) {
      const float* vp = cand_ptr(vs, b, l, g, min(j + u, limit));
#pragma unroll
      for (int e = 0; e < E; ++e) v[u][e] = vp[lane + e * kWave];
    }
  };

  for (int j0 = 0; j0 <= blk_limit; j0 += kWave) {
    const int j = j0 + lane;
    const bool valid = j <= limit;
    float v_now[kValueRows][E];
    if (out.ptr != nullptr && j0 <= limit) load_values(j0, v_now);
    Logit s = -INFINITY;
    if (valid) {
      const float* kp = cand_ptr(ks, b, l, g, j);
      Logit dot = 0;
#pragma unroll
      for (int e0 = 0; e0 < D; e0 += kKeyElems) {
        float kv[kKeyElems];
#pragma unroll
        for (int e = 0; e < kKeyElems; e += kVec) load16(kp + e0 + e, kv + e);
#pragma unroll
        for (int e = 0; e < kKeyElems; ++e) dot = fma(q_s[w][e0 + e], static_cast<Logit>(kv[e]), dot);
      }
      s = dot * static_cast<Logit>(dm.scale);
    }
    // the running maximum is an f32 value; it only has to be the same number wherever it is subtracted
    const float m_new = fmaxf(m, wave_max(static_cast<float>(s)));
    // tile 0 always holds candidate 0, which every row sees, so m_new is finite where there is a row
    const float p = valid ? expf(static_cast<float>(s - static_cast<Logit>(m_new))) : 0.f;
    const float corr = expf(m - m_new);
    lsum = lsum * corr + wave_sum(p);
    m = m_new;
    p_s[w][lane] = p;
    __syncthreads();
    if (out.ptr != nullptr) {
#pragma unroll
      for (int e = 0; e < E; ++e) acc[e] *= corr;
      const int cnt = min(kWave, limit + 1 - j0);  // may be <= 0 for rows that see nothing here
      for (int jj = 0; jj < cnt; jj += kValueRows) {
        float v_next[kValueRows][E];
        if (jj + kValueRows < cnt) load_values(j0 + jj + kValueRows, v_next);
#pragma unroll
        for (int u = 0; u < kValueRows; ++u) {
          const float pj = p_s[w][jj + u];
#pragma unroll
          for (int e = 0; e < E; ++e) acc[e] = jj + u < cnt ? fmaf(pj, v_now[u][e], acc[e]) : acc[e];
        }
#pragma unroll
        for (int u = 0; u < kValueRows; ++u)
#pragma unroll
          for (int e = 0; e < E; ++e) v_now[u][e] = v_next[u][e];
      }
    }
    __syncthreads();
  }

  if (!row_ok) return;
  if (out.ptr != nullptr) {
    float* op = const_cast<float*>(row_ptr(out, b, l, h, t));
    const float inv = 1.f / lsum;
#pragma unroll
    for (int e = 0; e < E; ++e) op[lane + e * kWave] = acc[e] * inv;
  }
  if (lse != nullptr && lane == 0)
    lse[(static_cast<int64_t>(blockIdx.z) * dm.Hq + h) * rows + t] = m + logf(lsum);
}

constexpr int kColsumWaves = 8;
constexpr int kColsumRows = 4;  // query rows per wave and step
constexpr int kColsumTile = kColsumWaves * kColsumRows;

// A workgroup owns 64 candidate keys, one per lane, and takes the KV group's query rows 32 at a time: each
// of its eight waves four rows, whose dot products are four independent chains (one thread per key that
// walked all rows alone was a single chain of G * rows * head_dim dependent f64 operations).  The
// probabilities meet in LDS, where the first wave adds them while the others go on.  The sum runs in a fixed
// order (heads, then rows), so it is reproducible.
// Loops that are mostly this kernel, same bits: 3 layers of 14/2 heads, head_dim 64, two caches 5990 -> 1423 us;
// 4 layers of 16/4 heads, head_dim 128, 128 instruction rows 8010 -> 3978 us.  The smallest (4 heads, 32 rows,
// 72 states a step; 26 of its 52 us were here) 858 -> 525 us a document.
template <int D>
__global__ __launch_bounds__(kWave* kColsumWaves) void colsum_f32_kernel(Dims dm, View q, int rows, Segments ks,
                                                                            int causal, const float* lse, float* score) {
  __shared__ __attribute__((aligned(16))) Logit q_s[kColsumTile][D];
  __shared__ float p_s[2][kColsumTile][kWave];
  const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int g = blockIdx.y, b = blockIdx.z / dm.L, l = blockIdx.z % dm.L;
  const int n = ks.n_c + ks.c;
  const int j = blockIdx.x * kWave + lane;
  const bool key_ok = j < n;

  float kreg[D];
  {
    const float* kp = cand_ptr(ks, b, l, g, key_ok ? j : n - 1);
#pragma unroll
    for (int e = 0; e < D; e += kVec) load16(kp + e, kreg + e);
  }
  // first chunk row that sees candidate j (cache candidates are seen by every row)
  const int t_first = (causal && j >= ks.n_c) ? j - ks.n_c : 0;

  const int total = dm.G * rows;  // row r of the group is row r % rows of its head r / rows
  float sum = 0.f;
  for (int r0 = 0, buf = 0; r0 < total; r0 += kColsumTile, buf ^= 1) {
    int t[kColsumRows];
    float lse_r[kColsumRows];
#pragma unroll
    for (int x = 0; x < kColsumRows; ++x) {
      const int r = min(r0 + w * kColsumRows + x, total - 1);  // rows past the end are computed and not added
      const int h = g * dm.G + r / rows;
      t[x] = r % rows;
      lse_r[x] = lse[(static_cast<int64_t>(blockIdx.z) * dm.Hq + h) * rows + t[x]];
      const float* qp = row_ptr(q, b, l, h, t[x]);
#pragma unroll
      for (int e = 0; e < D; e += kWave)
        q_s[w * kColsumRows + x][e + lane] = static_cast<Logit>(qp[e + lane]);
    }
    // a wave reads only the rows it has written
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if constexpr (D > 64) {  // the key stays f32: kept as f64 across the loop it would spill
#pragma unroll
      for (int e = 0; e < D; ++e) asm volatile("" : "+v"(kreg[e]));
    }
    Logit dot[kColsumRows];
#pragma unroll
    for (int x = 0; x < kColsumRows; ++x) dot[x] = 0;
#pragma unroll
    for (int e = 0; e < D; ++e)
#pragma unroll
      for (int x = 0; x < kColsumRows; ++x)
        dot[x] = fma(q_s[w * kColsumRows + x][e], static_cast<Logit>(kreg[e]), dot[x]);
#pragma unroll
    for (int x = 0; x < kColsumRows; ++x) {
      const float p = expf(static_cast<float>(dot[x] * static_cast<Logit>(dm.scale) - static_cast<Logit>(lse_r[x])));
      p_s[buf][w * kColsumRows + x][lane] = t[x] >= t_first ? p : 0.f;
    }
    // the first wave reads this buffer before the next barrier, the others write it again after that one
    __syncthreads();
    if (w == 0) {
      const int rn = min(kColsumTile, total - r0);
#pragma unroll
      for (int x = 0; x < kColsumTile; ++x) sum += x < rn ? p_s[buf][x][lane] : 0.f;
    }
  }
  if (w == 0 && key_ok) score[(static_cast<int64_t>(blockIdx.z) * dm.Hkv + g) * n + j] = sum;
}

template <int D>
hipError_t attn_launch(const Dims& dm, View q, int rows, Segments ks, Segments vs, int causal, View out,
                         float* lse, hipStream_t st) {
  dim3 grid((rows + kRowsPerBlock - 1) / kRowsPerBlock, dm.Hq, dm.B * dm.L);
  hipLaunchKernelGGL(attn_f32_kernel<D>, grid, dim3(kWave * kRowsPerBlock), 0, st, dm, q, rows, ks, vs,
                     causal, out, lse);
  return hipGetLastError();
}

template <int D>
hipError_t colsum_launch(const Dims& dm, View q, int rows, Segments ks, int causal, const float* lse,
                           float* score, hipStream_t st) {
  const int n = ks.n_c + ks.c;
  dim3 grid((n + kWave - 1) / kWave, dm.Hkv, dm.B * dm.L);
  hipLaunchKernelGGL(colsum_f32_kernel<D>, grid, dim3(kWave * kColsumWaves), 0, st, dm, q, rows, ks, causal,
                     lse, score);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(const Dims& dm, View q, int rows, Segments ks, Segments vs, int causal, View out, float* lse,
                           hipStream_t st) {
  return dm.D == 64 ? attn_launch<64>(dm, q, rows, ks, vs, causal, out, lse, st)
                    : attn_launch<128>(dm, q, rows, ks, vs, causal, out, lse, st);
}

hipError_t launch_colsum_f32(const Dims& dm, View q, int rows, Segments ks, int causal, const float* lse, float* score,
                             hipStream_t st) {
  return dm.D == 64 ? colsum_launch<64>(dm, q, rows, ks, causal, lse, score, st)
                    : colsum_launch<128>(dm, q, rows, ks, causal, lse, score, st);
}

}  // namespace citrus
