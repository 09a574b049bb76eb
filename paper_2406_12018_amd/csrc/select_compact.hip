// Selection (Eq. (2)-(3): keep the k highest importance scores) and compaction
// (Eq. (3), (5): the evicted cache holds exactly the selected states).
#include "citrus_internal.h"

namespace citrus {
namespace {

constexpr int kSelThreads = 256;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kWideThreads = 1024;

// Order-preserving map float -> uint32 (larger float <=> larger key).  -0 is
// folded onto +0 first so that equal values get equal keys.
__device__ inline uint32_t order_key(float f) {
  f += 0.0f;
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The value a selection unit ranks for candidate j: one head's score, or the
// sum over the layer's KV heads taken in head order (layer-wise eviction).
__device__ inline float unit_score(const float* base, int heads_to_sum, int n, int j) {
  float s = base[j];
  for (int g = 1; g < heads_to_sum; ++g) s += base[static_cast<int64_t>(g) * n + j];
  return s;
}

// The key candidate j is ranked by.  The first `forced` candidates (the initial document states
// that are never evicted) rank above every score.
__device__ inline uint32_t unit_key(const float* base, int heads_to_sum, int n, int forced, int j) {
  return j < forced ? 0xffffffffu : order_key(unit_score(base, heads_to_sum, n, j));
}

// One workgroup per selection unit.  A radix select over the 32-bit order keys
// (4 passes of 8 bits, integer LDS histograms) finds the k-th largest key T;
// then one ordered pass emits, in ascending position, every candidate with
// key > T and the first (k - count(key > T)) candidates with key == T.  The
// result is exactly the top-k under (score descending, position ascending).
__global__ __launch_bounds__(kSelThreads) void topk_kernel(const float* score, int heads_to_sum, int n, int k,
                                                          int forced, int32_t* idx) {
  __shared__ int hist[256];
  __shared__ uint32_t s_prefix;
  __shared__ int s_need;
  __shared__ int wave_tot[2][kSelWaves];
  const int unit = blockIdx.x, tid = threadIdx.x;
  const float* base = score + static_cast<int64_t>(unit) * heads_to_sum * n;
  int32_t* out = idx + static_cast<int64_t>(unit) * k;

  if (n <= k) {  // nothing to evict: keep every candidate
    for (int j = tid; j < n; j += kSelThreads) out[j] = j;
    return;
  }

  uint32_t prefix = 0;  // bits of T fixed so far (high bits)
  int need = k;         // rank of T among the keys that match the prefix
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    hist[tid] = 0;  // kSelThreads == 256 bins
    __syncthreads();
    const uint32_t hi_mask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
    for (int j = tid; j < n; j += kSelThreads) {
      const uint32_t key = unit_key(base, heads_to_sum, n, forced, j);
      if ((key & hi_mask) == prefix) atomicAdd(&hist[(key >> shift) & 0xff], 1);
    }
    __syncthreads();
    // Find the bin where the count of keys in higher bins first reaches `need`: thread t owns bin t,
    // computes the number of keys in bins above it with a suffix scan (wave shuffles + one LDS hop),
    // and the one bin with above < need <= above + own announces itself.
    {
      const int own = hist[tid];
      int incl = own;  // inclusive suffix sum within the wave: bins tid .. end of wave
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_down(incl, o, 64);
        if ((tid % 64) + o < 64) incl += v;
      }
      if (tid % 64 == 0) wave_tot[0][tid / 64] = incl;  // total of this wave's 64 bins
      __syncthreads();
      int above = incl - own;
      for (int x = tid / 64 + 1; x < kSelWaves; ++x) above += wave_tot[0][x];
      if (above < need && need <= above + own) {
        s_prefix = prefix | (static_cast<uint32_t>(tid) << shift);
        s_need = need - above;
      }
    }
    __syncthreads();
    prefix = s_prefix;
    need = s_need;
    __syncthreads();
  }
  const uint32_t thr = prefix;  // key of the k-th best candidate
  // `need` = how many candidates with key == thr are kept (lowest positions first)

  const int lane = tid % 64, w = tid / 64;
  int kept_before = 0, eq_before = 0;
  for (int j0 = 0; j0 < n; j0 += kSelThreads) {
    const int j = j0 + tid;
    uint32_t key = 0;
    bool in = j < n;
    if (in) key = unit_key(base, heads_to_sum, n, forced, j);
    const bool gt = in && key > thr, eq = in && key == thr;
    const uint64_t eq_ballot = __ballot(eq);
    const uint64_t below = (1ull << lane) - 1ull;
    if (lane == 0) wave_tot[0][w] = __popcll(eq_ballot);
    __syncthreads();
    int eq_rank = eq_before + __popcll(eq_ballot & below);
    int eq_total = 0;
    for (int x = 0; x < kSelWaves; ++x) {
      if (x < w) eq_rank += wave_tot[0][x];
      eq_total += wave_tot[0][x];
    }
    const bool keep = gt || (eq && eq_rank < need);
    const uint64_t keep_ballot = __ballot(keep);
    if (lane == 0) wave_tot[1][w] = __popcll(keep_ballot);
    __syncthreads();
    int pos = kept_before + __popcll(keep_ballot & below);
    int keep_total = 0;
    for (int x = 0; x < kSelWaves; ++x) {
      if (x < w) pos += wave_tot[1][x];
      keep_total += wave_tot[1][x];
    }
    if (keep) out[pos] = j;
    kept_before += keep_total;
    eq_before += eq_total;
    __syncthreads();
  }
}

// Inclusive prefix sum over the 64 lanes with data-parallel-primitive moves: six dependent vector adds, where
// __shfl_up would make six round trips through the LDS unit.
__device__ __forceinline__ int wave_prefix_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1: lanes without a source add 0
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

// The same selection for a unit whose keys fit the workgroup's registers (n <= ITEMS * THREADS): the scores
// are read once (candidate i * THREADS + tid is item i of thread tid), the radix passes run on the registers, and
// the ordered emission counts the kept candidates per row of THREADS candidates and wave in LDS; a candidate's
// position is the sum of the counts in front of it.  Exactly the result of topk_kernel.
//
// What bounds it: a chain of dependent steps (a launch that writes the identity takes 3.2 us), so the chain is kept
// short.  Every pass has a histogram of its own, cleared at the start, and every wave reads the whole histogram and
// finds the bin by itself: one barrier per pass.  A pass whose bin is kept as a whole is the last one (scores
// that differ need two or three of the four), and threshold-equal candidates are ranked only where some of them
// are left out.
// Measured against four passes of three barriers with a shuffled scan, kernel trace: 8 units of 1280 candidates 6.9 ->
// 5.1 us, 128 units 8.1 -> 5.8 us.
// How a workgroup forms the values it ranks: one head's scores, or the sums over a layer's heads.  The sums grow in head
// order (unit_score), either for all of a thread's candidates at a time, with about 32 loads in flight, or one candidate
// after the other, which waits for every load but needs no thread without a candidate.
enum class Scores { kOneHead, kSumByHead, kSumByCandidate };

template <int ITEMS, int THREADS, Scores FORM>
__device__ __forceinline__ void topk_regs_body(const float* score, int heads_to_sum, int n, int k, int forced,
                                               int32_t* idx) {
  constexpr int WAVES = THREADS / 64, kBins = 256, kPasses = 4;
  static_assert(THREADS >= kBins && ITEMS <= 32, "thread t < 256 clears bin t; one bit per item");
  __shared__ __attribute__((aligned(16))) int hist[kPasses][kBins];
  __shared__ int row_cnt[2][ITEMS][WAVES];
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid % 64, w = tid / 64;
  const float* base = score + static_cast<int64_t>(unit) * heads_to_sum * n;
  int32_t* out = idx + static_cast<int64_t>(unit) * k;

  if (n <= k) {  // nothing to evict: keep every candidate
    for (int j = tid; j < n; j += THREADS) out[j] = j;
    return;
  }

  if (tid < kBins) {
#pragma unroll
    for (int pass = 0; pass < kPasses; ++pass) hist[pass][tid] = 0;
  }
  uint32_t key[ITEMS];
  if constexpr (FORM == Scores::kSumByHead) {
    float sum[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) sum[i] = base[min(i * THREADS + tid, n - 1)];
#pragma unroll(ITEMS <= 2 ? 16 : 4)
    for (int g = 1; g < heads_to_sum; ++g) {
      const float* head = base + static_cast<int64_t>(g) * n;
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) sum[i] += head[min(i * THREADS + tid, n - 1)];
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) key[i] = i * THREADS + tid < forced ? 0xffffffffu : order_key(sum[i]);
  } else {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int j = i * THREADS + tid;
      key[i] = j < n ? unit_key(base, FORM == Scores::kOneHead ? 1 : heads_to_sum, n, forced, j) : 0u;
    }
  }
  __syncthreads();

  uint32_t prefix = 0;  // bits of T fixed so far (high bits)
  int need = k;         // rank of T among the keys that match the prefix
  bool whole = false;   // every key that matches the prefix is kept
#pragma unroll
  for (int pass = 0; pass < kPasses; ++pass) {
    if (whole) break;  // block-uniform
    const int shift = 24 - 8 * pass;
    const uint32_t hi_mask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (i * THREADS + tid < n && (key[i] & hi_mask) == prefix) atomicAdd(&hist[pass][(key[i] >> shift) & 0xff], 1);
    __syncthreads();
    // lane x holds the four bins from 4 (63 - x) up: the sum over the lanes in front counts the keys in higher bins
    const int4 own = *reinterpret_cast<const int4*>(&hist[pass][4 * (63 - lane)]);
    const int sum = own.x + own.y + own.z + own.w;
    const int incl = wave_prefix_sum(sum);
    const uint64_t hit = __ballot(incl - sum < need && need <= incl);  // exactly one lane: 1 <= need <= all keys
    const int at = __builtin_ctzll(hit);
    need -= __builtin_amdgcn_readlane(incl - sum, at);
    int bin = 4 * (63 - at) + 3;
    int in_bin = __builtin_amdgcn_readlane(own.w, at);
    const int lower[3] = {own.z, own.y, own.x};
#pragma unroll
    for (int x = 0; x < 3; ++x)
      if (need > in_bin) {
        need -= in_bin;
        --bin;
        in_bin = __builtin_amdgcn_readlane(lower[x], at);
      }
    prefix |= static_cast<uint32_t>(bin) << shift;
    whole = need == in_bin;
  }
  // Keys above `thr` are kept; of the keys equal to it the first `need`.  Where the last bin is kept as a whole, thr
  // lies just below it (prefix > 0: all n > k keys match prefix 0 and lie in bins from 0 up).
  const uint32_t thr = whole ? prefix - 1u : prefix;
  if (whole) need = 0;

  // set bits of a ballot below this lane (v_mbcnt: no per-lane mask to keep in registers)
  auto lanes_below = [](uint64_t ballot) {
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(ballot >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(ballot), 0u)));
  };
  // candidates of the same row and wave in front of this one (threshold-equal first, then kept): 0 .. 63, a byte each
  uint32_t rank_in_row[(ITEMS + 3) / 4] = {};
  auto set_rank = [&](int i, int r) { rank_in_row[i / 4] = (rank_in_row[i / 4] & ~(0xffu << (8 * (i % 4)))) | (static_cast<uint32_t>(r) << (8 * (i % 4))); };
  auto get_rank = [&](int i) { return static_cast<int>((rank_in_row[i / 4] >> (8 * (i % 4))) & 0xffu); };
  uint32_t keep_bits = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (i * THREADS + tid < n && key[i] > thr) keep_bits |= 1u << i;
  if (need > 0) {  // block-uniform: some, not all, of the threshold-equal candidates
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if (i * THREADS >= n) break;  // block-uniform
      const bool eq = i * THREADS + tid < n && key[i] == thr;
      const uint64_t ballot = __ballot(eq);
      set_rank(i, lanes_below(ballot));
      if (lane == 0) row_cnt[0][i][w] = __popcll(ballot);
    }
    __syncthreads();
    int eq_before = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if (i * THREADS >= n) break;
      int eq_rank = eq_before + get_rank(i);
#pragma unroll
      for (int x = 0; x < WAVES; ++x) {
        const int c = row_cnt[0][i][x];
        if (x < w) eq_rank += c;
        eq_before += c;
      }
      if (i * THREADS + tid < n && key[i] == thr && eq_rank < need) keep_bits |= 1u << i;
      __builtin_amdgcn_sched_barrier(0);  // one row's counts in registers at a time
    }
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (i * THREADS >= n) break;  // block-uniform
    const uint64_t ballot = __ballot((keep_bits >> i) & 1u);
    set_rank(i, lanes_below(ballot));
    if (lane == 0) row_cnt[1][i][w] = __popcll(ballot);
  }
  __syncthreads();
  int kept_before = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (i * THREADS >= n) break;
    int pos = kept_before + get_rank(i);
#pragma unroll
    for (int x = 0; x < WAVES; ++x) {
      const int c = row_cnt[1][i][x];
      if (x < w) pos += c;
      kept_before += c;
    }
    if (keep_bits & (1u << i)) out[pos] = i * THREADS + tid;
    __builtin_amdgcn_sched_barrier(0);
  }
}

// (The instance with eight keys per thread takes 31 registers.  Two waves of the chunk-attention kernel leave a SIMD 16, so
// on a second stream these workgroups wait for a compute unit of their own, as they do on the attention's stream.)
template <int ITEMS, int THREADS, Scores FORM>
__global__ __launch_bounds__(THREADS) void topk_regs_kernel(const float* score, int heads_to_sum, int n, int k, int forced,
                                                           int32_t* idx) {
  topk_regs_body<ITEMS, THREADS, FORM>(score, heads_to_sum, n, k, forced, idx);
}

__global__ void iota_kernel(int32_t* p, int base, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = base + i;
}

// Accumulated scores: the sum a cache state carries is added to this step's score of the same candidate
// (chunk candidates start at their first score) ...
__global__ __launch_bounds__(256) void score_add_kernel(float* score, const float* acc, int n, int n_c, int acc_pitch,
                                                        int heads) {
  const int64_t u = static_cast<int64_t>(blockIdx.z) * heads + blockIdx.y;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j < n_c) score[u * n + j] += acc[u * acc_pitch + j];
}
// ... and the kept states take their sums along: acc_new[r] = score[idx[r]].
__global__ __launch_bounds__(256) void score_gather_kernel(const float* score, const int32_t* idx, float* acc_new, int n,
                                                           int m, int idx_pitch, int idx_heads, int acc_pitch,
                                                           int heads) {
  const int g = blockIdx.y;
  const int64_t u = static_cast<int64_t>(blockIdx.z) * heads + g;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= m) return;
  const int gi = idx_heads == 1 ? 0 : g;
  int j = idx[(static_cast<int64_t>(blockIdx.z) * idx_heads + gi) * idx_pitch + r];
  j = max(0, min(j, n - 1));  // a bad index must never become an out-of-bounds read
  acc_new[u * acc_pitch + r] = score[u * n + j];
}

// Row gather: every thread moves 16 bytes of a K row and 16 bytes of a V row.
template <int ROW_BYTES>
__global__ __launch_bounds__(256) void compact_kernel(Dims dm, Segments ks, Segments vs, int elem_bytes,
                                                      const int32_t* idx, int idx_pitch, int idx_heads, int m,
                                                      View k_new, View v_new) {
  constexpr int kLanesPerRow = ROW_BYTES / 16;
  constexpr int kRowsPerBlock = 256 / kLanesPerRow;
  const int g = blockIdx.y, b = blockIdx.z / dm.L, l = blockIdx.z % dm.L;
  const int r = blockIdx.x * kRowsPerBlock + threadIdx.x / kLanesPerRow;
  const int seg = threadIdx.x % kLanesPerRow;
  if (r >= m) return;
  const int gi = idx_heads == 1 ? 0 : g;
  int j = idx[(static_cast<int64_t>(blockIdx.z) * idx_heads + gi) * idx_pitch + r];
  j = max(0, min(j, ks.n_c + ks.c - 1));  // a bad index must never become an out-of-bounds read
  const int64_t unit_cache_k = b * ks.cache.sb + l * ks.cache.sl + g * ks.cache.sh;
  const int64_t unit_chunk_k = b * ks.chunk.sb + l * ks.chunk.sl + g * ks.chunk.sh;
  const int64_t unit_cache_v = b * vs.cache.sb + l * vs.cache.sl + g * vs.cache.sh;
  const int64_t unit_chunk_v = b * vs.chunk.sb + l * vs.chunk.sl + g * vs.chunk.sh;
  const char* ksrc;
  const char* vsrc;
  if (j < ks.n_c) {
    ksrc = static_cast<const char*>(ks.cache.ptr) + (unit_cache_k + static_cast<int64_t>(j) * ks.cache.ss) * elem_bytes;
    vsrc = static_cast<const char*>(vs.cache.ptr) + (unit_cache_v + static_cast<int64_t>(j) * vs.cache.ss) * elem_bytes;
  } else {
    const int jc = j - ks.n_c;
    ksrc = static_cast<const char*>(ks.chunk.ptr) + (unit_chunk_k + static_cast<int64_t>(jc) * ks.chunk.ss) * elem_bytes;
    vsrc = static_cast<const char*>(vs.chunk.ptr) + (unit_chunk_v + static_cast<int64_t>(jc) * vs.chunk.ss) * elem_bytes;
  }
  char* kdst = static_cast<char*>(const_cast<void*>(k_new.ptr)) +
               (b * k_new.sb + l * k_new.sl + g * k_new.sh + static_cast<int64_t>(r) * k_new.ss) * elem_bytes;
  char* vdst = static_cast<char*>(const_cast<void*>(v_new.ptr)) +
               (b * v_new.sb + l * v_new.sl + g * v_new.sh + static_cast<int64_t>(r) * v_new.ss) * elem_bytes;
  const uint4 kv = reinterpret_cast<const uint4*>(ksrc)[seg];
  const uint4 vv = reinterpret_cast<const uint4*>(vsrc)[seg];
  reinterpret_cast<uint4*>(kdst)[seg] = kv;
  reinterpret_cast<uint4*>(vdst)[seg] = vv;
}

template <int ROW_BYTES>
hipError_t compact_launch(int elem_bytes, const Dims& dm, Segments ks, Segments vs, const int32_t* idx,
                          int idx_pitch, int idx_heads, int m, View k_new, View v_new, hipStream_t st) {
  constexpr int kRowsPerBlock = 256 / (ROW_BYTES / 16);
  dim3 grid((m + kRowsPerBlock - 1) / kRowsPerBlock, dm.Hkv, dm.B * dm.L);
  hipLaunchKernelGGL((compact_kernel<ROW_BYTES>), grid, dim3(256), 0, st, dm, ks, vs, elem_bytes, idx, idx_pitch,
                     idx_heads, m, k_new, v_new);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_topk(const float* score, int units, int heads_to_sum, int n, int k, int forced, int32_t* idx,
                       hipStream_t st) {
  forced = min(forced, k);
  // Four times the threads where a unit's chain is long and the units fit the chip side by side (32 units of 6144
  // candidates: 17.9 us with 256 threads, 10.6 with 1024; with more units the chip is full either way), and for the sums
  // over a layer's heads, a read of heads_to_sum * n floats through one compute unit that needs its loads in flight
  // (16 units of 32 heads x 2048 candidates: 70 us candidate by candidate, 62 head by head, 12.7 with 1024 threads).
  // Two such workgroups fit a compute unit.  With more units than that the chip is full, threads without a candidate are
  // time lost, and short sums go candidate by candidate on 256 threads.  us with 1024 | 256 threads: 1024 units of 32
  // heads x 100 candidates 14.1 | 6.9, 8 x 500 11.2 | 7.5, 8 x 1000 14.0 | 14.4, 8 x 2048 20.3 | 25.1; six times the
  // compute units: 8 x 1000 20.2 | 16.9, 16 x 1000 30.1 | 28.6, 8 x 2048 29.0 | 29.6.  Up to two rounds of workgroups:
  // 512 units of 2 x 300 4.8 | 4.2, of 8 x 1280 7.1 | 9.1.
  constexpr Scores kOne = Scores::kOneHead, kByHead = Scores::kSumByHead, kByCandidate = Scores::kSumByCandidate;
  const int cus = compute_units();
  const bool sums = heads_to_sum > 1;
  const int short_most = units > 5 * cus ? 16384 : n <= 2 * kWideThreads ? 8192 : 6144;
  const bool short_sums = sums && units > 2 * cus && static_cast<int64_t>(heads_to_sum) * n <= short_most;
  auto kern = topk_kernel;
  int threads = kSelThreads;
  if (n <= 2 * kWideThreads) {
    kern = short_sums ? topk_regs_kernel<8, kSelThreads, kByCandidate>
           : sums     ? topk_regs_kernel<2, kWideThreads, kByHead>
                      : topk_regs_kernel<8, kSelThreads, kOne>;
    threads = sums && !short_sums ? kWideThreads : kSelThreads;
  } else if (n <= 6 * kWideThreads) {
    const bool wide = sums ? !short_sums : units <= cus;
    kern = short_sums                      ? topk_regs_kernel<24, kSelThreads, kByCandidate>
           : sums && n <= 3 * kWideThreads ? topk_regs_kernel<3, kWideThreads, kByHead>
           : sums                          ? topk_regs_kernel<6, kWideThreads, kByHead>
           : wide                          ? topk_regs_kernel<6, kWideThreads, kOne>
                                           : topk_regs_kernel<24, kSelThreads, kOne>;
    threads = wide ? kWideThreads : kSelThreads;
  }
  hipLaunchKernelGGL(kern, dim3(units), dim3(threads), 0, st, score, heads_to_sum, n, k, forced, idx);
  return hipGetLastError();
}

hipError_t launch_iota(int32_t* p, int base, int count, hipStream_t st) {
  hipLaunchKernelGGL(iota_kernel, dim3((count + 255) / 256), dim3(256), 0, st, p, base, count);
  return hipGetLastError();
}

hipError_t launch_score_add(const Dims& dm, float* score, const float* acc, int n, int n_c, int acc_pitch,
                            hipStream_t st) {
  if (n_c <= 0) return hipSuccess;
  hipLaunchKernelGGL(score_add_kernel, dim3((n_c + 255) / 256, dm.Hkv, dm.B * dm.L), dim3(256), 0, st, score, acc, n,
                     n_c, acc_pitch, dm.Hkv);
  return hipGetLastError();
}

hipError_t launch_score_gather(const Dims& dm, const float* score, const int32_t* idx, float* acc_new, int n, int m,
                               int idx_pitch, int idx_heads, int acc_pitch, hipStream_t st) {
  hipLaunchKernelGGL(score_gather_kernel, dim3((m + 255) / 256, dm.Hkv, dm.B * dm.L), dim3(256), 0, st, score, idx,
                     acc_new, n, m, idx_pitch, idx_heads, acc_pitch, dm.Hkv);
  return hipGetLastError();
}

hipError_t launch_compact(int elem_bytes, const Dims& dm, Segments ks, Segments vs, const int32_t* idx,
                          int idx_pitch, int idx_heads, int m, View k_new, View v_new, hipStream_t st) {
  const int row_bytes = dm.D * elem_bytes;
  switch (row_bytes) {
    case 128: return compact_launch<128>(elem_bytes, dm, ks, vs, idx, idx_pitch, idx_heads, m, k_new, v_new, st);
    case 256: return compact_launch<256>(elem_bytes, dm, ks, vs, idx, idx_pitch, idx_heads, m, k_new, v_new, st);
    case 512: return compact_launch<512>(elem_bytes, dm, ks, vs, idx, idx_pitch, idx_heads, m, k_new, v_new, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace citrus
