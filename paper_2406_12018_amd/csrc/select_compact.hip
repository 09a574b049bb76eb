// Selection (Eq. (2)-(3): keep the k highest importance scores) and compaction
// (Eq. (3), (5): the evicted cache holds exactly the selected states).
#include <algorithm>
#include <type_traits>

#include "citrus_internal.h"
#include "evict_body.h"

namespace citrus {
namespace {

constexpr int kSelThreads = 256;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kWideThreads = 1024;

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

template <int ITEMS, int THREADS, Scores FORM, int BITS>
__global__ __launch_bounds__(THREADS) void topk_regs_kernel(const float* score, int heads_to_sum, int n, int k, int forced,
                                                           int32_t* idx) {
  __shared__ SelectLds<ITEMS, THREADS, BITS> lds;
  const float* base = score + static_cast<int64_t>(blockIdx.x) * heads_to_sum * n;
  int32_t* out = idx + static_cast<int64_t>(blockIdx.x) * k;
  if (n <= k) {  // nothing to evict: keep every candidate
    for (int j = threadIdx.x; j < n; j += THREADS) out[j] = j;
    return;
  }
  // a thread's kept candidates are neighbours in `out`: they go there through LDS, so that neighbouring lanes write neighbours
  topk_regs_body<ITEMS, THREADS, BITS, FORM>(lds, base, heads_to_sum, n, k, forced, nullptr, 0, [&](int pos, int j) { lds.key[pos] = j; });
  __syncthreads();
  for (int r = threadIdx.x; r < k; r += THREADS) out[r] = lds.key[r];
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

// Row gather: every thread moves 16 bytes of a K row and of a V row.  Output row r < kept is candidate idx[r]; the rows
// behind them are the candidates from append_from on.
struct CompactArgs {
  GatherViews v;
  const int32_t* idx;
  int idx_pitch, idx_heads, kept, rows, append_from, L;
  // accumulated scores (optional): the kept states take their sums along
  const float* score;
  float* acc_new;
  int n, acc_pitch;
};
__global__ __launch_bounds__(256) void compact_kernel(CompactArgs a) {
  const int g = blockIdx.y, b = blockIdx.z / a.L, l = blockIdx.z % a.L;
  const int r = (blockIdx.x * 256 + threadIdx.x) >> a.v.log_lanes;
  const int seg = threadIdx.x & ((1 << a.v.log_lanes) - 1);
  if (r >= a.rows) return;
  const int gi = a.idx_heads == 1 ? 0 : g;
  const int j = r < a.kept ? a.idx[(static_cast<int64_t>(blockIdx.z) * a.idx_heads + gi) * a.idx_pitch + r] : a.append_from + r - a.kept;
  const UnitRows u = unit_rows(a.v, b, l, g);
  u32x4 kv, vv;
  load_row(u, j, seg, kv, vv);
  store_row(u, r, seg, kv, vv);
  if (a.acc_new != nullptr && seg == 0 && r < a.kept) {
    const int64_t unit = static_cast<int64_t>(blockIdx.z) * gridDim.y + g;
    a.acc_new[unit * a.acc_pitch + r] = a.score[unit * a.n + max(0, min(j, a.n - 1))];
  }
}

// Selection and gather of a step in one launch: one head's selection per (document, layer, KV head), cut into `parts`
// workgroups that each repeat the selection and move `part_rows` of the rows it keeps.  Up to two evictions (the two
// caches of DUAL) share a launch.
// What bounds it: in small launches the chain arguments -> scores -> passes -> rows, four trips to memory of about 1 us
// each and 1.5 us of passes; the launches it replaces (sum of partial scores, selection, gather) took at least 4.4 us each
// whatever they did.  One layer of 32/8 heads, 1280 candidates, budget 768: 14.3 us in three launches, 9.0 in one.  Large
// ones are bound by memory and no faster than two launches (256 units 39.8 us against 6.7 + 33.0): evict_in_one_launch has the
// line.  A document with two caches of 128 units each, four launches of a step in one: 4.85 ms.
struct EvictArgs {
  EvictJob job[2];
  int first_blocks;  // workgroups of job 0
};
constexpr int kGatherRows = 4;  // rows of a thread in flight
template <int THREADS>
constexpr int kEvictBits = THREADS <= 256 ? 11 : 10;
constexpr int kMostKeptBytes = 6 * kWideThreads * sizeof(int32_t);  // the candidates of the rows that a unit keeps
// narrow instances stay within the LDS a launch may have without asking, whatever they keep
static_assert(sizeof(SelectLds<8, kSelThreads, kEvictBits<kSelThreads>>) + kMostKeptBytes <= 65536);

template <int ITEMS, int THREADS, Scores FORM>
__global__ __launch_bounds__(THREADS) void evict_kernel(EvictArgs args) {
  extern __shared__ int32_t sel[];  // the candidates of this part's kept rows
  __shared__ SelectLds<ITEMS, THREADS, kEvictBits<THREADS>> lds;
  const bool second = static_cast<int>(blockIdx.x) >= args.first_blocks;
  const EvictJob& a = args.job[second];
  const int block = second ? blockIdx.x - args.first_blocks : blockIdx.x;
  const int unit = block / a.parts, part = block - unit * a.parts;
  const int r0 = part * a.part_rows;
  evict_rows<ITEMS, THREADS, kEvictBits<THREADS>, FORM, kGatherRows>(a, unit, unit_scores(a, unit), r0, min(r0 + a.part_rows, a.rows),
                                                                            lds, sel);
}

}  // namespace

hipError_t launch_topk(const float* score, int units, int heads_to_sum, int n, int k, int forced, int32_t* idx,
                       hipStream_t st) {
  forced = min(forced, k);
  // Four times the threads where a unit's chain is long and the units fit the chip side by side, and for the sums over a layer's
  // heads, a read of heads_to_sum * n floats through one compute unit that needs its loads in flight (16 units of 32 heads x
  // 2048 candidates: 70 us candidate by candidate, 62 head by head, 12.7 with 1024 threads).  Two such workgroups fit a
  // compute unit.  From that number of units the chip is full, threads without a candidate are time lost, and short
  // sums go candidate by candidate on 256 threads.  us with 1024 threads | 256: 512 units of 2 heads x 300 candidates
  // 6.2 | 4.5, 4 x 1280 8.7 | 7.3, 8 x 1280 8.8 | 9.2; 1024 units of 8 x 500 10.7 | 9.1, 8 x 1000 13.9 | 14.4, 8 x 2048 20.4 |
  // 27.5, 2 x 3000 18.5 | 20.0; 2048 units of 8 x 1280 28.1 | 26.0, 8 x 2048 33.5 | 39.0.
  //
  // The radix: what a large one saves in passes shows where a unit has many candidates, what it costs in LDS where there are
  // many units of few.  us with 8 | 11 bits (1024 threads: 10), scores over six octaves: 8 units of 300 candidates 3.5 | 3.5, of
  // 1280 4.8 | 4.4, of 6144 8.4 | 7.8; 1024 units of 100 3.9 | 4.5, of 640 5.7 | 5.8, of 1280 7.6 | 6.8; 4096 units of 300 8.8 |
  // 11.7, of 640 13.0 | 14.6, of 1280 19.2 | 18.2.  Sums of 8 heads: 256 units of 640 5.5 | 6.1, of 2048 7.2 | 7.1, of 4096
  // 10.7 | 9.7; 1024 of 640 8.6 | 7.8; 4096 of 640 28 | 37.
  // (An instance whose threads hold more candidates than there are, and positions written by every thread for itself, took 1.2
  // to 1.9 times as long: 4096 units of 100 candidates 14.3 us, of 6144 132 instead of 88.)
  constexpr Scores kOne = Scores::kOneHead, kByHead = Scores::kSumByHead, kByCandidate = Scores::kSumByCandidate;
  const int cus = compute_units();
  const bool sums = heads_to_sum > 1;
  const int short_most = units > 5 * cus ? 10240 : units > 2 * cus ? 8192 : 5120;
  const bool short_sums = sums && n <= 2 * kWideThreads && units >= 2 * cus && static_cast<int64_t>(heads_to_sum) * n <= short_most;
  const bool wide = sums ? !short_sums : n > 2 * kWideThreads && units <= cus;
  auto kern = topk_kernel;
  int threads = kSelThreads;
  if (n <= 6 * kWideThreads) {
    threads = wide ? kWideThreads : kSelThreads;
    if (short_sums)
      kern = n <= 2 * kSelThreads ? topk_regs_kernel<2, kSelThreads, kByCandidate, 8>
             : units > 4 * cus    ? (n <= 5 * kSelThreads ? topk_regs_kernel<5, kSelThreads, kByCandidate, 8>
                                                          : topk_regs_kernel<8, kSelThreads, kByCandidate, 8>)
             : n <= 5 * kSelThreads ? topk_regs_kernel<5, kSelThreads, kByCandidate, 11>
                                    : topk_regs_kernel<8, kSelThreads, kByCandidate, 11>;
    else if (sums)
      kern = n <= kWideThreads       ? topk_regs_kernel<1, kWideThreads, kByHead, 8>
             : n <= 2 * kWideThreads ? (n <= 6 * kSelThreads ? topk_regs_kernel<2, kWideThreads, kByHead, 8>
                                                             : topk_regs_kernel<2, kWideThreads, kByHead, 10>)
             : n <= 3 * kWideThreads ? topk_regs_kernel<3, kWideThreads, kByHead, 10>
                                     : topk_regs_kernel<6, kWideThreads, kByHead, 10>;
    else
      kern = wide                    ? topk_regs_kernel<6, kWideThreads, kOne, 10>
             : n <= 2 * kSelThreads  ? topk_regs_kernel<2, kSelThreads, kOne, 8>
             : n <= 3 * kSelThreads  ? topk_regs_kernel<3, kSelThreads, kOne, 8>
             : n <= 5 * kSelThreads  ? topk_regs_kernel<5, kSelThreads, kOne, 11>
             : n <= 2 * kWideThreads ? topk_regs_kernel<8, kSelThreads, kOne, 11>
                                     : topk_regs_kernel<24, kSelThreads, kOne, 11>;
  }
  hipLaunchKernelGGL(kern, dim3(units), dim3(threads), 0, st, score, heads_to_sum, n, k, forced, idx);
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
                          int idx_pitch, int idx_heads, int kept, int appended, View k_new, View v_new,
                          const float* score, int n, float* acc_new, int acc_pitch, hipStream_t st) {
  CompactArgs a;
  a.v = gather_views(elem_bytes, dm, ks, vs, k_new, v_new);
  a.idx = idx;
  a.idx_pitch = idx_pitch;
  a.idx_heads = idx_heads;
  a.kept = kept;
  a.rows = kept + appended;
  a.append_from = ks.n_c + ks.c - appended;
  a.L = dm.L;
  a.score = score;
  a.n = n;
  a.acc_new = acc_new;
  a.acc_pitch = acc_pitch;
  const int rows_per_block = 256 >> a.v.log_lanes;
  hipLaunchKernelGGL(compact_kernel, dim3((a.rows + rows_per_block - 1) / rows_per_block, dm.Hkv, dm.B * dm.L), dim3(256), 0, st, a);
  return hipGetLastError();
}

bool evict_in_one_launch(int elem_bytes, const Dims& dm, int n, int rows) {
  if (n > 6 * kWideThreads) return false;
  // The launch that is saved is worth some microseconds.  Its gather is held up where it is bound by memory: workgroups that have
  // just selected all start to move rows together, and 1024 of their threads take a compute unit at a time.  us with two
  // launches | one, a score of one row per head included: head_dim 128 in bf16, 512 units, 400 rows (105 MB read) 56.5 | 58.2,
  // 200 rows 35.1 | 33.8; 512 units, 1536 rows 222 | 237; 2048 units, 768 rows 512 | 526.  head_dim 64: 256 units, 1536 rows
  // (101 MB) 54.3 | 52.7, 4096 units, 400 rows 269 | 267, but of 6144 candidates 256 units, 4096 rows (268 MB) 164 | 181.  More
  // than four units per compute unit of few rows: 4096 units, 31 of 2560 458 | 480.
  const int64_t units = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv, row_bytes = static_cast<int64_t>(dm.D) * elem_bytes;
  const bool wide = n > 8 * kSelThreads, much = 2 * units * rows * row_bytes >= 96 << 20;
  return !(much && (wide || row_bytes >= 256)) && !(wide && units > 4 * compute_units());
}

hipError_t launch_evict(int elem_bytes, const Dims& dm, const Eviction* e, int count, hipStream_t st) {
  if (count < 1 || count > 2) return hipErrorInvalidValue;
  EvictArgs args;
  const int units = dm.B * dm.L * dm.Hkv;
  int blocks = 0, lds = 0, n_max = 0;
  bool sums = false;
  for (int x = 0; x < count; ++x) {
    EvictJob& a = args.job[x];
    a = evict_job(elem_bytes, dm, e[x]);
    if (a.n > a.k) {
      n_max = std::max(n_max, a.n);
      sums = sums || a.sums > 1;
    }
  }
  // Workgroups of a job: two of 256 threads to a compute unit, one of 1024 (32 units of 6144 candidates, budget 4096, with
  // 256 | 1024 workgroups of 1024 threads: 29 | 48 us; two caches of 128 units, 256 threads: 256 | 512 | 1024
  // workgroups 4966 | 4944 | 5035 us a document), each with at least a wavefront's rows.
  const bool wide = n_max > 8 * kSelThreads;
  const int groups = wide ? compute_units() : 2 * compute_units();
  for (int x = 0; x < count; ++x) {
    EvictJob& a = args.job[x];
    cut_in_parts(a, 16, (groups + units - 1) / units);
    if (x == 0) args.first_blocks = units * a.parts;
    blocks += units * a.parts;
    lds = std::max(lds, static_cast<int>(std::min(a.part_rows, a.kept) * sizeof(int32_t)));
  }
  if (count == 1) args.job[1] = args.job[0];
  constexpr Scores kOne = Scores::kOneHead, kSums = Scores::kSumByHead;
  auto kern = sums ? evict_kernel<2, kSelThreads, kSums> : evict_kernel<2, kSelThreads, kOne>;
  int threads = kSelThreads;
  if (wide) {
    kern = sums ? evict_kernel<6, kWideThreads, kSums> : evict_kernel<6, kWideThreads, kOne>;
    threads = kWideThreads;
  } else if (n_max > 5 * kSelThreads) {
    kern = sums ? evict_kernel<8, kSelThreads, kSums> : evict_kernel<8, kSelThreads, kOne>;
  } else if (n_max > 2 * kSelThreads) {
    kern = sums ? evict_kernel<5, kSelThreads, kSums> : evict_kernel<5, kSelThreads, kOne>;
  }
  // One part per unit of a budget above 5344 rows, as on a part of the chip: the selection's LDS and the kept rows together are
  // more than the 64 KB a launch may have without asking.
  constexpr int kUnasked = 65536;
  if (wide && static_cast<int>(sizeof(SelectLds<6, kWideThreads, kEvictBits<kWideThreads>>)) + lds > kUnasked) {
    static LdsLimit limit[2];
    const hipError_t e = raise_lds_limit(limit[sums], reinterpret_cast<const void*>(kern), kMostKeptBytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(threads), lds, st, args);
  return hipGetLastError();
}

}  // namespace citrus
