// Selection (Eq. (2)-(3): keep the k highest importance scores) and compaction
// (Eq. (3), (5): the evicted cache holds exactly the selected states).
#include <algorithm>
#include <type_traits>

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

// How a workgroup forms the values it ranks: one head's scores, or sums of several rows of scores (a layer's heads, the
// partial sums of a head).  The sums grow in row order (unit_score), either for all of a thread's candidates at a time,
// with several rows' loads in flight, or one candidate after the other, which waits for every load but needs no thread
// without a candidate.
enum class Scores { kOneHead, kSumByHead, kSumByCandidate };

// Radix passes of BITS bits: a large radix needs fewer passes, each a chain of dependent steps, and spreads the votes of
// scores that share their exponents over more bins; the histograms are cleared, every wave reads a whole one in each pass, and
// their LDS (24 KB at 11 bits, 4 KB at 8) is what the units side by side on a compute unit share.
template <int BITS>
struct Radix {
  static constexpr int kBits = BITS;
  static constexpr int kPasses = (32 + kBits - 1) / kBits;
  static constexpr int kBins = 1 << kBits;
  __host__ __device__ static constexpr int shift(int pass) { return 32 - kBits * (pass + 1) > 0 ? 32 - kBits * (pass + 1) : 0; }
};
__device__ __forceinline__ int padded(int j) { return j + (j >> 3); }  // candidates apart by 8 in different banks

// LDS of a selection.
template <int ITEMS, int THREADS, int BITS>
struct SelectLds {
  alignas(16) int hist[Radix<BITS>::kPasses][Radix<BITS>::kBins];
  uint32_t key[ITEMS * THREADS + ITEMS * THREADS / 8];
  alignas(16) int total[2][THREADS / 64];
};

// The same selection for a unit whose keys fit the workgroup's registers (n <= ITEMS * THREADS).  The scores are read once;
// the keys change hands through LDS so that a thread ranks consecutive candidates and the ordered emission is one prefix
// sum over the threads.  Exactly the result of topk_kernel.
//
// base: the unit's [rows][n] values.  acc (optional): a candidate j < n_acc carries acc[j] from earlier steps, added
// to its value.  n > k.  emit(position, candidate) is called once for each kept candidate.
//
// What bounds it: a chain of dependent steps (a launch that writes the identity takes 3.2 us), so the chain is kept
// short.  Every pass has a histogram of its own, cleared at the start, and every wave finds the bin by itself: one barrier
// per pass.  A pass whose bin is kept as a whole is the last one (scores that differ need two), and
// threshold-equal candidates are ranked only where some of them are left out.
template <int ITEMS, int THREADS, int BITS, Scores FORM, typename Emit>
__device__ __forceinline__ void topk_regs_body(SelectLds<ITEMS, THREADS, BITS>& lds, const float* base, int rows, int n, int k,
                                               int forced, const float* acc, int n_acc, Emit&& emit) {
  typedef Radix<BITS> R;
  constexpr int WAVES = THREADS / 64, kLaneBins = R::kBins / 64;
  static_assert(ITEMS <= 32, "one bit per item");
  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64;

  // ---- keys: read in the scores' order, handed over through LDS ----
  auto put = [&](int j, float value) {
    if (j < n) lds.key[padded(j)] = j < forced ? 0xffffffffu : order_key(value);
  };
  if constexpr (FORM == Scores::kSumByHead) {
    float sum[ITEMS];
    auto add_rows = [&](auto in_flight, int g0) {  // up to so many rows from g0 on
      constexpr int kRows = decltype(in_flight)::value;
      float v[kRows][ITEMS];
#pragma unroll
      for (int x = 0; x < kRows; ++x)
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
          v[x][i] = base[static_cast<int64_t>(min(g0 + x, rows - 1)) * n + min(i * THREADS + tid, n - 1)];
#pragma unroll
      for (int x = 0; x < kRows; ++x)
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          if (x == 0)
            sum[i] = g0 == 0 ? v[0][i] : sum[i] + v[0][i];
          else
            sum[i] = g0 + x < rows ? sum[i] + v[x][i] : sum[i];
        }
    };
    int g0 = 0;
    for (; rows - g0 > 2; g0 += 8) add_rows(std::integral_constant<int, 8>{}, g0);
    if (g0 < rows) add_rows(std::integral_constant<int, 2>{}, g0);
    if (acc != nullptr) {
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
        if (i * THREADS + tid < n_acc) sum[i] += acc[i * THREADS + tid];
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) put(i * THREADS + tid, sum[i]);
  } else {
    float value[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int j = i * THREADS + tid;
      value[i] = j < n ? unit_score(base, FORM == Scores::kOneHead ? 1 : rows, n, j) : 0.f;
    }
    if (acc != nullptr) {
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
        if (i * THREADS + tid < n_acc) value[i] += acc[i * THREADS + tid];
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) put(i * THREADS + tid, value[i]);
  }
  for (int x = tid; x < R::kPasses * R::kBins / 4; x += THREADS)
    reinterpret_cast<int4*>(&lds.hist[0][0])[x] = make_int4(0, 0, 0, 0);
  __syncthreads();
  // thread t ranks candidates t * per .. t * per + per - 1
  const int per = (n + THREADS - 1) / THREADS, j0 = tid * per, mine = min(per, n - j0);  // mine <= 0: none
  uint32_t key[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) key[i] = i < mine ? lds.key[padded(j0 + i)] : 0u;

  uint32_t prefix = 0;  // bits of T fixed so far (high bits)
  int need = k;         // rank of T among the keys that match the prefix
  bool whole = false;   // every key that matches the prefix is kept
#pragma unroll
  for (int pass = 0; pass < R::kPasses; ++pass) {
    if (whole) break;  // block-uniform
    const int shift = R::shift(pass);
    const uint32_t hi_mask = pass == 0 ? 0u : 0xffffffffu << R::shift(pass - 1 < 0 ? 0 : pass - 1);
    const uint32_t bin_mask = pass == 0 ? R::kBins - 1 : (1u << (R::shift(pass - 1 < 0 ? 0 : pass - 1) - shift)) - 1u;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (i < mine && (key[i] & hi_mask) == prefix) atomicAdd(&lds.hist[pass][(key[i] >> shift) & bin_mask], 1);
    __syncthreads();
    // lane x holds bins kLaneBins (63 - x) ..: the sum over the lanes in front counts the keys in higher bins.  The lanes
    // take their pieces in different orders: neighbouring lanes' bins lie in the same banks.
    const int4* const own = reinterpret_cast<const int4*>(&lds.hist[pass][kLaneBins * (63 - lane)]);
    int sum = 0;
#pragma unroll
    for (int x = 0; x < kLaneBins / 4; ++x) {
      const int4 v = own[(x + lane) % (kLaneBins / 4)];
      sum += v.x + v.y + v.z + v.w;
    }
    int incl = wave_prefix_sum(sum);
    int at = __builtin_ctzll(__ballot(incl - sum < need && need <= incl));  // exactly one lane: 1 <= need <= all keys
    need -= __builtin_amdgcn_readlane(incl - sum, at);
    // the same within that lane's bins, one per lane, the highest first
    const int top = kLaneBins * (63 - at) + kLaneBins - 1;
    const int own1 = lane < kLaneBins ? lds.hist[pass][top - lane] : 0;
    incl = wave_prefix_sum(own1);
    at = __builtin_ctzll(__ballot(incl - own1 < need && need <= incl));
    need -= __builtin_amdgcn_readlane(incl - own1, at);
    prefix |= static_cast<uint32_t>(top - at) << shift;
    whole = need == __builtin_amdgcn_readlane(own1, at);
  }
  // Keys above `thr` are kept; of the keys equal to it the first `need`.  Where the last bin is kept as a whole, thr
  // lies just below it (prefix > 0: all n > k keys match prefix 0 and lie in bins from 0 up).
  const uint32_t thr = whole ? prefix - 1u : prefix;
  if (whole) need = 0;

  // candidates of the threads in front (list 0: threshold-equal ones, 1: kept ones)
  auto in_front = [&](int list, int count) {
    const int incl = wave_prefix_sum(count);
    if (lane == 63) lds.total[list][w] = incl;
    __syncthreads();
    int before = incl - count;
#pragma unroll
    for (int x = 0; x < WAVES; ++x) {
      const int c = lds.total[list][x];
      before += x < w ? c : 0;
    }
    return before;
  };
  uint32_t keep_bits = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (i < mine && key[i] > thr) keep_bits |= 1u << i;
  if (need > 0) {  // block-uniform: some, not all, of the threshold-equal candidates
    uint32_t eq_bits = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (i < mine && key[i] == thr) eq_bits |= 1u << i;
    int left = need - in_front(0, __popc(eq_bits));
    for (; eq_bits != 0 && left > 0; eq_bits &= eq_bits - 1, --left) keep_bits |= eq_bits & -eq_bits;
  }
  int pos = in_front(1, __popc(keep_bits));
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (keep_bits & (1u << i)) emit(pos++, j0 + i);
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

// ---- the eviction's gather ----
// A tensor as the gathers address it: everything in bytes.
struct ByteView {
  char* ptr;
  int64_t sb, sl, sh, ss;
};
inline ByteView byte_view(const View& v, int esize) {
  return ByteView{static_cast<char*>(const_cast<void*>(v.ptr)), v.sb * esize, v.sl * esize, v.sh * esize, v.ss * esize};
}
__device__ inline char* unit_base(const ByteView& v, int b, int l, int g) { return v.ptr + (b * v.sb + l * v.sl + g * v.sh); }

// The rows of one unit that a gather moves: candidate j < n_c is cache row j, else chunk row j - n_c; output row r.
struct UnitRows {
  const char *k_cache, *k_chunk, *v_cache, *v_chunk;
  char *k_new, *v_new;
  int64_t ks_cache, ks_chunk, vs_cache, vs_chunk, ks_new, vs_new;  // row strides
  int n_c, n;  // cache rows, candidates
};
struct GatherViews {
  ByteView k_cache, k_chunk, v_cache, v_chunk, k_new, v_new;
  int n_c, n;
  int log_lanes;  // log2 of the 16-byte pieces of a row
};
__device__ inline UnitRows unit_rows(const GatherViews& a, int b, int l, int g) {
  return UnitRows{unit_base(a.k_cache, b, l, g), unit_base(a.k_chunk, b, l, g), unit_base(a.v_cache, b, l, g),
                  unit_base(a.v_chunk, b, l, g), unit_base(a.k_new, b, l, g),   unit_base(a.v_new, b, l, g),
                  a.k_cache.ss, a.k_chunk.ss, a.v_cache.ss, a.v_chunk.ss, a.k_new.ss, a.v_new.ss, a.n_c, a.n};
}
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;  // stays in registers, where an array of the struct uint4 does not
// 16 bytes (piece `seg`) of candidate j's key and value row
__device__ inline void load_row(const UnitRows& u, int j, int seg, u32x4& kv, u32x4& vv) {
  j = max(0, min(j, u.n - 1));  // a bad index must never become an out-of-bounds read
  // both addresses, then the choice: a choice between fields would become a load of the chosen field
  const char *const k_a = u.k_cache + j * u.ks_cache, *const k_b = u.k_chunk + (j - u.n_c) * u.ks_chunk;
  const char *const v_a = u.v_cache + j * u.vs_cache, *const v_b = u.v_chunk + (j - u.n_c) * u.vs_chunk;
  const bool cached = j < u.n_c;
  kv = reinterpret_cast<const u32x4*>(cached ? k_a : k_b)[seg];
  vv = reinterpret_cast<const u32x4*>(cached ? v_a : v_b)[seg];
}
__device__ inline void store_row(const UnitRows& u, int r, int seg, const u32x4& kv, const u32x4& vv) {
  reinterpret_cast<u32x4*>(u.k_new + r * u.ks_new)[seg] = kv;
  reinterpret_cast<u32x4*>(u.v_new + r * u.vs_new)[seg] = vv;
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
struct EvictJob {
  GatherViews v;
  const float* score;  // [units][sums][n]
  int sums, n, k, forced;   // the candidates that are ranked
  int kept, rows, append_from;  // output rows: the kept candidates, then candidates append_from ..
  int parts, part_rows, L, Hkv;
  int32_t* idx;        // optional, [units][k]
  const float* acc;    // optional: sums of earlier steps, [units][acc_pitch]
  float* acc_new;
  int acc_pitch;
};
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
  const int r0 = part * a.part_rows, r1 = min(r0 + a.part_rows, a.rows), s1 = min(r1, a.kept);  // rows r0 .. s1 are selected
  const int tid = threadIdx.x;
  const int bl = unit / a.Hkv, g = unit - bl * a.Hkv, b = bl / a.L, l = bl - b * a.L;
  const float* const base = a.score + static_cast<int64_t>(unit) * a.sums * a.n;
  const float* const acc = a.acc != nullptr ? a.acc + static_cast<int64_t>(unit) * a.acc_pitch : nullptr;
  if (r0 < s1) {  // block-uniform
    if (a.n <= a.k) {
      for (int r = r0 + tid; r < s1; r += THREADS) sel[r - r0] = r;
    } else {
      topk_regs_body<ITEMS, THREADS, kEvictBits<THREADS>, FORM>(lds, base, a.sums, a.n, a.k, a.forced, acc, a.v.n_c, [&](int pos, int j) {
        if (pos >= r0 && pos < s1) sel[pos - r0] = j;
      });
    }
    __syncthreads();
    if (a.idx != nullptr) {
      int32_t* const out = a.idx + static_cast<int64_t>(unit) * a.k;
      for (int r = r0 + tid; r < s1; r += THREADS) out[r] = sel[r - r0];
    }
    if (a.acc_new != nullptr) {
      float* const out = a.acc_new + static_cast<int64_t>(unit) * a.acc_pitch;
      for (int r = r0 + tid; r < s1; r += THREADS) {
        const int j = sel[r - r0];
        float s = unit_score(base, a.sums, a.n, j);
        if (j < a.v.n_c) s += acc[j];
        out[r] = s;
      }
    }
  }
  const UnitRows u = unit_rows(a.v, b, l, g);
  const int seg = tid & ((1 << a.v.log_lanes) - 1), step = THREADS >> a.v.log_lanes;
  for (int r = r0 + (tid >> a.v.log_lanes); r < r1; r += kGatherRows * step) {
    u32x4 kv[kGatherRows], vv[kGatherRows];
#pragma unroll
    for (int x = 0; x < kGatherRows; ++x) {
      const int rx = min(r + x * step, r1 - 1);
      load_row(u, rx < a.kept ? sel[rx - r0] : a.append_from + rx - a.kept, seg, kv[x], vv[x]);
    }
#pragma unroll
    for (int x = 0; x < kGatherRows; ++x)
      if (r + x * step < r1) store_row(u, r + x * step, seg, kv[x], vv[x]);
  }
}

GatherViews gather_views(int elem_bytes, const Dims& dm, const Segments& ks, const Segments& vs, const View& k_new, const View& v_new) {
  const int lanes = dm.D * elem_bytes / 16;  // 8, 16 or 32
  return GatherViews{byte_view(ks.cache, elem_bytes), byte_view(ks.chunk, elem_bytes), byte_view(vs.cache, elem_bytes),
                     byte_view(vs.chunk, elem_bytes), byte_view(k_new, elem_bytes),    byte_view(v_new, elem_bytes),
                     ks.n_c, ks.n_c + ks.c, lanes == 8 ? 3 : lanes == 16 ? 4 : 5};
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
    a.v = gather_views(elem_bytes, dm, e[x].ks, e[x].vs, e[x].k_new, e[x].v_new);
    a.score = e[x].score.ptr;
    a.sums = e[x].score.sums;
    a.n = e[x].n;
    a.k = e[x].k;
    a.forced = std::min(e[x].forced, e[x].k);
    a.kept = std::min(e[x].n, e[x].k);
    a.rows = a.kept + e[x].appended;
    a.append_from = e[x].ks.n_c + e[x].ks.c - e[x].appended;
    a.L = dm.L;
    a.Hkv = dm.Hkv;
    a.idx = e[x].idx;
    a.acc = e[x].acc;
    a.acc_new = e[x].acc_new;
    a.acc_pitch = e[x].acc_pitch;
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
    a.parts = std::min((a.rows + 15) / 16, (groups + units - 1) / units);
    a.part_rows = (a.rows + a.parts - 1) / a.parts;
    a.parts = (a.rows + a.part_rows - 1) / a.part_rows;
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
