// Selection and gather of one unit by one workgroup: what the launches that evict share.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "citrus_internal.h"

namespace citrus {
namespace {

// Order-preserving map float -> uint32 (larger float <=> larger key).  -0 is
// folded onto +0 first so that equal values get equal keys.
__device__ inline uint32_t order_key(float f) {
  f += 0.0f;
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The value a selection unit ranks for candidate j: one head's score, or the
// sum over the layer's KV heads taken in head order (layer-wise eviction).
// SHARED: other workgroups of this launch have written the scores (store_shared), maybe on another XCD.
template <bool SHARED = false>
__device__ inline float load_score(const float* p) {
  if constexpr (SHARED) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return *p;
}
template <bool SHARED = false>
__device__ inline float unit_score(const float* base, int heads_to_sum, int n, int j) {
  float s = load_score<SHARED>(base + j);
  for (int g = 1; g < heads_to_sum; ++g) s += load_score<SHARED>(base + static_cast<int64_t>(g) * n + j);
  return s;
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
enum class Scores { kOneHead, kSumByHead, kSumByCandidate, kSumShared };  // kSumShared: kSumByHead of what this launch writes

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
  if constexpr (FORM == Scores::kSumByHead || FORM == Scores::kSumShared) {
    float sum[ITEMS];
    auto add_rows = [&](auto in_flight, int g0) {  // up to so many rows from g0 on
      constexpr int kRows = decltype(in_flight)::value;
      float v[kRows][ITEMS];
#pragma unroll
      for (int x = 0; x < kRows; ++x)
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
          v[x][i] = load_score<FORM == Scores::kSumShared>(base + static_cast<int64_t>(min(g0 + x, rows - 1)) * n + min(i * THREADS + tid, n - 1));
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

// The eviction of one cache as the kernels take it.
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

__device__ inline const float* unit_scores(const EvictJob& a, int unit) { return a.score + static_cast<int64_t>(unit) * a.sums * a.n; }

// Output rows r0 .. r1 - 1 of a unit: the selection by the scores at base, then the rows that it keeps and those behind them, ROWS of a thread in
// flight.  sel: room for the candidates of the part's kept rows.  Every thread of the workgroup takes part.
template <int ITEMS, int THREADS, int BITS, Scores FORM, int ROWS>
__device__ __forceinline__ void evict_rows(const EvictJob& a, int unit, const float* base, int r0, int r1, SelectLds<ITEMS, THREADS, BITS>& lds,
                                           int32_t* sel) {
  const int s1 = min(r1, a.kept);  // rows r0 .. s1 are selected
  const int tid = threadIdx.x;
  const int bl = unit / a.Hkv, g = unit - bl * a.Hkv, b = bl / a.L, l = bl - b * a.L;
  const float* const acc = a.acc != nullptr ? a.acc + static_cast<int64_t>(unit) * a.acc_pitch : nullptr;
  if (r0 < s1) {  // block-uniform
    if (a.n <= a.k) {
      for (int r = r0 + tid; r < s1; r += THREADS) sel[r - r0] = r;
    } else {
      topk_regs_body<ITEMS, THREADS, BITS, FORM>(lds, base, a.sums, a.n, a.k, a.forced, acc, a.v.n_c, [&](int pos, int j) {
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
        float s = unit_score<FORM == Scores::kSumShared>(base, a.sums, a.n, j);
        if (j < a.v.n_c) s += acc[j];
        out[r] = s;
      }
    }
  }
  const UnitRows u = unit_rows(a.v, b, l, g);
  const int seg = tid & ((1 << a.v.log_lanes) - 1), step = THREADS >> a.v.log_lanes;
  // A thread's rows are requested together; where there are few, no more of them than there are (a row past the end is the last one again).
  auto move = [&](auto in_flight) {
    constexpr int kRows = decltype(in_flight)::value;
    for (int r = r0 + (tid >> a.v.log_lanes); r < r1; r += kRows * step) {
      u32x4 kv[kRows], vv[kRows];
#pragma unroll
      for (int x = 0; x < kRows; ++x) {
        const int rx = min(r + x * step, r1 - 1);
        load_row(u, rx < a.kept ? sel[rx - r0] : a.append_from + rx - a.kept, seg, kv[x], vv[x]);
      }
#pragma unroll
      for (int x = 0; x < kRows; ++x)
        if (r + x * step < r1) store_row(u, r + x * step, seg, kv[x], vv[x]);
    }
  };
  if (ROWS > 4 && r1 - r0 <= 2 * step)
    move(std::integral_constant<int, 2>{});
  else
    move(std::integral_constant<int, ROWS>{});
}

inline GatherViews gather_views(int elem_bytes, const Dims& dm, const Segments& ks, const Segments& vs, const View& k_new, const View& v_new) {
  const int lanes = dm.D * elem_bytes / 16;  // 8, 16 or 32
  return GatherViews{byte_view(ks.cache, elem_bytes), byte_view(ks.chunk, elem_bytes), byte_view(vs.cache, elem_bytes),
                     byte_view(vs.chunk, elem_bytes), byte_view(k_new, elem_bytes),    byte_view(v_new, elem_bytes),
                     ks.n_c, ks.n_c + ks.c, lanes == 8 ? 3 : lanes == 16 ? 4 : 5};
}

// The whole of a unit's rows is one part until the launcher cuts it.
inline EvictJob evict_job(int elem_bytes, const Dims& dm, const Eviction& e) {
  EvictJob a;
  a.v = gather_views(elem_bytes, dm, e.ks, e.vs, e.k_new, e.v_new);
  a.score = e.score.ptr;
  a.sums = e.score.sums;
  a.n = e.n;
  a.k = e.k;
  a.forced = std::min(e.forced, e.k);
  a.kept = std::min(e.n, e.k);
  a.rows = a.kept + e.appended;
  a.append_from = e.ks.n_c + e.ks.c - e.appended;
  a.parts = 1;
  a.part_rows = a.rows;
  a.L = dm.L;
  a.Hkv = dm.Hkv;
  a.idx = e.idx;
  a.acc = e.acc;
  a.acc_new = e.acc_new;
  a.acc_pitch = e.acc_pitch;
  return a;
}

// Cuts a unit into at most `most` parts of at least `least` rows.
inline void cut_in_parts(EvictJob& a, int least, int most) {
  a.parts = std::max(1, std::min((a.rows + least - 1) / least, most));
  a.part_rows = (a.rows + a.parts - 1) / a.parts;
  a.parts = (a.rows + a.part_rows - 1) / a.part_rows;
}

// What the score's workgroups of a merged launch do besides: nothing, the eviction of their unit once its scores are there
// (kEvict), or only the gather, where every candidate stays (kGather: job.parts workgroups per unit).
enum class Then { kNothing, kEvict, kGather };
struct StepTail {
  Then then;
  EvictJob job;
  int32_t* tickets;  // kEvict with several workgroups per unit: one per unit, zero before and after the launch
};

}  // namespace
}  // namespace citrus
