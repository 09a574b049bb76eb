// Instruction score (Eq. (1) with the instruction as the text, Section 4.2; summed form) with ONE product
// q.k per (instruction row, candidate key), bf16, head_dim 64 and 128, gfx950.
//
// The score of a key is a sum over instruction rows of softmax weights, and every row has its own
// normaliser, which is known only after the row has seen all keys.  Instead of a second pass over the
// keys, a workgroup keeps the un-normalised weights of a STRIP of instruction rows on chip:
//   * a workgroup owns one (document, layer, KV head) and one strip of 32 or 64 of the group's
//     instruction rows (heads x rows, flattened); its eight waves split the candidate keys, each wave
//     streaming its own 32-key tiles from global memory straight into a private double-buffered LDS
//     region (buffer_load ... lds) and waiting on its own vector-memory counter: no barrier in the key loop;
//   * S^T = K.Q^T on v_mfma_f32_32x32x16_bf16 puts one instruction row per lane; the lane keeps a lazy
//     reference (within 2^8 of its running maximum), turns the logits into weights exp2(s - reference)
//     right away and keeps them in registers in f32 (a strip of 32 rows x 1280 keys is 80
//     registers per lane over the 512 lanes), together with the reference each key tile was taken against;
//   * when the keys are through, the waves' (reference, sum) pairs meet in LDS and give each row's
//     normaliser; the column sums  sum_rows weight[row][key] * 2^(reference - row maximum) / row sum  are a
//     multiplication per weight and an exchange over the lanes;
//   * each strip writes its partial column; a second, tiny kernel adds the partial sums of a KV head
//     in a fixed order, or the selection that follows does.  No atomics: bit-reproducible.
// Against two passes over the keys this halves the matrix and the exponential work, the strips of a KV head
// run at the same time on one XCD, so that its keys come from HBM once, and a KV head is spread over several
// compute units.  What it pays for that is a fixed cost per workgroup (first tile and instruction rows,
// normaliser exchange), and keys that cross the L2 -> compute unit path once per strip.
#include "mfma_common.h"
#include "strip_score.h"

namespace citrus {
namespace {

template <int D, int ROW_TILES, int TPW>
__global__ __launch_bounds__(kStripThreads, 1) void instr_strip_kernel(StripArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  strip_score_body<D, ROW_TILES, TPW>(a, blockIdx.x, smem);
}

// score[u][j] = sum over the strips s (ascending) of part[u][s][j]
__global__ __launch_bounds__(256) void strip_sum_kernel(const float* __restrict__ part, int strips, int n, int64_t total,
                                                       float* __restrict__ score) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int64_t u = idx / n;
  const int j = static_cast<int>(idx - u * n);
  const float* p = part + u * strips * n + j;
  float v = p[0];
  for (int s = 1; s < strips; ++s) v += p[static_cast<int64_t>(s) * n];
  score[idx] = v;
}

template <int D, int ROW_TILES, int TPW>
hipError_t strip_launch(const Dims& dm, View q, int rows, Segments ks, float* part, float* score, hipStream_t st,
                        ScoreSums* sums) {
  const int n = ks.n_c + ks.c;
  StripArgs a = strip_args(dm, q, rows, ks, 32 * ROW_TILES, part);
  const int units = dm.B * dm.L * dm.Hkv, strips = a.strips;
  if (strips == 1) a.part = score;
  constexpr int lds = strip_lds_bytes<D, ROW_TILES>();
  auto kern = instr_strip_kernel<D, ROW_TILES, TPW>;
  static LdsLimit limit;
  hipError_t e = raise_lds_limit(limit, reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(units * strips), dim3(kStripThreads), lds, st, a);
  e = hipGetLastError();
  return e != hipSuccess ? e : finish_strip_scores(dm, a.part, strips, n, score, st, sums);
}

constexpr int kStripMaxRows = 4096;  // instruction rows per KV group: bounds a selection's sums over the strips

}  // namespace

int compute_units() {
  static std::atomic<int> cached[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  int cus = cached[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    cached[dev].store(cus, std::memory_order_relaxed);
  }
  return cus;
}

hipError_t finish_strip_scores(const Dims& dm, const float* part, int strips, int n, float* score, hipStream_t st,
                               ScoreSums* sums) {
  if (strips == 1) return hipSuccess;  // the only strip's column is the score
  if (sums != nullptr) {  // the consumer adds the strips' columns itself
    *sums = ScoreSums{part, strips};
    return hipSuccess;
  }
  const int64_t total = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv * n;
  hipLaunchKernelGGL(strip_sum_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, st, part, strips, n,
                     total, score);
  return hipGetLastError();
}

// Rows of a strip: 32 while such strips fit the compute units side by side (more workgroups, each with half the work), else
// 64 where a wave can hold them.
int instr_strip_rows(const Dims& dm, int rows, int n) {
  const int64_t groups32 = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv * ((dm.G * rows + 31) / 32);
  return n <= kStripMaxKeysShort && dm.G * rows > 32 && groups32 > compute_units() ? 64 : 32;
}

// Workgroups per compute unit up to which the strips of G * rows instruction rows per KV head are taken: where they are as fast as
// the two-pass kernels, or nearly.  Both were measured for 8 to 4096 KV heads, 1 to 4096 rows and 40 to 2560 keys, the sum over
// the strips included.  us with strips | two passes (KV heads):
//   up to 32 rows, one strip: ahead at every number of KV heads, head_dim 128, 1280 keys 11.2 | 24.4 (64), 261 | 380 (4096); the
//     lines lie where the larger groups' once did and could move out.
//   up to 64: one strip of 64 or two of 32.  head_dim 128: 1280 keys 78.5 | 104 (1024), but 40 keys 10.2 | 9.0 (512) and 96
//     keys 19.9 | 17.9 (1024), where a strip's fixed cost shows.  head_dim 64: ahead while the strips fit side by side, 1000 keys 11.9 | 16.1 (128).
//   up to 128: the two-pass kernel has one workgroup per KV head, the strips two to four.  head_dim 128, 700 keys 14.7 | 22.7
//     (128), 26.6 | 25.9 (256); 96 rows 25.8 | 22.5 (256); 1600 keys 27.8 | 37.1 (128), 50.8 | 43.5 (256), 2560 keys
//     54.3 | 57.7 (192).  head_dim 64, 2000 keys 47.9 | 39.4 (256).
//   up to 256: the two-pass kernel holds the keys in registers, at head_dim 128 all of them, and is through in one round while the
//     KV heads fit side by side: 1280 keys 32.0 | 43.8 (128), 44.3 | 46.6 (192), 59.6 | 54.2 (256); 160 rows, 700 keys 34.7 | 28.0
//     (256).  head_dim 64, where that instance spills: 90.5 | 108 (512); 2560 keys 78.8 | 90.6 (192), 104 | 94.9 (256).
//   more: two launches against one.  head_dim 128, 512 rows, 1280 keys 58.8 | 75.3 (128); head_dim 64 88.6 | 93.6 (64, 2048 rows),
//     4 x 128 rows, 2000 keys 50.3 | 43.6 (64), but 8 x 64 rows, 2560 keys 33.6 | 37.3 (32): the first launch takes a head's rows
//     128 at a time; head_dim 128, 4 x 256 rows, 2000 keys 65.4 | 58.7 (32).
// A strip of 64 rows works on 64 also where fewer are left (full_strips: none or up to 31 wanting); the two-pass kernels work on
// tiles of 32.
static int strip_rounds(const Dims& dm, int rows, int n, int64_t units) {
  const int total = dm.G * rows;
  const bool wide_head = dm.D == 128, full_strips = (total + 31) / 32 % 2 == 0, crowded = units > compute_units();
  if (total <= 32) return wide_head ? 4 : 1;
  if (n <= kStripMaxKeysShort) {
    if (total <= 64) return wide_head && n >= 64 ? (n >= 256 ? 4 : 3) : 1;
    if (total <= 128) return wide_head && full_strips && n >= 700 ? 3 : 1;
    if (total <= 256) return !wide_head ? 8 : crowded ? 4 : full_strips && n >= 300 ? 3 : 2;
    return !wide_head && (n >= 1000 || total >= 2048) ? 8 : 4;
  }
  if (total <= 64) return wide_head ? 4 : 2;
  if (total <= 128) return wide_head && crowded ? 4 : full_strips && n >= 2000 ? 3 : 2;
  if (total <= 256) return wide_head ? 4 : 6;
  if (wide_head) return total <= 512 ? 4 : 2;
  return rows >= 128 ? 1 : total <= 384 ? 5 : 2;
}

bool instr_strip_supported(const Dims& dm, const View& q, int rows, const Segments& ks) {
  const int n = ks.n_c + ks.c;
  if (n < 1 || n > kStripMaxKeysLong || rows < 1 || dm.G * rows > kStripMaxRows) return false;
  const int per_strip = instr_strip_rows(dm, rows, n);
  const int64_t units = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv, strips = (dm.G * rows + per_strip - 1) / per_strip;
  if (units * strips > static_cast<int64_t>(strip_rounds(dm, rows, n, units)) * compute_units()) return false;
  // The columns of several strips have to fit the scratch that a call of this shape has wherever it is made (one strip's
  // column is the score): what is launched, and so the bits, follow from the call alone and not from the block behind it.
  if (strips > 1 && static_cast<size_t>(units * strips) * n > instr_score_mfma_workspace_floats(dm, rows, n)) return false;
  // per-lane byte offsets into the group's instruction rows and into a key segment are 32-bit
  constexpr int64_t kSpan = int64_t{1} << 31;
  if (q.sh < 0 || q.ss <= 0 || ((dm.G - 1) * q.sh + (rows - 1) * q.ss + dm.D) * 2 >= kSpan) return false;
  auto fits = [&](const View& v, int r) { return v.ss > 0 && ((r > 0 ? r - 1 : 0) * v.ss + dm.D) * 2 < kSpan; };
  return fits(ks.cache, ks.n_c) && fits(ks.chunk, ks.c);
}

size_t instr_strip_workspace_floats(const Dims& dm, int rows, int n) {
  // Sized without a device query (the size of a workspace must not depend on where it is asked for): two columns per 32
  // rows, for up to 512 rows of a KV group and while 64-row strips make no more than 608 workgroups.  A larger call takes
  // strips where the scratch of the two-pass kernels, 16 floats per instruction row, holds its columns (512 keys with strips of
  // 32 rows, 1024 with 64) or where it needs none.
  constexpr size_t kRows = 512, kGroups = 608;
  const size_t units = static_cast<size_t>(dm.B) * dm.L * dm.Hkv;
  if (units < 1 || units > kGroups || dm.G < 1 || static_cast<size_t>(dm.G) > kRows || rows < 1 || n < 1) return 0;
  const size_t tall_strips = kGroups / units;    // 64-row strips per KV head, at most
  size_t r = kRows / dm.G;                       // G r <= kRows
  if (64 * tall_strips / dm.G < r) r = 64 * tall_strips / dm.G;  // ceil(G r / 64) <= tall_strips
  if (static_cast<size_t>(rows) < r) r = rows;
  if (r < 1) return 0;
  const int m = n < kStripMaxKeysLong ? n : kStripMaxKeysLong;
  return units * ((dm.G * r + 31) / 32) * 2 * m;
}

hipError_t launch_instr_strip(const Dims& dm, View q, int rows, Segments ks, float* workspace, size_t workspace_floats,
                              float* score, hipStream_t st, ScoreSums* sums) {
  const int n = ks.n_c + ks.c;
  if (!instr_strip_supported(dm, q, rows, ks)) return hipErrorInvalidValue;
  if (workspace_floats < instr_score_mfma_workspace_floats(dm, rows, n)) return hipErrorInvalidValue;
  const bool tall = instr_strip_rows(dm, rows, n) == 64, shorter = n <= kStripMaxKeysShort;
  auto launch = tall ? strip_launch<128, 2, 5> : shorter ? strip_launch<128, 1, 5> : strip_launch<128, 1, 10>;
  if (dm.D == 64) launch = tall ? strip_launch<64, 2, 5> : shorter ? strip_launch<64, 1, 5> : strip_launch<64, 1, 10>;
  return launch(dm, q, rows, ks, workspace, score, st, sums);
}

}  // namespace citrus
