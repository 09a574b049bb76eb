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
static int strip_rows(const Dims& dm, int rows, int n) {
  const int64_t groups32 = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv * ((dm.G * rows + 31) / 32);
  return n <= kStripMaxKeysShort && dm.G * rows > 32 && groups32 > compute_units() ? 64 : 32;
}

bool instr_strip_supported(const Dims& dm, const View& q, int rows, const Segments& ks) {
  const int n = ks.n_c + ks.c;
  if (n < 1 || n > kStripMaxKeysLong || rows < 1 || dm.G * rows > kStripMaxRows) return false;
  // Against the two-pass kernels, us with strips | two passes, 32/8 heads.  head_dim 128, 64 instruction rows, 1280 keys (64-row
  // strips; workgroups in brackets): 1 layer (64) 13.1 | 39, 16 layers (512) 32 | 42, 32 layers (1024) 56.9 | 57.8; 2560 keys,
  // 32-row strips: 16 layers (1024) 67 | 85, 32 layers (2048) 110 | 114.  So up to four workgroups per compute unit.
  // head_dim 64, where two workgroups share a compute unit: 8 layers 15 | 51, 32 layers (1024) 46 | 62, 64 layers (2048)
  // 85 | 117; 2560 keys, 32 layers (2048) 101 | 106; up to eight.  With one strip per KV head the two-pass kernel has one
  // workgroup per KV head too, and at head_dim 64 fits more of them: 700 keys, 16 rows, 32 layers (256) 11.6 | 13.9, 64
  // layers (512) 23.1 | 20.1.
  // Four 64-row strips per KV head against one round of the two-pass kernel with its 256 rows: up to three workgroups per
  // compute unit.  us per document of 4096 tokens, strips | two passes: 25 layers (800 workgroups) 2531 | 2484, 28 layers
  // (896) 2590 | 2559, 32 layers (1024), 640 keys 2328 | 2282; with two strips per KV head the two are level (512 units,
  // 128 rows: 2317 | 2284, 3167 | 3206), and 512 rows take the two-pass path two launches (128 units: 2577 | 2749).
  const int per_strip = strip_rows(dm, rows, n);
  const int64_t units = static_cast<int64_t>(dm.B) * dm.L * dm.Hkv, strips = (dm.G * rows + per_strip - 1) / per_strip;
  const bool one_round = per_strip == 64 && dm.G * rows <= 256 && units <= compute_units();
  const int rounds = dm.D == 128 ? (one_round ? 3 : 4) : strips > 1 ? 8 : 1;
  if (units * strips > rounds * compute_units()) return false;
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
  const bool tall = strip_rows(dm, rows, n) == 64, shorter = n <= kStripMaxKeysShort;
  auto launch = tall ? strip_launch<128, 2, 5> : shorter ? strip_launch<128, 1, 5> : strip_launch<128, 1, 10>;
  if (dm.D == 64) launch = tall ? strip_launch<64, 2, 5> : shorter ? strip_launch<64, 1, 5> : strip_launch<64, 1, 10>;
  return launch(dm, q, rows, ks, workspace, score, st, sums);
}

}  // namespace citrus
