// Attention over columns of any width where few keys are selected: one wavefront per query row reads the keys of
// the row's selected columns one by one, straight from the mask words (sea_gather.h; no key lists are
// written).  Bound: vector issue (1.2 instructions in flight per SIMD on bf16, 0.8 on fp32 tensors; rows come from
// the caches).
#include <algorithm>

#include "sea_columns.h"
#include "sea_gather.h"
#include "sea_internal.h"

namespace sea {
namespace {

constexpr int kGatherWaves = 4;
constexpr int kMaxColumns = 1024;

template <typename E>
struct GatherArgs {
  const E* Q;
  const E* K;
  const E* V;
  const uint32_t* mbits;  // [N][T][KW] selected-column bits
  E* O;
  const int32_t* seq_len;
  int32_t N, H, T, KW, causal;
  ColumnList g;
  double f;  // scale * log2(e)
};

template <typename E>
__global__ __launch_bounds__(kGatherWaves* kWave) void column_gather_kernel(GatherArgs<E> a) {
  __shared__ uint16_t cols[kGatherWaves][kMaxColumns];
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = static_cast<int64_t>(xcd_contiguous(blockIdx.x, gridDim.x)) * kGatherWaves + wid;
  if (row >= static_cast<int64_t>(a.N) * a.T) return;  // (no barrier below)
  const int64_t head = row / a.T, first = head * a.T * kHeadDim, at = row * kHeadDim;
  const int32_t t = static_cast<int32_t>(row - head * a.T), b = static_cast<int32_t>(head / a.H);
  const int32_t len = a.seq_len ? min(max(a.seq_len[b], 0), a.T) : a.T;
  const int32_t jmax = t < len ? (a.causal ? t : len - 1) : -1;
  ColumnKeys keys(a.g, a.mbits + row * a.KW, a.KW, jmax, cols[wid]);
  if (jmax < 0) keys.n = 0;
  if constexpr (sizeof(E) == 2)
    gather_row_bf16(keys, static_cast<float>(a.f), a.Q + at, a.K + first, a.V + first, a.O + at);
  else
    gather_row_f32(keys, a.f, a.Q + at, a.K + first, a.V + first, a.O + at);
}

template <typename E>
hipError_t launch(const Shape& s, const void* Q, const void* K, const void* V, const uint32_t* mbits, void* O, hipStream_t st) {
  GatherArgs<E> a{};
  a.Q = static_cast<const E*>(Q); a.K = static_cast<const E*>(K); a.V = static_cast<const E*>(V);
  a.mbits = mbits; a.O = static_cast<E*>(O); a.seq_len = s.seq_len;
  a.N = s.N; a.H = s.H; a.T = s.T; a.KW = (s.K + 31) / 32; a.causal = s.causal;
  a.g = column_list(s);
  a.f = sizeof(E) == 2 ? static_cast<double>(s.scale * kLog2e) : static_cast<double>(s.scale) * 1.4426950408889634;
  const int64_t rows = static_cast<int64_t>(s.N) * s.T;
  hipLaunchKernelGGL(column_gather_kernel<E>, dim3(static_cast<uint32_t>((rows + kGatherWaves - 1) / kGatherWaves)),
                     dim3(kGatherWaves * kWave), 0, st, a);
  return hipGetLastError();
}

}  // namespace

// Times of the two forms in us, from sweeps over T = 101 to 65535, K = 25 to 300 and 1 to 384 heads.  A row of its
// own takes a time per row and one per key it selects, n = k^ r of them (never less than a batch of 32); tiles walk
// the U keys of the list for all their rows, half of them when causal (chunks that no row selected are left out,
// which moves the line a little).  Launches that do not fill the chip take as long as one row or the longest
// list does.  Whole forward in us, tiles / rows, K = 128, H = 12: bf16, bidirectional, B = 2, T = 8001 k^ = 2, 4, 8
// 525 / 354, 658 / 606, 767 / 1108, T = 2041 k^ = 2, 4, 8, 16 97 / 59, 109 / 76, 112 / 107, 113 / 173, B = 1,
// T = 65535 one column of 64 keys 1626 / 863; causal, T = 8001 k^ = 2, 4 453 / 357, 496 / 601; H = 32, K = 256,
// B = 4, T = 1000, k^ = 1 120 / 142; H = 2, B = 1, T = 3001, k^ = 4, 16, 32 54 / 29, 55 / 48, 56 / 75.  fp32,
// B = 1, T = 3200 k^ = 4, 16, 32 460 / 242, 670 / 538, 715 / 950, causal 327 / 250, 404 / 526, 415 / 883.
// (A grid has at most 2^32 threads.)
bool column_gather_pays(const Shape& s, sea_dtype dt) {
  const int64_t rows = static_cast<int64_t>(s.N) * s.T;
  if (!column_list_supported(s) || s.K > kMaxColumns || rows > (int64_t(1) << 25)) return false;
  const ColumnList g = column_list(s);
  const double r = g.r == 0 ? g.cg.w0 + (g.cg.rm > 0 ? 1 : 0) : g.r;
  const double n = s.k_hat * r, U = g.U, walked = s.causal ? U / 2 : U, krows = rows * 1e-3;
  const bool bf16 = dt == SEA_BF16;
  // (heads that share a quota: a row may select up to sel_stride columns)
  const double one_row = (bf16 ? 0.05 : 0.06) * s.sel_stride * r, all_rows = krows * std::max(0.72, 0.45 + (bf16 ? 0.010 : 0.027) * n);
  const double one_list = bf16 ? 3.5 + 0.0115 * U : 2.0 + 0.0165 * U;
  const double all_lists = krows * (bf16 ? 0.65e-3 * walked : 0.35 + 4.3e-3 * walked);
  return std::max(one_row, all_rows) <= std::max(one_list, all_lists);
}

hipError_t launch_column_gather(const Shape& s, sea_dtype dt, const void* Q, const void* K, const void* V,
                                const uint32_t* mbits, void* O, hipStream_t st) {
  if (!column_list_supported(s) || s.K > kMaxColumns) return hipErrorNotSupported;
  StageScope scope(SEA_STAGE_SPARSE, st);
  return dt == SEA_BF16 ? launch<uint16_t>(s, Q, K, V, mbits, O, st) : launch<float>(s, Q, K, V, mbits, O, st);
}

}  // namespace sea
