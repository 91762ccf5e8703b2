// FlatCSR tensor of the expanded mask (Sec. 3.1.1 "FlatCSR", App. A.5 "FlatCSR: Modified CSR
// Format To Handle Grouped Mask"): M* [B][H][T][T] with the head and query axes exchanged and
// (head, key) flattened into one column axis, stored as CSR.  Row b T + t lists h T + j for the
// keys j head h attends from query t, heads ascending, keys ascending inside a head.
//
// Built from the per-(head, row) key lists in three launches: per-row entry counts with an
// exclusive scan inside each 256-row block, a one-block scan of the block totals, and a copy that
// moves each list to its place with one block (short lists: one wave) per CSR row (reads and writes
// contiguous).
#include "sea_internal.h"

namespace sea {
namespace {

constexpr int kScanRows = 256;
typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));  // lists start at any entry

__device__ __forceinline__ int64_t wave_inclusive(int64_t v, int lane) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int64_t u = __shfl_up(v, d, kWave);
    if (lane >= d) v += u;
  }
  return v;
}

__device__ __forceinline__ int32_t list_len(const int32_t* __restrict__ cnt, int64_t i, int32_t L) {
  return min(max(cnt[i], 0), L);
}

__global__ __launch_bounds__(kScanRows) void flat_count_kernel(Shape s, const int32_t* __restrict__ cnt,
                                                               int32_t L, int64_t R,
                                                               int64_t* __restrict__ crow,
                                                               int64_t* __restrict__ bsum) {
  __shared__ int64_t wtot[kScanRows / kWave];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * kScanRows + threadIdx.x;
  int64_t n = 0;
  if (row < R) {
    const int64_t b = row / s.T, t = row - b * s.T;
    for (int32_t h = 0; h < s.H; ++h) n += list_len(cnt, (b * s.H + h) * s.T + t, L);
  }
  const int64_t inc = wave_inclusive(n, lane);
  if (lane == kWave - 1) wtot[wave] = inc;
  __syncthreads();
  int64_t off = 0;
  for (int w = 0; w < wave; ++w) off += wtot[w];
  if (row < R) crow[row] = off + inc - n;  // exclusive inside the block; the block base comes later
  if (threadIdx.x == kScanRows - 1) bsum[blockIdx.x] = off + inc;
}

// exclusive scan of the block totals in place, grand total to *total
__global__ __launch_bounds__(1024) void flat_scan_kernel(int64_t* __restrict__ bsum, int64_t nblk,
                                                         int64_t* __restrict__ total) {
  __shared__ int64_t wtot[1024 / kWave];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t carry = 0;
  for (int64_t base = 0; base < nblk; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int64_t v = i < nblk ? bsum[i] : 0;
    const int64_t inc = wave_inclusive(v, lane);
    if (lane == kWave - 1) wtot[wave] = inc;
    __syncthreads();
    int64_t off = 0, all = 0;
    for (int w = 0; w < 1024 / kWave; ++w) {
      if (w < wave) off += wtot[w];
      all += wtot[w];
    }
    if (i < nblk) bsum[i] = carry + off + inc - v;
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = carry;
}

// One block per CSR row, its waves take the heads in turn: the head's place comes from a prefix sum over
// the counts (one lane per head), the list moves as 16-byte pieces, up to four per lane in flight.
// Bound: memory.  75 M entries (B = 4, H = 12, T = 2048): 0.19 -> 0.108 ms, 5.6 TB/s read and written (0.12 to 0.148
// with lists that go through the caches); one wave per CSR row with 4-byte pieces, heads one after the other, before.
template <bool PAST_CACHE>
__global__ __launch_bounds__(256) void flat_copy_kernel(Shape s, const int32_t* __restrict__ idx,
                                                        const int32_t* __restrict__ cnt, int32_t L,
                                                        int64_t* __restrict__ crow,
                                                        const int64_t* __restrict__ bsum,
                                                        int32_t* __restrict__ col, int64_t cap) {
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = blockIdx.x;
  const int64_t b = row / s.T, t = row - b * s.T;
  const int64_t start = crow[row] + bsum[row / kScanRows];
  __syncthreads();
  if (threadIdx.x == 0) crow[row] = start;  // only this block reads crow[row], before this store
  int64_t off0 = start;
  for (int32_t hb = 0; hb < s.H; hb += kWave) {
    const int32_t nh = min(s.H - hb, static_cast<int32_t>(kWave));
    int32_t n_l = lane < nh ? list_len(cnt, (b * s.H + hb + lane) * s.T + t, L) : 0;
    const int64_t incl = wave_inclusive(n_l, lane);
    for (int32_t hi = wid; hi < nh; hi += 4) {
      const int32_t n = __builtin_amdgcn_readlane(n_l, hi), h = hb + hi;
      const int64_t off = off0 + __shfl(incl, hi, kWave) - n;
      const int32_t* src = idx + ((b * s.H + h) * s.T + t) * L;
      const int32_t add = h * s.T;
      if (off + n > cap) {  // the tensor ends inside this list
        for (int32_t i = lane; i < n; i += kWave)
          if (off + i < cap) col[off + i] = add + src[i];
        continue;
      }
      int32_t* dst = col + off;
      const int32_t n4 = n & ~3;
      for (int32_t i0 = 0; i0 < n4; i0 += 1024) {
        i32x4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (i0 + 256 * q < n4) {
            const i32x4* const at = reinterpret_cast<const i32x4*>(src + min(i0 + 256 * q + 4 * lane, n4 - 4));
            if constexpr (PAST_CACHE) v[q] = __builtin_nontemporal_load(at); else v[q] = *at;
          }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (i0 + 256 * q + 4 * lane < n4) *reinterpret_cast<i32x4*>(dst + i0 + 256 * q + 4 * lane) = v[q] + add;
      }
      if (lane < n - n4) dst[n4 + lane] = add + src[n4 + lane];
    }
    off0 += __shfl(incl, kWave - 1, kWave);
  }
}

// Lists of at most 4 G entries: one wave per CSR row, G lanes per head, a 16-byte piece each, so that 64 / G heads
// move at a time and a row costs no barrier.  All three launches in us, a wave per CSR row with 4-byte pieces / a
// block per CSR row / this: B = 4, H = 12, T = 2048, 16 entries 16 / 25 / 13, 64 entries 21 / 29 / 18, 128 entries 29 /
// 29 / 25; H = 8, T = 8192, 64 entries 17 / 24 / 14; H = 32, T = 2048, 128 entries 46 / 27 / 27.  Above 64 entries only
// with 4096 rows and more, since a wave per row leaves the chip idle otherwise (B = 2, H = 32, T = 1000, up to 128
// entries 47 / 28 / 35).
template <int G>
__global__ __launch_bounds__(256) void flat_copy_short_kernel(Shape s, const int32_t* __restrict__ idx,
                                                              const int32_t* __restrict__ cnt, int32_t L, int64_t R,
                                                              int64_t* __restrict__ crow,
                                                              const int64_t* __restrict__ bsum,
                                                              int32_t* __restrict__ col, int64_t cap) {
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= R) return;
  const int64_t b = row / s.T, t = row - b * s.T;
  const int64_t start = crow[row] + bsum[row / kScanRows];
  int64_t off0 = start;
  for (int32_t hb = 0; hb < s.H; hb += kWave) {
    const int32_t nh = min(s.H - hb, static_cast<int32_t>(kWave));
    const int32_t n_l = lane < nh ? list_len(cnt, (b * s.H + hb + lane) * s.T + t, L) : 0;
    int32_t incl = n_l;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int32_t below = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += below;
    }
#pragma unroll 4
    for (int32_t h0 = 0; h0 < nh; h0 += kWave / G) {
      const int32_t hi = h0 + lane / G, i = 4 * (lane % G), h = hb + hi;
      const int32_t n = __shfl(n_l, hi, kWave), left = n - i;  // (0 entries past the last head)
      const int64_t at = off0 + __shfl(incl, hi, kWave) - left;
      const int32_t* src = idx + ((b * s.H + h) * s.T + t) * L + i;
      const int32_t add = h * s.T;
      if (left >= 4 && at + 4 <= cap) {
        *reinterpret_cast<i32x4*>(col + at) = *reinterpret_cast<const i32x4*>(src) + add;
      } else {
        for (int32_t e = 0; e < min(left, 4); ++e)
          if (at + e < cap) col[at + e] = add + src[e];
      }
    }
    off0 += __builtin_amdgcn_readlane(incl, kWave - 1);
  }
  if (lane == 0) crow[row] = start;  // only this wave reads crow[row], before this store
}

}  // namespace

size_t flatcsr_workspace(const Shape& s) {
  const int64_t R = static_cast<int64_t>(s.N / s.H) * s.T;
  return static_cast<size_t>((R + kScanRows - 1) / kScanRows) * sizeof(int64_t);
}

hipError_t launch_flatcsr(const Shape& s, const int32_t* idx, const int32_t* cnt, int32_t L, int64_t* crow,
                          int32_t* col, int64_t cap, void* ws, hipStream_t st) {
  const int64_t R = static_cast<int64_t>(s.N / s.H) * s.T;
  const int64_t nblk = (R + kScanRows - 1) / kScanRows;
  int64_t* bsum = static_cast<int64_t*>(ws);
  StageScope scope(SEA_STAGE_TOPK_MASK, st);
  hipLaunchKernelGGL(flat_count_kernel, dim3(static_cast<uint32_t>(nblk)), dim3(kScanRows), 0, st, s, cnt, L, R,
                     crow, bsum);
  hipLaunchKernelGGL(flat_scan_kernel, dim3(1), dim3(1024), 0, st, bsum, nblk, crow + R);
  const dim3 rows4(static_cast<uint32_t>((R + 3) / 4));
  if (L <= 64) hipLaunchKernelGGL(flat_copy_short_kernel<16>, rows4, dim3(256), 0, st, s, idx, cnt, L, R, crow, bsum, col, cap);
  else if (L <= 128 && R >= 4096) hipLaunchKernelGGL(flat_copy_short_kernel<32>, rows4, dim3(256), 0, st, s, idx, cnt, L, R, crow, bsum, col, cap);
  else if (lists_outgrow_cache(static_cast<int64_t>(s.N) * s.T, L)) hipLaunchKernelGGL(flat_copy_kernel<true>, dim3(static_cast<uint32_t>(R)), dim3(256), 0, st, s, idx, cnt, L, crow, bsum, col, cap);
  else hipLaunchKernelGGL(flat_copy_kernel<false>, dim3(static_cast<uint32_t>(R)), dim3(256), 0, st, s, idx, cnt, L, crow, bsum, col, cap);
  return hipGetLastError();
}

}  // namespace sea
