// Fused random-feature estimate for the common shapes (bf16, m in {64, 128, 256}, K <= 256): two kernels;
// no feature tensor reaches HBM.  Columns of a power-of-two width have a key kernel of their own, all
// other widths (K that does not divide T among them) take key_columns_kernel.  For causal
// columns wider than 16 keys the key side also leaves, per 16-key tile, the sum of the rounded
// features of the column's earlier tiles, split into three bf16 planes (24 bits, i.e. the fp32
// sum itself), which is all the own-column term needs from outside the wave.
// (Sec. 3 "Performer (FAVOR+)", Sec. 3.1 "Attention Matrix Estimation".)
//
//   key_state_kernel      phi(K) on the matrix cores -> per-column sums -> state (bf16, K x m)
//   estimate_rows_kernel  phi(Q) on the matrix cores, kept in registers as MFMA fragments ->
//                         A_hat tile = phi(Q) state^T (state streamed through LDS) -> causal
//                         masking, the row's own column from phi(Q) phi(K_own)^T with a
//                         lower-triangular mask -> row normalisation -> fp32 A_hat (optional)
//                         -> per-row top-k^ in registers -> selected-column bits (optional)
//
// Both projections are computed transposed, C[feature][row] = W X^T with v_mfma_f32_16x16x32_bf16,
// so lane l owns row l % 16 and, per 16-feature tile ft, the four features 16 ft + 4 (l / 16) + i.
// Two consecutive tiles give a lane 8 values = one MFMA operand fragment; the contraction slot
// <-> feature map this implies (slot 8 lg + e of chunk kc <-> feature 32 kc + 16 (e / 4) + 4 lg +
// e % 4) is used consistently for phi(Q), phi(K) and the stored state ("fragment order"), so
// accumulators feed the next product without any shuffle or memory round trip.
#include <algorithm>

#include "sea_columns.h"
#include "sea_internal.h"
#include "sea_lds.h"
#include "sea_rowlanes.h"
#include "sea_select.h"
#include "sea_tile.h"

namespace sea {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWRow = 72;  // halfwords per staged W row (128 B + 16 B pad): conflict-free b128 reads

__device__ __forceinline__ floatx4 mfma16(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float sumsq8(bf16x8 v) {
  const uint4 u = __builtin_bit_cast(uint4, v);
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
  float a = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = bf16lo_to_f32(w[i]), hi = bf16hi_to_f32(w[i]);
    a = fmaf(lo, lo, a);
    a = fmaf(hi, hi, a);
  }
  return a;
}
// eight floats (two feature tiles x four features) -> one operand fragment, RNE
__device__ __forceinline__ bf16x8 pack8(const float* lo4, const float* hi4) {
  uint4 u;
  u.x = pack_bf16(lo4[0], lo4[1]);
  u.y = pack_bf16(lo4[2], lo4[3]);
  u.z = pack_bf16(hi4[0], hi4[1]);
  u.w = pack_bf16(hi4[2], hi4[3]);
  return __builtin_bit_cast(bf16x8, u);
}

// sum over the 16 lanes of a DPP row (lanes with equal l / 16); every lane gets the total
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false);
  return x + __int_as_float(y);
}
constexpr int kQuadXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kQuadXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kRowHalfMirror = 0x141;  // lane i <-> 7 - i within each 8
constexpr int kRowMirror = 0x140;      // lane i <-> 15 - i within each 16
// all-reduce over aligned groups of W lanes (W = 1, 2, 4, 8, 16) of a row
template <int W>
__device__ __forceinline__ uint32_t group_sum_u(uint32_t x) {  // integer counts
  if (W >= 2) x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kQuadXor1, 0xf, 0xf, false));
  if (W >= 4) x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kQuadXor2, 0xf, 0xf, false));
  if (W >= 8) x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowHalfMirror, 0xf, 0xf, false));
  if (W >= 16) x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowMirror, 0xf, 0xf, false));
  return x;
}
// four independent 16-lane sums, step by step
__device__ __forceinline__ void group_sum4_u(uint32_t (&x)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x[i]), kQuadXor1, 0xf, 0xf, false));
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x[i]), kQuadXor2, 0xf, 0xf, false));
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x[i]), kRowHalfMirror, 0xf, 0xf, false));
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x[i]), kRowMirror, 0xf, 0xf, false));
}
template <int W>
__device__ __forceinline__ uint32_t group_max_u(uint32_t x) {
  if (W >= 2) x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kQuadXor1, 0xf, 0xf, false)));
  if (W >= 4) x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kQuadXor2, 0xf, 0xf, false)));
  if (W >= 8) x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowHalfMirror, 0xf, 0xf, false)));
  if (W >= 16) x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowMirror, 0xf, 0xf, false)));
  return x;
}
template <int W>
__device__ __forceinline__ float group_sum(float x) {
  if (W >= 2) x = dpp_add<kQuadXor1>(x);
  if (W >= 4) x = dpp_add<kQuadXor2>(x);
  if (W >= 8) x = dpp_add<kRowHalfMirror>(x);
  if (W >= 16) x = dpp_add<kRowMirror>(x);
  return x;
}

// Counters that later kernels of the layer add to.  (In a launch of their own they cost the layer 1.0 to 1.8 us, bidirectional,
// one column per row, H = 12: T = 8192 41.2 -> 39.6, 32768 92.4 -> 90.6, 131072 258.5 -> 257.5.)
template <int THREADS>
__device__ __forceinline__ void zero_counters(int32_t* counts, uint32_t n) {
  for (uint32_t x = blockIdx.x * THREADS + threadIdx.x; x < n; x += gridDim.x * THREADS) counts[x] = 0;
}

// ------------------------------------------------------------------------------------------
// key side: state[c] = bf16( sum over the keys of column c of phi(k_j) ), in fragment order.
// Bound: vector issue (an exponential and a multiply-add per key and feature, 40 % of the instructions).  W straight to LDS in
// unpadded rows, so that a CU holds a fourth block at m = 256 (three before, with twice the registers), and a tile's rows on
// their way under the tile before: 256 heads of 2048 keys, m = 256, 48.6 -> 40.9 us, 32 of 32768 85.9 -> 80.1, 12 of 131072,
// m = 128, 64.1 -> 60.6, 48 of 2048 7.0 -> 6.3.  (Two places for the sums in turn and one barrier less per tile: the same.)
// Block = 4 waves = 64 keys of one head (8 waves = 128 keys for 128-key columns, so that a column
// never spans two blocks; wider columns are finished by wide_columns_kernel).  WLOG = log2(column
// width), 0..7.
//
// Here the projection is taken with the keys as accumulator rows, C[key][feature] = X W^T: a lane
// then holds, per 16-feature tile, feature 16 ft + lr of the four keys 4 lg + i, so a column sum
// is three adds in the lane plus at most two cross-lane steps, which four tiles share (three swaps
// and three additions for four tiles), and no feature array is kept in registers.  Sums meet in LDS (one m-vector per wave and column part) and leave as
// coalesced bf16 rows.
// ------------------------------------------------------------------------------------------
// W rows lie without padding, pieces exchanged as in the rows kernel: four blocks of four waves share a CU at m = 256.
constexpr int key_waves(int WLOG) { return WLOG > 6 ? 8 : 4; }  // per block
template <int MC, int WLOG>
__global__ __launch_bounds__(64 * key_waves(WLOG), MC == 8 && WLOG > 2 && WLOG < 7 ? 4 : 1) void key_state_kernel(
    Shape s, const uint16_t* __restrict__ K, const uint16_t* __restrict__ W, uint16_t* __restrict__ state,
    uint16_t* __restrict__ pref, float* __restrict__ bsum_u, float* __restrict__ bsum_r, float c_dot,
    float c_norm, int32_t iters, int32_t* __restrict__ counts, uint32_t ncounts) {
  constexpr int m = 32 * MC;
  constexpr int w = 1 << WLOG;
  constexpr int kWaves = key_waves(WLOG);
  constexpr int kRows = 16 * kWaves;
  constexpr int kPartsWave = (w >= 4 && w < 16) ? 16 / w : 1;  // column sums a wave leaves in LDS
  constexpr int kSlots = kWaves * kPartsWave;
  __shared__ __attribute__((aligned(16))) uint16_t Ws[m * kHeadDim];
  // sums per wave and column part, and sums of the wave's bf16-rounded features
  constexpr int kParts = w >= 4 ? kSlots * m : 0, kRounded = w > 16 ? kWaves * m : 0;
  __shared__ __attribute__((aligned(16))) float part[kParts + kRounded > 0 ? kParts + kRounded : 1];
  float* const tpart = part + kParts;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  // a block takes `iters` consecutive key tiles of one head, so W is parked once for all of them
  const uint32_t tiles = (s.T + kRows - 1) / kRows;
  const uint32_t bph = (tiles + iters - 1) / iters;  // blocks per head
  const int64_t head = blockIdx.x / bph;
  const uint32_t tile_first = (blockIdx.x % bph) * iters;
  bf16x8 y0, y1;  // the next tile's rows
  auto request = [&](uint32_t tile) __attribute__((always_inline)) {
    const uint16_t* X = K + (head * s.T + min(static_cast<int32_t>(tile) * kRows + 16 * wid + lr, s.T - 1)) * kHeadDim;
    y0 = *reinterpret_cast<const bf16x8*>(X + 8 * lg);
    y1 = *reinterpret_cast<const bf16x8*>(X + 32 + 8 * lg);
  };
  {
    const u32x4 Wres = buffer_words(W, m * kHeadDim * 2);
    const uint32_t woff = (tid >> 3) * (kHeadDim * 2) + 16 * ((tid & 7) ^ ((tid >> 3) & 7));
    if ((Wres[0] & 3u) == 0u) {
#pragma unroll
      for (int q = 0; q < m / (8 * kWaves); ++q) buffer_load_lds16(Wres, Ws + (q * kWaves + wid) * 512, woff + q * 1024u * kWaves);
    } else {
#pragma unroll 1
      for (int q = 0; q < m / (8 * kWaves); ++q) buffer_load_lds16_odd(Wres, Ws + (q * kWaves + wid) * 512, woff + q * 1024u * kWaves);
    }
  }
  lds_loads_done();
  request(tile_first);  // (behind W, which would wait for them)
  zero_counters<64 * kWaves>(counts, ncounts);
  __syncthreads();
  const int32_t b = static_cast<int32_t>(head / s.H);
  const int32_t len = s.seq_len ? min(max(s.seq_len[b], 0), s.T) : s.T;
  const uint32_t tile_end = min(tile_first + static_cast<uint32_t>(iters), tiles);
  for (uint32_t tile = tile_first; tile < tile_end; ++tile) {
  if (tile != tile_first) __syncthreads();  // the sums of the previous tile have left LDS
  const int32_t blk_r0 = static_cast<int32_t>(tile) * kRows;
  const int32_t r0 = blk_r0 + wid * 16;
  uint16_t* sh = state + head * static_cast<int64_t>(s.K) * m;
  if (blk_r0 >= len) {  // no keys past the sequence's end: all sums are zero
    if (w < 4) {
      const int32_t n = min(kRows, s.T - blk_r0) / w * (m / 2);
      uint32_t* const to = reinterpret_cast<uint32_t*>(sh + static_cast<int64_t>(blk_r0 / w) * m);
      for (int32_t x = tid; x < n; x += 64 * kWaves) to[x] = 0u;
    } else {
      for (int32_t x = tid; x < kSlots * m; x += 64 * kWaves) part[x] = 0.f;
      if (w > 16 && pref)
        for (int32_t x = tid; x < kWaves * m; x += 64 * kWaves) tpart[x] = 0.f;
    }
  } else {
  // operand rows: key r0 + lr; accumulator rows: keys r0 + 4 lg + i
  const bf16x8 x0 = y0, x1 = y1;
  if (tile + 1 < tile_end) request(tile + 1);
  float nx = sumsq8(x0) + sumsq8(x1);
  nx += __shfl_xor(nx, 16, kWave);
  nx += __shfl_xor(nx, 32, kWave);  // |k|^2 of key lr, in every lane group
  float bias[4];
  bool act[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    act[i] = r0 + 4 * lg + i < len;
    // keys past the sequence end get an infinite bias: their features are exp2(-inf) = 0
    bias[i] = act[i] ? c_norm * __shfl(nx, (lane & 48) | (4 * lg + i), kWave) : INFINITY;
  }
  // Feature tiles are taken four at a time, so that the cross-lane part of the column sums can be
  // shared: a row swap of two tiles' sums leaves, after one addition, tile a's pair sums in the even
  // lane groups and tile b's in the odd ones; a half swap of two such registers and one more addition
  // leave the full sums of the four tiles in lane groups 0..3 -- three swaps and three additions for
  // four tiles, the same order of additions as summing each tile on its own, and one LDS store.
  static_assert((2 * MC) % 4 == 0, "feature tiles in groups of four");
  // slot of this lane's feature in a fragment-ordered row, for the tile its lane group ends up with
  const int slot_lane = 8 * (lr >> 2) + (lr & 3);
  const int wat0 = lr * kHeadDim + 8 * (lg ^ (lr & 7)), wat1 = lr * kHeadDim + 8 * ((lg + 4) ^ (lr & 7));
#pragma unroll
  for (int ft0 = 0; ft0 < 2 * MC; ft0 += 4) {
    float sum4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int ft = ft0 + q;
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = mfma16(x0, *reinterpret_cast<const bf16x8*>(Ws + ft * 16 * kHeadDim + wat0), acc);
      acc = mfma16(x1, *reinterpret_cast<const bf16x8*>(Ws + ft * 16 * kHeadDim + wat1), acc);
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_exp2f(fmaf(c_dot, acc[i], -bias[i]));
      // where feature 16 ft + lr sits in a fragment-ordered row
      const int slot = 32 * (ft >> 1) + 4 * (ft & 1) + slot_lane;
      if (w == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (r0 + 4 * lg + i < s.T) sh[static_cast<int64_t>(r0 + 4 * lg + i) * m + slot] = f32_to_bf16(v[i]);
      } else if (w == 2) {
#pragma unroll
        for (int i = 0; i < 4; i += 2)
          if (r0 + 4 * lg + i < s.T)
            sh[static_cast<int64_t>((r0 + 4 * lg + i) >> 1) * m + slot] = f32_to_bf16(v[i] + v[i + 1]);
      } else {
        sum4[q] = (v[0] + v[1]) + (v[2] + v[3]);  // the four keys share a column
        if (w == 4) part[(wid * kPartsWave + lg) * m + slot] = sum4[q];
        if (w > 16 && pref) {
          // The same tile sum over the ROUNDED features (what a causal row's own-column term uses), on
          // the matrix pipe: the four keys of this lane, rounded, are the contraction slots of an
          // operand whose column is the feature; against an all-ones operand every result row is the
          // sum over the wave's 16 keys, accumulated in fp32.
          // (the four-slot product: exactly the lane's four keys, no zero padding of the operand)
          const uint2 u = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
          const uint2 one = {0x3f803f80u, 0x3f803f80u};
          const floatx4 rs = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
              __builtin_bit_cast(shortx4, one), __builtin_bit_cast(shortx4, u), floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          if (lg == 0) tpart[wid * m + slot] = rs[0];
        }
      }
    }
    if (w >= 8) {
      // lane groups (0, 1, 2, 3) after the row swaps: pair sums of tiles (a, b, a, b) for keys
      // 0-7 in groups 0, 1 and keys 8-15 in groups 2, 3
      const auto ab = __builtin_amdgcn_permlane16_swap(__float_as_uint(sum4[0]), __float_as_uint(sum4[1]), false, false);
      const auto cd = __builtin_amdgcn_permlane16_swap(__float_as_uint(sum4[2]), __float_as_uint(sum4[3]), false, false);
      const float s_ab = __uint_as_float(ab[0]) + __uint_as_float(ab[1]);
      const float s_cd = __uint_as_float(cd[0]) + __uint_as_float(cd[1]);
      if (w == 8) {
        // two column parts per wave: group lg holds tile (lg & 1) of its pair, keys 8 (lg >> 1) ..
        const int tq = lg & 1, pw = lg >> 1;
        part[(wid * kPartsWave + pw) * m + 32 * (ft0 >> 1) + 4 * tq + slot_lane] = s_ab;
        part[(wid * kPartsWave + pw) * m + 32 * ((ft0 + 2) >> 1) + 4 * tq + slot_lane] = s_cd;
      } else {
        // full sums: lane group lg ends up with tile ft0 + lg
        const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(s_ab), __float_as_uint(s_cd), false, false);
        const float tot = __uint_as_float(t[0]) + __uint_as_float(t[1]);
        part[wid * kPartsWave * m + 32 * ((ft0 + lg) >> 1) + 4 * (lg & 1) + slot_lane] = tot;
      }
    }
  }
  }
  if (w < 4) continue;
  __syncthreads();
  if (w <= 16) {
    // each LDS vector is one finished column: columns blk_r0 / w + 0 .. kSlots - 1
    const int32_t col0 = blk_r0 >> WLOG;
    for (int x = tid; x < kSlots * m / 2; x += 64 * kWaves) {
      const int cl = (2 * x) / m, p = 2 * x - cl * m;
      if (col0 + cl < s.K)
        *reinterpret_cast<uint32_t*>(&sh[static_cast<int64_t>(col0 + cl) * m + p]) =
            pack_bf16(part[cl * m + p], part[cl * m + p + 1]);
    }
  } else {
    // column spans several waves of this block
    constexpr int wpc = w / 16;            // waves per column
    constexpr int cols = kRows / w;        // columns per block
    const int32_t col0 = static_cast<int32_t>(tile) * cols;
    for (int x = tid; x < cols * m; x += 64 * kWaves) {
      const int cl = x / m, p = x - cl * m;
      float acc = 0.f;
#pragma unroll
      for (int q = 0; q < wpc; ++q) acc += part[(cl * wpc + q) * m + p];
      if (WLOG == 7 && bsum_u) {
        // columns wider than this block: leave the block's sums (and, causal, the sums of the
        // rounded features) for the kernel that walks each column's blocks
        const int64_t blk = head * tiles + tile;
        bsum_u[blk * m + p] = acc;
        if (bsum_r) {
          float racc = 0.f;
#pragma unroll
          for (int q = 0; q < wpc; ++q) racc += tpart[q * m + p];
          bsum_r[blk * m + p] = racc;
        }
      } else if (col0 + cl < s.K) {
        sh[static_cast<int64_t>(col0 + cl) * m + p] = f32_to_bf16(acc);
      }
    }
    if (pref) {
      // exclusive prefix over the column's tiles, as bf16 planes hi + lo + lo2 (each difference is
      // exact in fp32, so the three planes carry the leading 24 bits of the sum)
      const int64_t ntile = s.T >> 4;
      const int64_t tile0 = static_cast<int64_t>(tile) * kWaves;
      // four consecutive features per thread: 16-byte reads of the tile sums, 8-byte stores
      for (int x = tid; x < kWaves * m / 4; x += 64 * kWaves) {
        const int q = x / (m / 4), p = (x - q * (m / 4)) * 4, qc = q & (wpc - 1);
        if (qc == 0 || tile0 + q >= ntile) continue;  // a column's first tile has nothing before it
        float4 P = {0.f, 0.f, 0.f, 0.f};
        for (int j = q - qc; j < q; ++j) {
          const float4 tp = *reinterpret_cast<const float4*>(&tpart[j * m + p]);
          P.x += tp.x; P.y += tp.y; P.z += tp.z; P.w += tp.w;
        }
        const float Pv[4] = {P.x, P.y, P.z, P.w};
        uint16_t hi[4], lo[4], lo2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          hi[e] = f32_to_bf16(Pv[e]);
          const float r1 = Pv[e] - bf16_to_f32(hi[e]);
          lo[e] = f32_to_bf16(r1);
          lo2[e] = f32_to_bf16(r1 - bf16_to_f32(lo[e]));
        }
        uint16_t* dst = pref + ((head * ntile + tile0 + q) * 3) * m + p;
        auto pack4 = [](const uint16_t* h) {
          return make_uint2(static_cast<uint32_t>(h[0]) | (static_cast<uint32_t>(h[1]) << 16),
                            static_cast<uint32_t>(h[2]) | (static_cast<uint32_t>(h[3]) << 16));
        };
        *reinterpret_cast<uint2*>(dst) = pack4(hi);
        *reinterpret_cast<uint2*>(dst + m) = pack4(lo);
        *reinterpret_cast<uint2*>(dst + 2 * m) = pack4(lo2);
      }
    }
  }
  }  // tiles of this block
}

// Columns of 256 keys or more: one block per (head, column) adds up the column's 128-key blocks.
// Causal: the sum of the rounded features of the column's earlier blocks goes out per block as
// three bf16 planes, like the tile prefixes inside a block.
__global__ __launch_bounds__(256) void wide_columns_kernel(Shape s, const float* __restrict__ bsum_u,
                                                           const float* __restrict__ bsum_r,
                                                           uint16_t* __restrict__ state,
                                                           uint16_t* __restrict__ bpref, int32_t nb) {
  const int32_t m = s.m, p = threadIdx.x;
  if (p >= m) return;
  const int64_t head = blockIdx.x / static_cast<uint32_t>(s.K);
  const int32_t c = static_cast<int32_t>(blockIdx.x % static_cast<uint32_t>(s.K));
  const int64_t blk0 = head * (s.T >> 7) + static_cast<int64_t>(c) * nb;
  float acc_u = 0.f, acc_r = 0.f;
  for (int32_t j = 0; j < nb; ++j) {
    if (bpref && j > 0) {
      const uint16_t hi = f32_to_bf16(acc_r);
      const float r1 = acc_r - bf16_to_f32(hi);
      const uint16_t lo = f32_to_bf16(r1);
      const uint16_t lo2 = f32_to_bf16(r1 - bf16_to_f32(lo));
      uint16_t* dst = bpref + ((blk0 + j) * 3) * m + p;
      dst[0] = hi;
      dst[m] = lo;
      dst[2 * m] = lo2;
    }
    acc_u += bsum_u[(blk0 + j) * m + p];
    if (bsum_r) acc_r += bsum_r[(blk0 + j) * m + p];
  }
  state[(head * s.K + c) * m + p] = f32_to_bf16(acc_u);
}

// ------------------------------------------------------------------------------------------
// key side for columns of any width.  A block takes G consecutive columns of one head (G <= 16, about
// 256 keys) and walks their keys in 16-key tiles; wave w owns a quarter of the features, whose rows of W
// stay in registers as operands.  Column sums are matrix products as well: with the block's columns as
// accumulator rows, sum[c][f] += onehot[c][key] phi[key][f], phi as the sum of three bf16 values (sea_tile.h; the
// accumulator layout of the projection is the operand layout of these products, so phi goes from one to
// the other in place), and the accumulators stay in registers over the whole walk -- no width, alignment
// or column boundary needs a case of its own.  Norms and columns of a 64-key step are taken once per
// block (wave w: its 16 keys) and shared through LDS.
// The first of the three, the ROUNDED features, has accumulators of its own (one 16x16x16 product per 16 features; the
// other two share the slots of one 16x16x32 product).  Causal: those are the running sum of the current column; before
// each tile that a column began in front of, the sum of that column's earlier keys goes out as fp32.
// A key whose features are not finite must not leave its column (causal rows before it do not know it): a block
// that finds such a sum takes its columns one by one.
// Bound: vector issue, two thirds of the time (135 instructions per 16 keys and wave, 100 of them exponentials and the
// splits), and the loads of W and of the first keys in front of nine tiles.  B = 8, H = 32, T = 2000, K = 256, m = 256,
// padded by 0-25 %: 91.3 -> 88.6 us against sums in fp32 products (two per 16 features and keys where a lane's four keys were
// added up per column first, four for narrow columns; half of the matrix pipe's time), T = 2001, m = 128, 48 heads
// 19.6 -> 19.0.  The rows of the next tile and step are requested ahead.
// Waves per SIMD, bidirectional: as many as with fp32 products, whose sums took half the registers (64 features keep two
// registers in memory for it): B = 32, H = 12, T = 500, K = 64, m = 128 34.4 -> 28.0 us with 80 registers in place of 86, m = 64,
// 512 heads 36.9 -> 33.0; launches of whole rounds are the same.
// ------------------------------------------------------------------------------------------
template <int MC, bool CAUSAL>
__global__ __launch_bounds__(256, CAUSAL || MC == 8 ? 4 : MC == 4 ? 6 : 8) void key_columns_kernel(Shape s, Columns cg, const uint16_t* __restrict__ K,
                                                          const uint16_t* __restrict__ W, uint16_t* __restrict__ state,
                                                          float* __restrict__ pref, float c_dot, float c_norm,
                                                          int32_t G, int32_t* __restrict__ counts, uint32_t ncounts) {
  constexpr int m = 32 * MC, FT = MC / 2;  // FT = 16-feature tiles per wave
  __shared__ __attribute__((aligned(16))) float bias_s[2][64];
  __shared__ __attribute__((aligned(16))) int32_t col_s[2][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const uint32_t groups = (s.K + G - 1) / G;
  const int64_t head = blockIdx.x / groups;
  const int32_t c0 = static_cast<int32_t>(blockIdx.x % groups) * G, c1 = min(c0 + G, s.K);
  const int32_t b = static_cast<int32_t>(head / s.H);
  const int32_t len = s.seq_len ? min(max(s.seq_len[b], 0), s.T) : s.T;
  const int32_t key0 = column_start(cg, c0), key1 = min(column_start(cg, c1), len);
  const uint16_t* Kh = K + head * static_cast<int64_t>(s.T) * kHeadDim;
  // W rows of this wave's features, in slot order: slot 16 (wid FT + ft) + lr of a fragment-ordered row
  bf16x8 w0[FT], w1[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const int slot = 16 * (wid * FT + ft) + lr;
    const int f = (slot & ~31) + 16 * ((slot >> 2) & 1) + 4 * ((slot & 31) >> 3) + (slot & 3);
    w0[ft] = *reinterpret_cast<const bf16x8*>(W + f * kHeadDim + 8 * lg);
    w1[ft] = *reinterpret_cast<const bf16x8*>(W + f * kHeadDim + 32 + 8 * lg);
  }
  floatx4 rsum[FT], rest[FT];  // sums of the rounded features, and of what rounding took off
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) rsum[ft] = rest[ft] = floatx4{0.f, 0.f, 0.f, 0.f};
  const MinusOnes minus = minus_ones();
  zero_counters<256>(counts, ncounts);

  const int32_t base = key0 & ~15;
  const int32_t nsteps = key1 > key0 ? (key1 - base + 63) / 64 : 0;
  // rows requested ahead: the next tile's, and the next step's own tile for its norms
  bf16x8 x0, x1, y0, y1;
  auto request = [&](int32_t j, bf16x8& a, bf16x8& b) {
    const uint16_t* X = Kh + static_cast<int64_t>(max(min(j, len - 1), 0)) * kHeadDim;
    a = *reinterpret_cast<const bf16x8*>(X + 8 * lg);
    b = *reinterpret_cast<const bf16x8*>(X + 32 + 8 * lg);
  };
  request(base + 16 * wid + lr, y0, y1);
  request(base + lr, x0, x1);
  for (int32_t st = 0; st < nsteps; ++st) {
    const int32_t s0 = base + 64 * st, buf = st & 1;
    {
      // norm and local column of key s0 + 16 wid + lr (keys outside the block's columns: no column)
      const int32_t j = s0 + 16 * wid + lr;
      float nx = sumsq8(y0) + sumsq8(y1);
      request(j + 64, y0, y1);
      nx += __shfl_xor(nx, 16, kWave);
      nx += __shfl_xor(nx, 32, kWave);
      if (lg == 0) {
        bias_s[buf][16 * wid + lr] = c_norm * nx;
        col_s[buf][16 * wid + lr] = (j >= key0 && j < key1) ? column_of(cg, j) - c0 : -1;
      }
    }
    __syncthreads();  // (the buffers alternate: one barrier per step)
#pragma unroll 1
    for (int tile = 0; tile < 4; ++tile) {
      const int32_t r0 = s0 + 16 * tile;
      if (r0 >= key1) break;
      const bf16x8 k0 = x0, k1 = x1;
      request(r0 + 16 + lr, x0, x1);
      const float4 bias = *reinterpret_cast<const float4*>(&bias_s[buf][16 * tile + 4 * lg]);
      const int4 cl = *reinterpret_cast<const int4*>(&col_s[buf][16 * tile + 4 * lg]);
      const float bv[4] = {bias.x, bias.y, bias.z, bias.w};
      const uint2 oh = {(cl.x == lr ? 0x3f80u : 0u) | (cl.y == lr ? 0x3f800000u : 0u),
                        (cl.z == lr ? 0x3f80u : 0u) | (cl.w == lr ? 0x3f800000u : 0u)};
      if (CAUSAL) {
        // keys of the tile's first column that lie before the tile: their sum is accumulator row lc
        const int32_t lc = col_s[buf][16 * tile];  // (uniform; -1: the column belongs to another block)
        if (lc >= 0 && column_start(cg, c0 + lc) < r0) {
          float* dst = pref + (head * ((s.T + 15) >> 4) + (r0 >> 4)) * m + 16 * wid * FT + lr;
          const int ri = __builtin_amdgcn_readfirstlane(lc & 3);
#pragma unroll
          for (int ft = 0; ft < FT; ++ft) {
            const float v = ri == 0 ? rsum[ft][0] : (ri == 1 ? rsum[ft][1] : (ri == 2 ? rsum[ft][2] : rsum[ft][3]));
            if (lg == (lc >> 2)) dst[16 * ft] = v;
          }
        }
      }
      const uint4 oh2 = {oh.x, oh.y, oh.x, oh.y};
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma16(k0, w0[ft], acc);
        acc = mfma16(k1, w1[ft], acc);
        bf16x2 part[3][2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          floatx2 f = {__builtin_amdgcn_exp2f(fmaf(c_dot, acc[2 * e], -bv[2 * e])),
                       __builtin_amdgcn_exp2f(fmaf(c_dot, acc[2 * e + 1], -bv[2 * e + 1]))};
#pragma unroll
          for (int n = 0; n < 3; ++n) {
            part[n][e] = __builtin_convertvector(f, bf16x2);
            if (n < 2)
              f = floatx2{__builtin_amdgcn_fdot2_f32_bf16(part[n][e], minus.lo, f[0], false),
                          __builtin_amdgcn_fdot2_f32_bf16(part[n][e], minus.hi, f[1], false)};
          }
        }
        const bf16x4 rounded = __builtin_shufflevector(part[0][0], part[0][1], 0, 1, 2, 3);
        const bf16x2 left[4] = {part[1][0], part[1][1], part[2][0], part[2][1]};
        rsum[ft] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(shortx4, oh), __builtin_bit_cast(shortx4, rounded), rsum[ft], 0, 0, 0);
        rest[ft] = mfma16(__builtin_bit_cast(bf16x8, oh2), join_pairs(left), rest[ft]);
      }
    }
  }
  float zero = 0.f;  // NaN if a sum is not finite
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int i = 0; i < 4; ++i) zero = fmaf(0.f, rsum[ft][i], fmaf(0.f, rest[ft][i], zero));
  if (__ballot(zero != 0.f) != 0ull) {
    // A feature that is not finite has reached every column of the block (zero times it): the wave's sums again,
    // column by column from the keys of each alone.
    __threadfence();  // (after the sums the walk has stored)
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      const int64_t f = 16 * (wid * FT + ft) + lr;
#pragma unroll 1
      for (int32_t c = c0; c < c1; ++c) {
        const int32_t first = column_start(cg, c), end = min(column_start(cg, c + 1), len);
        float total = 0.f, rounded = 0.f;
#pragma unroll 1
        for (int32_t r0 = first & ~15; r0 < end; r0 += 16) {
          if (CAUSAL && r0 > first && lg == 0) pref[(head * ((s.T + 15) >> 4) + (r0 >> 4)) * m + f] = rounded;
          request(r0 + lr, x0, x1);
          float nx = sumsq8(x0) + sumsq8(x1);
          nx += __shfl_xor(nx, 16, kWave);
          nx += __shfl_xor(nx, 32, kWave);
          floatx4 acc = {0.f, 0.f, 0.f, 0.f};
          acc = mfma16(x0, w0[ft], acc);
          acc = mfma16(x1, w1[ft], acc);
          float part = 0.f, part_r = 0.f;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int32_t j = r0 + 4 * lg + i;
            const float v = __builtin_amdgcn_exp2f(fmaf(c_dot, acc[i], -c_norm * __shfl(nx, 4 * lg + i, kWave)));
            part += j >= first && j < end ? v : 0.f;
            part_r += j >= first && j < end ? bf16_to_f32(f32_to_bf16(v)) : 0.f;
          }
          part += __shfl_xor(part, 16, kWave);
          part_r += __shfl_xor(part_r, 16, kWave);
          total += part + __shfl_xor(part, 32, kWave);
          rounded += part_r + __shfl_xor(part_r, 32, kWave);
        }
        if (lg == 0) state[(head * s.K + c) * m + f] = f32_to_bf16(total);
      }
    }
    return;
  }
  // accumulator register i of a lane: column c0 + 4 lg + i
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (c0 + 4 * lg + i < c1)
        state[(head * s.K + c0 + 4 * lg + i) * m + 16 * (wid * FT + ft) + lr] = f32_to_bf16(rsum[ft][i] + rest[ft][i]);
}

// the 16 rows' selected columns as mask words
template <int NCT>
__device__ __forceinline__ void store_mask_words(const Shape& s, const uint32_t (&sel)[NCT / 2], int64_t head, int32_t trow, int lg,
                                                 uint32_t* __restrict__ mbits) {
  // mask words: word j holds columns 32 j .. 32 j + 31 = tiles 2 j (low half) and 2 j + 1; this lane's
  // four columns of a tile sit at bits 4 lg .. 4 lg + 3 of the tile's half.  The four lanes of a row
  // combine their parts; the lane of the first row stores them as vectors.
  const int32_t kw = (s.K + 31) >> 5;
  constexpr int kWords = NCT / 2;
  if constexpr (kWords % 4 == 0) {
    // Four words at a time: a row swap of two words' parts and an OR leave word a's halves in the
    // even lane groups and word b's in the odd ones; a half swap of two such registers and an OR
    // leave the four finished words in lane groups 0..3 (three swaps for four words instead of
    // eight), and every lane stores the word of its group.
    uint32_t* mrow = mbits + (head * s.T + min(trow, s.T - 1)) * kw;
#pragma unroll
    for (int j = 0; j < kWords; j += 4) {
      uint32_t pw[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) pw[q] = sel[j + q] << (4 * lg);
      const auto ab = __builtin_amdgcn_permlane16_swap(pw[0], pw[1], false, false);
      const auto cd = __builtin_amdgcn_permlane16_swap(pw[2], pw[3], false, false);
      const auto t = __builtin_amdgcn_permlane32_swap(ab[0] | ab[1], cd[0] | cd[1], false, false);
      if (trow < s.T && j + lg < kw) mrow[j + lg] = t[0] | t[1];
    }
  } else {
    uint32_t words[kWords];
#pragma unroll
    for (int j = 0; j < kWords; ++j) words[j] = rows_or_u(sel[j] << (4 * lg));
    if (trow >= s.T || lg != 0) return;
    uint32_t* mrow = mbits + (head * s.T + trow) * kw;
    if (kw == kWords) {
      *reinterpret_cast<uint2*>(mrow) = make_uint2(words[0], words[1]);
    } else {
#pragma unroll
      for (int j = 0; j < kWords; ++j)
        if (j < kw) mrow[j] = words[j];
    }
  }
}

// ------------------------------------------------------------------------------------------
// From raw scores to mask bits, for 16 rows of a wave.  acc[ct][i] = raw score of row trow, column
// cc = 16 ct + 4 lg + i; ncnd = the row's number of admissible columns (0: inactive row), a causal row takes its
// own column (the last of them) from diag.  Tiles below ct_free lie wholly below every row's last column and
// need no test; tiles from column ncols_wave on hold nothing.
// A column that is no candidate of its row is a positive NaN from its first test on: v_mul_f32 keeps its sign whatever the
// factor, and as a selection key it lies below every score.  (Before, every column was tested in three passes, with copies that the compiler
// made around the tests, and the selected columns were put together from comparisons and shifts: about 230 of the 1800 vector
// instructions of a wave at m = K = 256.  Rows kernel alone, c4 at T = 32768 / c3: 320 -> 300 us, 166 -> 153 us.)
// ------------------------------------------------------------------------------------------
constexpr uint32_t kNoCandidate = 0x7fc00000u;
// One tile of finish_rows' first pass, in place.  Tiles below ct_free add their scores to the sum; in the others that hold
// candidates (`edges` = one past them) a lane's column `last` is its row's last candidate: that one takes diag (causal), the
// ones past it become kNoCandidate, like all of the tiles past those, and the sum gains the rest.  (Written with its branches, which are uniform: where two
// ways lead to the same four values the compiler copies them on both.  Masks are read two instructions after they are
// written at the earliest.)
template <bool CAUSAL>
__device__ __forceinline__ void bound_tile(floatx4& v, int ct, int32_t ct_free, int32_t edges, int32_t last, float diag, float& sum) {
  uint64_t m0, m1, m2, m3;
  float x0 = v[0], x1 = v[1], x2 = v[2], x3 = v[3], t, u;
#define SEA_TILE_FREE \
  "s_cmp_gt_i32 %[free], %[ct]\n\ts_cbranch_scc0 .Lsea_edge%=\n\t" \
  "v_add_f32 %[t], %[x0], %[x1]\n\tv_add_f32 %[u], %[x2], %[x3]\n\tv_add_f32 %[t], %[t], %[u]\n\tv_add_f32 %[sum], %[sum], %[t]\n\t" \
  "s_branch .Lsea_done%=\n.Lsea_edge%=:\n\ts_cmp_gt_i32 %[edges], %[ct]\n\ts_cbranch_scc0 .Lsea_none%=\n\t"
#define SEA_TILE_DIAG \
  "v_cmp_eq_u32 %[m0], 0, %[last]\n\tv_cmp_eq_u32 %[m1], 1, %[last]\n\tv_cmp_eq_u32 %[m2], 2, %[last]\n\tv_cmp_eq_u32 %[m3], 3, %[last]\n\t" \
  "v_cndmask_b32 %[x0], %[x0], %[diag], %[m0]\n\tv_cndmask_b32 %[x1], %[x1], %[diag], %[m1]\n\t" \
  "v_cndmask_b32 %[x2], %[x2], %[diag], %[m2]\n\tv_cndmask_b32 %[x3], %[x3], %[diag], %[m3]\n\t"
#define SEA_TILE_EDGE \
  "v_cmp_gt_i32 %[m0], 0, %[last]\n\tv_cmp_gt_i32 %[m1], 1, %[last]\n\tv_cmp_gt_i32 %[m2], 2, %[last]\n\tv_cmp_gt_i32 %[m3], 3, %[last]\n\t" \
  "v_cndmask_b32 %[t], %[x0], 0, %[m0]\n\tv_add_f32 %[sum], %[sum], %[t]\n\tv_cndmask_b32 %[t], %[x1], 0, %[m1]\n\tv_add_f32 %[sum], %[sum], %[t]\n\t" \
  "v_cndmask_b32 %[t], %[x2], 0, %[m2]\n\tv_add_f32 %[sum], %[sum], %[t]\n\tv_cndmask_b32 %[t], %[x3], 0, %[m3]\n\tv_add_f32 %[sum], %[sum], %[t]\n\t" \
  "v_cndmask_b32 %[x0], %[x0], %[none], %[m0]\n\tv_cndmask_b32 %[x1], %[x1], %[none], %[m1]\n\t" \
  "v_cndmask_b32 %[x2], %[x2], %[none], %[m2]\n\tv_cndmask_b32 %[x3], %[x3], %[none], %[m3]\n\t" \
  "s_branch .Lsea_done%=\n.Lsea_none%=:\n\t" \
  "v_mov_b32 %[x0], %[none]\n\tv_mov_b32 %[x1], %[none]\n\tv_mov_b32 %[x2], %[none]\n\tv_mov_b32 %[x3], %[none]\n.Lsea_done%=:"
#define SEA_TILE_OPERANDS \
  : [x0] "+&v"(x0), [x1] "+&v"(x1), [x2] "+&v"(x2), [x3] "+&v"(x3), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3), \
    [sum] "+&v"(sum), [t] "=&v"(t), [u] "=&v"(u) \
  : [free] "s"(ct_free), [edges] "s"(edges), [ct] "n"(ct), [last] "v"(last), [diag] "v"(diag), [none] "v"(kNoCandidate) \
  : "scc"
  if constexpr (CAUSAL)
    asm(SEA_TILE_FREE SEA_TILE_DIAG SEA_TILE_EDGE SEA_TILE_OPERANDS);
  else
    asm(SEA_TILE_FREE SEA_TILE_EDGE SEA_TILE_OPERANDS);
#undef SEA_TILE_FREE
#undef SEA_TILE_DIAG
#undef SEA_TILE_EDGE
#undef SEA_TILE_OPERANDS
  v = floatx4{x0, x1, x2, x3};
}
template <bool CAUSAL, int NCT>
__device__ __forceinline__ void finish_rows(const Shape& s, floatx4 (&acc)[NCT], int64_t head, int32_t trow, int32_t ncnd,
                                            int32_t ct_free, int32_t ncols_wave, float diag, int lg,
                                            float* __restrict__ A_hat, uint32_t* __restrict__ mbits) {
  const int32_t e = ncnd - 1 - 4 * lg;  // column 16 ct + 4 lg + i is the last admissible one iff 16 ct + i == e
  const int32_t edges = __builtin_amdgcn_readfirstlane((ncols_wave + 15) >> 4);
  ct_free = __builtin_amdgcn_readfirstlane(ct_free);
  float rsum = 0.f;
  // (what the instructions below read has left the matrix pipe: the compiler keeps that distance for its own only)
#pragma unroll
  for (int ct = 0; ct < NCT; ct += 4)
    asm volatile("s_nop %5" : "+v"(rsum), "+v"(acc[ct]), "+v"(acc[ct + 1]), "+v"(acc[ct + 2]), "+v"(acc[ct + 3]) : "n"(ct + 4 < NCT ? 0 : 15));
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    bound_tile<CAUSAL>(acc[ct], ct, ct_free, edges, e - ct * 16, diag, rsum);
  }
  const float r = rows_sum(rsum);
  // The normalised scores are kept NEGATED from here on: the bit pattern of -x (x >= +0) is
  // 0x80000000 | bits(x), which is the selection key itself, so the keys cost no instruction.
  const float ninv = r > 0.f ? -1.f / r : -0.f;
  // (as instructions: the sign of a NaN is kept by the multiplier and not by the language, whose compiler may move a negation)
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float x = acc[ct][i];
      asm("v_mul_f32 %0, %1, %0" : "+v"(x) : "v"(ninv));
      acc[ct][i] = x;
    }
  if (A_hat && trow < s.T) {
    float* out = A_hat + (head * s.T + trow) * s.K;
    if ((s.K & 3) == 0) {
      // a scratch A_hat read only by the grouped selection needs no zeros past a row's candidates
      const int32_t cend = s.cand_only ? min(s.K, ncnd) : s.K;
// Columns that are no candidates are written as zeros: the larger of zero and a NaN, or, in a wave with a row whose own
      // scores may be NaN or infinite, by a test.  (By a test in every wave: the estimate of causal layers of 256 x 2000 rows, m = 128,
      // K = 256 232 against 225 us, of 32 x 8192 100.0 / 95.0, m = 64, 32 x 16384 172 / 169.)
      auto write = [&](auto&& value) __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
          if (ct * 16 + 4 * lg < cend)
            *reinterpret_cast<float4*>(out + ct * 16 + 4 * lg) = make_float4(value(ct, 0), value(ct, 1), value(ct, 2), value(ct, 3));
      };
      if (__ballot(!(r == 0.f || (r > 0x1p-100f && r < 0x1p100f))) == 0ull)
        write([&](int ct, int i) { return fmaxf(-acc[ct][i], 0.f); });
      else
        write([&](int ct, int i) { return ct * 16 + i > e ? 0.f : -acc[ct][i]; });
    } else {
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (ct * 16 + 4 * lg + i < s.K) out[ct * 16 + 4 * lg + i] = ct * 16 + i > e ? 0.f : -acc[ct][i];
    }
  }
  if (!mbits) return;

  // ---- per-row top-k^ on the normalised scores, in registers (Sec. 3.1 "Grouped Top-k^
  // Selection", per-query grouping).  A row lives in four lanes, 4 NCT scores each.
  const uint32_t nsel = static_cast<uint32_t>(min(s.k_hat, ncnd));
  uint32_t key[NCT][4];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int i = 0; i < 4; ++i) key[ct][i] = __float_as_uint(acc[ct][i]);
  uint32_t sel[NCT / 2];
  select_columns<NCT>(key, nsel, ncnd, CAUSAL ? min(NCT, (ncols_wave + 15) >> 4) : NCT, s.k_hat,
                      search_top(nsel, r > 0x1p-100f && r < 0x1p100f), lg, sel);
  store_mask_words<NCT>(s, sel, head, trow, lg, mbits);
}

// ------------------------------------------------------------------------------------------
// query side.  Block = 4 waves = 64 rows of one head (16 per wave).
// ------------------------------------------------------------------------------------------
constexpr int kColStage = 32;   // columns of the state staged in LDS per step

// NCT = 16-column tiles a row can have (4, 8 or 16 for K <= 64, 128, 256).  WLOG = log2(column
// width) for widths up to 16; 5 stands for every wider power of two (the shift is then read from the
// shape), kAnyWidth for widths that are none, or that differ from column to column (K does not divide T).
constexpr int kAnyWidth = 6;

// (Waves per SIMD: what LDS leaves room for at m = 256; at fewer features what the registers of the widest case need.  Left to
// itself the compiler takes 150 registers for 65 to 128 columns where 84 do, and half of the waves are gone.  Three everywhere / so:
// c2 16.7 / 16.3 us, 48 heads of 4096, m = 128, K = 256 42.9 / 42.0, other shapes the same.)
template <int MC, bool CAUSAL, int WLOG, int NCT>
__global__ __launch_bounds__(256, MC == 8 ? 3 : NCT == 16 ? 4 : 5) void estimate_rows_kernel(Shape s, const uint16_t* __restrict__ Q,
                                                            const uint16_t* __restrict__ K,
                                                            const uint16_t* __restrict__ W,
                                                            const uint16_t* __restrict__ state,
                                                            const uint16_t* __restrict__ pref,
                                                            const uint16_t* __restrict__ bpref,
                                                            float* __restrict__ A_hat,
                                                            uint32_t* __restrict__ mbits, float c_dot,
                                                            float c_norm, int32_t group_heads, Columns cg) {
  constexpr int m = 32 * MC;
  constexpr bool ANYW = WLOG == kAnyWidth;
  const int wl = WLOG >= 5 ? 31 - __clz(s.T / s.K) : WLOG;  // log2(column width)
  auto col_of = [&](int32_t j) { return ANYW ? column_of(cg, j) : j >> wl; };
  // W, then the even stages of the state, each row without padding and its 16-byte pieces p at slot p ^ (row & 7):
  // rows come straight from memory, and the reads of eight neighbouring lanes hit distinct banks.  W is dead once
  // both projections are done; the odd stages and, causal with columns wider than 16 keys, the three prefix planes of
  // each wave's tile (requested with the wave's rows) then take its place.  (Through registers a stage cost 28 vector
  // instructions, four LDS stores and sixteen registers; this kernel, us without / with: c4 at T = 32768 359 / 342, ragged
  // T = 2000 183 / 168.)
  constexpr int kStageHalfwords = kColStage * m;
  __shared__ __attribute__((aligned(16))) uint16_t smem[m * kHeadDim + kStageHalfwords];
  static_assert(kStageHalfwords + 4 * 3 * m <= m * kHeadDim, "an odd stage and the planes fit W's place");
  uint16_t* const Ws = smem;
  uint16_t* const planes_s = smem + kStageHalfwords;
  auto stage_at = [&](int st) { return (st & 1) ? smem : smem + m * kHeadDim; };
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const uint32_t tiles = (s.T + 63) / 64;
  // Launch order = longest first: heads in groups whose state fits the L2s, inside a group the
  // row tiles from the last (most columns, causal) to the first, heads fastest.  Blocks are dealt
  // round-robin to the 8 XCDs, so with 8 | group size a head's state stays in one XCD's L2.
  const uint32_t per_group = static_cast<uint32_t>(group_heads) * tiles;
  const uint32_t grp = blockIdx.x / per_group, rem = blockIdx.x - grp * per_group;
  const uint32_t nh = min(static_cast<uint32_t>(group_heads), static_cast<uint32_t>(s.N) - grp * group_heads);
  const int64_t head = static_cast<int64_t>(grp) * group_heads + rem % nh;
  const int32_t wg_r0 = static_cast<int32_t>(tiles - 1 - rem / nh) * 64;
  const int32_t r0 = wg_r0 + wid * 16;
  const int32_t b = static_cast<int32_t>(head / s.H);
  const int32_t len = s.seq_len ? min(max(s.seq_len[b], 0), s.T) : s.T;

  // state staging: 32 columns x m halfwords per step, contiguous in memory; piece tid + 256 q of a step
  constexpr int kVecPerThread = m / 64;  // 16-byte pieces per thread and step
  static_assert(MC >= 2, "m >= 64");
  const int32_t ncols_wg = CAUSAL ? __builtin_amdgcn_readfirstlane(min(s.K, col_of(min(wg_r0 + 63, s.T - 1)) + 1)) : s.K;
  const int32_t nstages = (ncols_wg + kColStage - 1) / kColStage;
  const uint32_t state_bytes = static_cast<uint32_t>(s.K) * m * 2;
  const u32x4 Sres = buffer_words(state + head * static_cast<int64_t>(s.K) * m, state_bytes);
  auto fetch_stage = [&](int st, int tid_) __attribute__((always_inline)) {
    const int srow = tid_ / (m / 8), spart = tid_ % (m / 8);
    const uint32_t soff = srow * m * 2 + 16 * (spart ^ (srow & 7));
#pragma unroll
    for (int q = 0; q < kVecPerThread; ++q) {
      // (columns past K read the state's last piece; nobody looks at them)
      const uint32_t from = static_cast<uint32_t>(st) * kStageHalfwords * 2 + q * 4096u;
      buffer_load_lds16(Sres, stage_at(st) + q * 2048 + wid * 512, min(soff + from, state_bytes - 16u));
    }
  };
  if (nstages > 0) fetch_stage(0, tid);
  {
    const u32x4 Wres = buffer_words(W, m * kHeadDim * 2);
    const uint32_t woff = (tid >> 3) * (kHeadDim * 2) + 16 * ((tid & 7) ^ ((tid >> 3) & 7));
    if ((Wres[0] & 3u) == 0u) {
#pragma unroll
      for (int q = 0; q < m / 32; ++q) buffer_load_lds16(Wres, Ws + q * 2048 + wid * 512, woff + q * 4096u);
    } else {
#pragma unroll 1
      for (int q = 0; q < m / 32; ++q) buffer_load_lds16_odd(Wres, Ws + q * 2048 + wid * 512, woff + q * 4096u);
    }
  }

  // the wave's query (and, causal, key) rows
  const int32_t t = r0 + lr, tc = min(t, s.T - 1);
  const uint16_t* Xq = Q + (head * s.T + tc) * kHeadDim;
  const bf16x8 x0 = *reinterpret_cast<const bf16x8*>(Xq + 8 * lg);
  const bf16x8 x1 = *reinterpret_cast<const bf16x8*>(Xq + 32 + 8 * lg);
  const uint16_t* Xk = K + (head * s.T + tc) * kHeadDim;
  bf16x8 y0 = x0, y1 = x1;
  if (CAUSAL) {
    y0 = *reinterpret_cast<const bf16x8*>(Xk + 8 * lg);
    y1 = *reinterpret_cast<const bf16x8*>(Xk + 32 + 8 * lg);
  }
  // Nothing but padding: no scores, no columns.  (Decided behind the first loads, whose latency the sequence's length would
  // otherwise add to.  B = 8, T = 2000, padded by 0-25 %: 157 -> 136 us.)
  if (wg_r0 >= len) {
    lds_loads_done();
    const int64_t row = head * s.T + wg_r0, rows = min(64, s.T - wg_r0);
    if (A_hat && !s.cand_only)
      for (int64_t x = tid; x < rows * s.K; x += 256) A_hat[row * s.K + x] = 0.f;
    const int32_t kw = (s.K + 31) / 32;
    if (mbits)
      for (int64_t x = tid; x < rows * kw; x += 256) mbits[row * kw + x] = 0u;
    return;
  }
  // Prefix planes of the wave's tile inside its 128-key block (its column, if narrower): 3 m
  // halfwords, contiguous; lane l takes 16-byte pieces l and l + 64.
  bool tile_planes = false;
  // Any width: the sum of the rounded features of the column's keys before the wave's tile comes as m
  // fp32 values; each lane splits its share into the planes.
  int32_t own0 = 0;  // first key of the column the wave's first row lies in
  if (CAUSAL && ANYW) {
    own0 = __builtin_amdgcn_readfirstlane(column_start(cg, col_of(min(r0, s.T - 1))));
    tile_planes = r0 < s.T && own0 < r0;
  } else if (CAUSAL && WLOG >= 5) {
    const int tl = min(wl, 7) - 4;  // log2(tiles per prefix group)
    tile_planes = r0 < s.T && ((r0 >> 4) & ((1 << tl) - 1)) != 0;  // wave-uniform
  }
  uint4 preg0 = {0u, 0u, 0u, 0u}, preg1 = preg0;
  constexpr int kPieceLen = m >= 256 ? 4 : m / 64;  // any width: features per lane
  float pw[kPieceLen];
  if (ANYW && tile_planes) {
    const float* psrc = reinterpret_cast<const float*>(pref) + (head * ((s.T + 15) >> 4) + (r0 >> 4)) * m + lane * kPieceLen;
#pragma unroll
    for (int q = 0; q < kPieceLen; ++q) pw[q] = psrc[q];
  } else if (tile_planes) {
    const uint4* psrc = reinterpret_cast<const uint4*>(pref + (head * (s.T >> 4) + (r0 >> 4)) * 3 * m);
    constexpr int kPieces = 3 * m / 8;
    if (lane < kPieces) preg0 = psrc[lane];
    if (lane + 64 < kPieces) preg1 = psrc[lane + 64];
  }
  // bidirectional: the same candidates for every row (taken here, while the rows are on their way)
  const int32_t ncnd_all = CAUSAL ? 0 : __builtin_amdgcn_readfirstlane(col_of(max(len - 1, 0)) + 1);
  lds_loads_done();
  __syncthreads();

  // this lane's pieces lg and lg + 4 (mod 8) of a row of W
  const int wat0 = lr * kHeadDim + 8 * (lg ^ (lr & 7)), wat1 = lr * kHeadDim + 8 * ((lg + 4) ^ (lr & 7));
  // ---- phi(Q) of this wave's 16 rows, as contraction fragments ----
  bf16x8 afrag[MC];
  // causal: phi(K) of the same 16 rows (the keys of the rows' own column inside the wave), taken in
  // the same pass over W's fragments, so that each is read from LDS once for both projections; a
  // key's features need no row shift and are rounded and packed tile by tile
  bf16x8 kfrag[CAUSAL ? MC : 1];
  {
    float nx = sumsq8(x0) + sumsq8(x1);
    nx += __shfl_xor(nx, 16, kWave);
    nx += __shfl_xor(nx, 32, kWave);
    floatx4 dots[2 * MC];
    if (CAUSAL) {
      float ny = sumsq8(y0) + sumsq8(y1);
      ny += __shfl_xor(ny, 16, kWave);
      ny += __shfl_xor(ny, 32, kWave);
      const float kbias = c_norm * ny;
#pragma unroll
      for (int kc = 0; kc < MC; ++kc) {
        float lo[4], hi[4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int ft = 2 * kc + h;
          const bf16x8 w0 = *reinterpret_cast<const bf16x8*>(Ws + ft * 16 * kHeadDim + wat0);
          const bf16x8 w1 = *reinterpret_cast<const bf16x8*>(Ws + ft * 16 * kHeadDim + wat1);
          floatx4 acc = {0.f, 0.f, 0.f, 0.f};
          acc = mfma16(w0, x0, acc);
          dots[ft] = mfma16(w1, x1, acc);
          floatx4 ka = {0.f, 0.f, 0.f, 0.f};
          ka = mfma16(w0, y0, ka);
          ka = mfma16(w1, y1, ka);
#pragma unroll
          for (int i = 0; i < 4; ++i) (h == 0 ? lo : hi)[i] = __builtin_amdgcn_exp2f(fmaf(c_dot, ka[i], -kbias));
        }
        kfrag[kc] = pack8(lo, hi);
        asm volatile("" : "+v"(kfrag[kc]));  // (now, not where it is used: sixteen values would wait in place of eight)
      }
    } else {
#pragma unroll
      for (int ft = 0; ft < 2 * MC; ++ft) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma16(*reinterpret_cast<const bf16x8*>(Ws + ft * 16 * kHeadDim + wat0), x0, acc);
        dots[ft] = mfma16(*reinterpret_cast<const bf16x8*>(Ws + ft * 16 * kHeadDim + wat1), x1, acc);
      }
    }
    float dmax = -INFINITY;
#pragma unroll
    for (int ft = 0; ft < 2 * MC; ++ft)
#pragma unroll
      for (int i = 0; i < 4; ++i) dmax = fmaxf(dmax, dots[ft][i]);
    dmax = fmaxf(dmax, __shfl_xor(dmax, 16, kWave));
    dmax = fmaxf(dmax, __shfl_xor(dmax, 32, kWave));
    // Largest exponent argument of the row (the map dot -> c_dot dot - bias is monotone), rounded up:
    // a power-of-two row scale, which commutes with the bf16 rounding.  Inactive rows get an
    // infinite shift, i.e. all-zero features.
    const float bias = c_norm * nx;
    const float shift = t < len ? ceilf(fmaf(c_dot, dmax, -bias)) : INFINITY;
    const float off = -(bias + shift);
#pragma unroll
    for (int kc = 0; kc < MC; ++kc) {
      float lo[4], hi[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lo[i] = __builtin_amdgcn_exp2f(fmaf(c_dot, dots[2 * kc][i], off));
        hi[i] = __builtin_amdgcn_exp2f(fmaf(c_dot, dots[2 * kc + 1][i], off));
      }
      afrag[kc] = pack8(lo, hi);
    }
  }
  // From here on every product is taken with the query rows as accumulator COLUMNS: lane l % 16 is
  // the query row, so a row of A_hat lives in the four lanes l % 16 + 16 q (16 values each per 64
  // columns) and every per-row reduction is two row-swap steps.
  __syncthreads();  // every wave is done with W
  int tid2 = tid;  // (what the stages need from here on is computed from here on: registers are short before)
  asm volatile("" : "+v"(tid2));
  const int sat0 = (tid2 & 15) * m + 8 * (((tid2 >> 4) & 3) ^ (tid2 & 7)), sat1 = sat0 ^ 32;
  if (nstages > 1) fetch_stage(1, tid2);
  if (ANYW && tile_planes) {
    uint16_t* pdst = &planes_s[wid * 3 * m + lane * kPieceLen];
#pragma unroll
    for (int q = 0; q < kPieceLen; ++q) {
      const uint16_t hi = f32_to_bf16(pw[q]);
      const float r1 = pw[q] - bf16_to_f32(hi);
      const uint16_t lo = f32_to_bf16(r1);
      pdst[q] = hi;
      pdst[m + q] = lo;
      pdst[2 * m + q] = f32_to_bf16(r1 - bf16_to_f32(lo));
    }
  } else if (tile_planes) {
    constexpr int kPieces = 3 * m / 8;
    uint4* pdst = reinterpret_cast<uint4*>(&planes_s[wid * 3 * m]);
    if (lane < kPieces) pdst[lane] = preg0;
    if (lane + 64 < kPieces) pdst[lane + 64] = preg1;
  }
  float diag = 0.f;
  if (CAUSAL) {
    // the row's own column: sum over keys j <= t of that column of phi(q_t) . phi(k_j).  Those
    // keys are the wave's own 16 rows (S = phi(Q) phi(K_own)^T with a lower-triangular, same-column
    // mask) and, for columns wider than 16, the 16-key tiles of the column before the wave.
    const int32_t own_t = ANYW ? column_start(cg, col_of(tc)) : 0;  // first key of the row's own column
    floatx4 sd = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < MC; ++kc) sd = mfma16(kfrag[kc], afrag[kc], sd);  // rows = keys 4 lg + i, col = query lr
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int rk = 4 * lg + i;  // key row within the wave; the query row within the wave is lr
      const bool ok = ANYW ? (rk <= lr && r0 + rk >= own_t)
                           : (rk <= lr) && (WLOG >= 4 || (rk >> WLOG) == (lr >> WLOG));
      sd[i] = ok ? sd[i] : 0.f;
    }
    // Earlier keys of the same column: every one of them precedes every row of the wave, so only
    // their sum matters.  It comes as three bf16 planes = operand rows 0..2 (the rest zero);
    // the sum over the 16 result rows below then adds the three partial dots to the
    // in-wave ones.  Two levels: tiles before this one inside its 128-key block (its column, if
    // narrower), and, for columns wider than that, the column's blocks before this one.
    if (WLOG >= 5 && r0 < s.T) {
      if (tile_planes) {
        const uint16_t* src = &planes_s[(wid * 3 + min(lr, 2)) * m + 8 * lg];
        // any width: only the rows of the wave's first column have keys before the tile
        floatx4 sp = ANYW ? floatx4{0.f, 0.f, 0.f, 0.f} : sd;
#pragma unroll
        for (int kc = 0; kc < MC; ++kc) {
          uint4 f = *reinterpret_cast<const uint4*>(src + 32 * kc);
          if (lr > 2) f = uint4{0u, 0u, 0u, 0u};
          sp = mfma16(__builtin_bit_cast(bf16x8, f), afrag[kc], sp);
        }
        if (ANYW) {
#pragma unroll
          for (int i = 0; i < 4; ++i) sd[i] += own_t == own0 ? sp[i] : 0.f;
        } else {
          sd = sp;
        }
      }
      if (!ANYW && wl > 7 && ((r0 >> 7) & ((1 << (wl - 7)) - 1)) != 0) {
        const uint16_t* src = bpref + ((head * (s.T >> 7) + (r0 >> 7)) * 3 + min(lr, 2)) * m + 8 * lg;
#pragma unroll
        for (int kc = 0; kc < MC; ++kc) {
          uint4 f = *reinterpret_cast<const uint4*>(src + 32 * kc);
          if (lr > 2) f = uint4{0u, 0u, 0u, 0u};
          sd = mfma16(__builtin_bit_cast(bf16x8, f), afrag[kc], sd);
        }
      }
    }
    diag = rows_sum((sd[0] + sd[1]) + (sd[2] + sd[3]));
  }

  // ---- A_hat tile = phi(Q) state^T, state streamed through LDS ----
  floatx4 acc[NCT];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) asm volatile("" : "=v"(acc[ct]));  // (anything: finish_rows sets the tiles that no stage reaches)
  const int32_t ncols_wave = CAUSAL ? __builtin_amdgcn_readfirstlane(min(s.K, col_of(min(r0 + 15, s.T - 1)) + 1)) : s.K;
#pragma unroll
  for (int st = 0; st < NCT * 16 / kColStage; ++st) {
    if (st < nstages) {
      if (st > 0 && st + 1 < nstages) fetch_stage(st + 1, tid2);
      if (r0 < s.T && st * kColStage < ncols_wave) {
#pragma unroll
        for (int h = 0; h < kColStage / 16; ++h) {
          const uint16_t* brow = stage_at(st) + 16 * h * m;
          floatx4 a4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kc = 0; kc < MC; ++kc)
            a4 = mfma16(*reinterpret_cast<const bf16x8*>(brow + 64 * (kc >> 1) + ((kc & 1) ? sat1 : sat0)), afrag[kc], a4);
          acc[st * (kColStage / 16) + h] = a4;
        }
      }
      lds_loads_done();
      __syncthreads();
    }
  }
  if (r0 >= s.T) return;  // no barrier below

  // ---- masking, the own column, normalisation, selection ----
  const int32_t trow = r0 + lr;
  const int32_t ncnd = trow < len ? (CAUSAL ? col_of(min(trow, len - 1)) + 1 : ncnd_all) : 0;
  const bool act_all = r0 + 15 < len;  // wave-uniform
  const int32_t ct_free = act_all ? (CAUSAL ? __builtin_amdgcn_readfirstlane(col_of(r0)) : ncnd_all - 1) >> 4 : 0;
  finish_rows<CAUSAL, NCT>(s, acc, head, trow, ncnd, ct_free, ncols_wave, diag, lg, A_hat, mbits);
}

// ------------------------------------------------------------------------------------------
// query side, bidirectional, one column of 65 to 128 per row (k^ = 1, m <= 128), every row active: with no
// search to do, what is left of a row is two contractions and a maximum.  W and a head's whole state fit LDS
// together (53 KB for m = K = 128), so a block stages them once per head and its waves take 32 rows after 32
// rows with no barrier in between (the kernel above stages W per 64 rows and steps the state through LDS
// behind four barriers).  Two blocks of eight waves per CU, each with an equal share of all heads' tiles.  The winner of
// a row is its largest raw score: scaling by the row's sum can only make scores equal that are within a few units in the
// last place of each other, and a wave that holds such a row, or scores outside the middle of fp32's range, scales them
// and lets the lowest of the equal columns win, as the kernel above does (which adds up a row's scores in another order, so
// that scores a unit in the last place apart may be equal there and not here).  With that, and without a test per column, 32
// rows take 540 vector instructions (1110 before, most of them tests and the scalars they spilled); with 32 rows per wave an
// operand read from LDS serves twice the rows it does in tiles of 16 (48 KB each, 70 us of LDS time per launch).  Bound:
// vector pipe 62 % and matrix pipe 38 % busy at the 1.9 GHz the chip keeps here, one after the other.  B = 1, H = 12,
// T = 131072, m = K = 128: 152 -> 102 us (2.0 TB/s), the whole forward 303 -> 265.  1024 to 4096 blocks, or six or
// twelve waves to a block: the same or slower.  The search for k^ > 1 wants more waves than stay resident here, shares of
// sequences of different lengths are unequal, and K <= 64 needs no steps to begin with.
// SCORES: the scores leave as well, held in registers (174; one block per CU) and written through LDS in whole lines.  Bound:
// those writes (805 MB, 4.3 TB/s with the reads).  sea_estimate, us, with three passes over the contraction and four bytes a
// store / 16 bytes a store from one pass / so: 12 heads of 131072 rows, m = K = 128 590 / 338 / 276, m = 64, K = 100
// 600 / 366 / 335, 12 of 32768 154 / 88 / 78, 16 of 8192 55 / 34 / 27, of 8200, K = 65 56 / 58 / 43, 32 of 16384, m = 64
// 195 / 122 / 92; the kernel above 345, 289, 96, 28, 46, 100.
// ------------------------------------------------------------------------------------------
constexpr int kBidirWaves = 8, kBidirBlocks = 512;  // two blocks per CU (one where the scores are written)
constexpr int kPlaceRow = 68;  // floats per row of 64 scores on their way out: sixteen rows on distinct banks
__device__ __forceinline__ floatx16 mfma32(bf16x8 a, bf16x8 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
template <int MC, int NCT, bool SCORES>
__global__ __launch_bounds__(64 * kBidirWaves, SCORES ? 2 : 4) void estimate_rows_bidir_kernel(Shape s, const uint16_t* __restrict__ Q,
                                                                                  const uint16_t* __restrict__ W,
                                                                                  const uint16_t* __restrict__ state,
                                                                                  float* __restrict__ A_hat,
                                                                                  uint32_t* __restrict__ mbits,
                                                                                  int32_t* __restrict__ counts, float c_dot,
                                                                                  float c_norm, Columns cg) {
  constexpr int m = 32 * MC, kThreads = 64 * kBidirWaves;
  constexpr int kTiles = NCT / 2;      // of 32 columns
  constexpr int kPieces = m / 8;       // 16-byte pieces of a state row
  static_assert(NCT == 8, "a lane's scores are two mask words");
  // Rows end in a 16-byte pad: the sixteen lanes that an LDS read serves at a time (one piece of rows that differ mod 16)
  // hit distinct banks.  Piece 2 ks + g of a state row, the eight features 32 (ks / 2) + 16 (e / 4) + 8 (ks % 2) + 4 g + e % 4,
  // is the operand of lane half g in contraction step ks: registers 4 (ks % 2) + 8 (e / 4) + e % 4 of a feature tile hold the
  // same ones.  Two steps add up in the order of one 16x16x32 product, so scores are those of the kernel above, bit for bit.
  constexpr int kSRow = m + 8;
  extern __shared__ __attribute__((aligned(16))) uint16_t rows_lds[];
  uint16_t* const Ws = rows_lds;              // [m][kWRow]
  uint16_t* const Ss = rows_lds + m * kWRow;  // [16 NCT][kSRow]
  float* const place = reinterpret_cast<float*>(Ss + 16 * NCT * kSRow) + (threadIdx.x >> 6) * 32 * kPlaceRow;  // (SCORES)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, g = lane >> 5;
  // this block's share of all heads' 32-row tiles, in order: [lo, hi)
  const uint32_t tiles = (s.T + 31) / 32;
  const uint64_t all = static_cast<uint64_t>(tiles) * s.N;
  const uint32_t lb = xcd_contiguous(blockIdx.x, gridDim.x);
  const uint32_t lo = static_cast<uint32_t>(all * lb / gridDim.x), hi = static_cast<uint32_t>(all * (lb + 1) / gridDim.x);

  // Rows of the head in hand per column, added to the layer's counters when the head changes: the attention that groups rows by
  // column needs no pass over the mask for them (12 heads of 131072 rows: 9.7 us, this kernel the same, though at m = 128 four of its
  // registers are kept in memory around the inner loop for it; the layer 263.0 -> 256.6).
  __shared__ int32_t taken[16 * NCT];
  if (tid < 16 * NCT) taken[tid] = 0;
  auto hand_in = [&](uint32_t head) {
    if (counts && tid < s.K && taken[tid] != 0) atomicAdd(&counts[static_cast<int64_t>(head) * s.K + tid], taken[tid]);
    if (tid < 16 * NCT) taken[tid] = 0;
  };
  for (int v = tid; v < m * 8; v += kThreads)
    *reinterpret_cast<uint4*>(Ws + (v >> 3) * kWRow + 8 * (v & 7)) = *reinterpret_cast<const uint4*>(W + 8 * v);
  const int32_t ncnd = column_of(cg, s.T - 1) + 1;  // every column that holds a key is a candidate of every row
  const uint16_t* const wrow = Ws + lr * kWRow + 8 * g;
  const uint16_t* const srow = Ss + lr * kSRow + 8 * g;

  for (uint32_t first = lo; first < hi;) {
    const uint32_t head = first / tiles;
    const uint32_t end = min(hi, (head + 1) * tiles);
    if (first != lo) {
      __syncthreads();  // every wave is done with the last head's state
      hand_in(head - 1);
    }
    const uint16_t* sh = state + head * static_cast<int64_t>(s.K) * m;
    for (int v = tid; v < 16 * NCT * kPieces; v += kThreads) {
      const int col = v / kPieces, p = v % kPieces;  // (columns that hold no key score zero)
      uint4 x = {0u, 0u, 0u, 0u};
      if (col < ncnd) x = *reinterpret_cast<const uint4*>(sh + static_cast<int64_t>(col) * m + 8 * p);
      *reinterpret_cast<uint4*>(Ss + col * kSRow + 8 * p) = x;
    }
    __syncthreads();

    bf16x8 x[4];  // the next rows on their way
    auto request = [&](uint32_t tile) {
      const uint16_t* X = Q + (static_cast<int64_t>(head) * s.T + min(static_cast<int32_t>(tile - head * tiles) * 32 + lr, s.T - 1)) * kHeadDim + 8 * g;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) x[ks] = *reinterpret_cast<const bf16x8*>(X + 16 * ks);
    };
    if (first + wid < end) request(first + wid);
    for (uint32_t tile = first + wid; tile < end; tile += kBidirWaves) {
      asm volatile("" ::: "memory");  // (operands are read from LDS where they are used, not ahead of the loop into spilled registers)
      const int32_t trow = static_cast<int32_t>(tile - head * tiles) * 32 + lr;
      const float n02 = sumsq8(x[0]) + sumsq8(x[2]), n13 = sumsq8(x[1]) + sumsq8(x[3]);
      const float nx = (n02 + __shfl_xor(n02, 32, kWave)) + (n13 + __shfl_xor(n13, 32, kWave));
      floatx16 dots[MC];
      float dmax = -INFINITY;
#pragma unroll
      for (int ft = 0; ft < MC; ++ft) {
        dots[ft] = floatx16{};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          dots[ft] = mfma32(*reinterpret_cast<const bf16x8*>(wrow + 32 * ft * kWRow + 16 * ks), x[ks], dots[ft]);
      }
#pragma unroll
      for (int ft = 0; ft < MC; ++ft)
#pragma unroll
        for (int i = 0; i < 16; ++i) dmax = fmaxf(dmax, dots[ft][i]);
      dmax = fmaxf(dmax, __shfl_xor(dmax, 32, kWave));
      const float bias = c_norm * nx;
      const float off = -(bias + ceilf(fmaf(c_dot, dmax, -bias)));  // (rows past T repeat the last one)
      bf16x8 afrag[2 * MC];
#pragma unroll
      for (int ft = 0; ft < MC; ++ft)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          float a[4], b[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            a[i] = __builtin_amdgcn_exp2f(fmaf(c_dot, dots[ft][4 * j + i], off));
            b[i] = __builtin_amdgcn_exp2f(fmaf(c_dot, dots[ft][8 + 4 * j + i], off));
          }
          afrag[2 * ft + j] = pack8(a, b);
        }
      if (tile + kBidirWaves < end) request(tile + kBidirWaves);
      // scores of N x 32 columns from 32 ct on, register i: row trow, column 32 ct + 8 (i / 4) + 4 g + i % 4.  Operands are on
      // their way for four products (left alone, the compiler reads each into the register of the one before it and waits).
      auto scores = [&](int ct, auto& acc) {
        constexpr int N = sizeof(acc) / sizeof(floatx16), kSteps = 2 * MC, kAhead = 4;
        const uint16_t* from = srow + 32 * ct * kSRow;
        auto operand = [&](int u) { return *reinterpret_cast<const bf16x8*>(from + 32 * (u / kSteps) * kSRow + 16 * (u % kSteps)); };
        bf16x8 f[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) f[u] = operand(u);
#pragma unroll
        for (int u = 0; u < N * kSteps; ++u) {
          asm volatile("" ::: "memory");
          acc[u / kSteps] = mfma32(f[u % kAhead], afrag[u % kSteps], u % kSteps ? acc[u / kSteps] : floatx16{});
          if (u + kAhead < N * kSteps) f[u % kAhead] = operand(u + kAhead);
        }
      };
      uint32_t marks[2];
      if constexpr (SCORES) {
        // all of the row's scores, scaled and marked as below, and to memory in whole lines: 64 columns of the wave's rows at a time
        // through LDS
        floatx16 sc[kTiles];
        scores(0, sc);
        float r = 0.f;
#pragma unroll
        for (int ct = 0; ct < kTiles; ++ct)
#pragma unroll
          for (int i = 0; i < 16; ++i) r += sc[ct][i];
        r += __shfl_xor(r, 32, kWave);
        const float ninv = r > 0.f ? -1.f / r : -0.f;
#pragma unroll
        for (int ct = 0; ct < kTiles; ++ct)
#pragma unroll
          for (int i = 0; i < 16; ++i) sc[ct][i] *= ninv;
        const int32_t row0 = static_cast<int32_t>(tile - head * tiles) * 32;
        float* const out = A_hat + (static_cast<int64_t>(head) * s.T + row0) * s.K;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int q = 0; q < 8; ++q) {  // registers 4 (q % 4) .. of a tile: columns 8 q + 4 g .. of the 64
            const floatx16 a = sc[2 * h + (q >> 2)];
            const int j = 4 * (q & 3);
            *reinterpret_cast<float4*>(place + lr * kPlaceRow + 8 * q + 4 * g) = make_float4(-a[j], -a[j + 1], -a[j + 2], -a[j + 3]);
          }
          __builtin_amdgcn_wave_barrier();
          if ((s.K & 3) == 0) {
            const int32_t c = 64 * h + 4 * (lane & 15);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              const int32_t row = 4 * q + (lane >> 4);
              const float4 v = *reinterpret_cast<const float4*>(place + row * kPlaceRow + 4 * (lane & 15));
              if (row0 + row < s.T && c < s.K) *reinterpret_cast<float4*>(out + static_cast<int64_t>(row) * s.K + c) = v;
            }
          } else {
            const int32_t c = 64 * h + lane;
#pragma unroll 8
            for (int row = 0; row < 32; ++row) {
              const float v = place[row * kPlaceRow + lane];
              if (row0 + row < s.T && c < s.K) out[static_cast<int64_t>(row) * s.K + c] = v;
            }
          }
          __builtin_amdgcn_wave_barrier();
        }
        if (!mbits) continue;
        uint32_t top = 0u;
#pragma unroll
        for (int ct = 0; ct < kTiles; ++ct)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            if (32 * ct + 8 * (i >> 2) + 4 * g + (i & 3) >= ncnd) sc[ct][i] = __uint_as_float(0x40000000u);
            top = max(top, __float_as_uint(sc[ct][i]));
          }
        const auto o = __builtin_amdgcn_permlane32_swap(top, top, false, false);
        top = max(o[0], o[1]);
#pragma unroll
        for (int h = 0; h < 2; ++h) marks[h] = mark_at_least(sc[2 * h], top, mark_at_least(sc[2 * h + 1], top, 0u));
      } else {
        // Half of the columns at a time (all of them would leave no registers to read operands ahead): the lane's largest
        // (scores are not negative, their bit patterns have their order, NaN above all), and which ones are within four units
        // in the last place of it.
        uint32_t most[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          floatx16 ab[2];
          scores(2 * h, ab);
          const floatx16 a = ab[0], b = ab[1];
          uint32_t mx0 = 0, mx1 = 0;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            mx0 = max(mx0, __float_as_uint(a[i]));
            mx1 = max(mx1, __float_as_uint(b[i]));
          }
          most[h] = max(mx0, mx1);
          marks[h] = mark_at_least(a, most[h] - 4u, mark_at_least(b, most[h] - 4u, 0u));
        }
        uint32_t top = max(most[0], most[1]);
        {
          const auto o = __builtin_amdgcn_permlane32_swap(top, top, false, false);
          top = max(o[0], o[1]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) marks[h] = most[h] >= top - 4u ? marks[h] : 0u;
        const uint32_t cnt = __popc(marks[0]) + __popc(marks[1]);
        const auto both = __builtin_amdgcn_permlane32_swap(cnt, cnt, false, false);
        // 2^-100 < largest < 2^100, and no other within 2^-22 of it
        const bool plain = both[0] + both[1] == 1u && top - 0x0d800000u < 0x71800000u - 0x0d800000u;
        if (__ballot(!plain) != 0ull) {
          float r = 0.f;
#pragma unroll 1
          for (int ct = 0; ct < kTiles; ++ct) {
            floatx16 a[1];
            scores(ct, a);
#pragma unroll
            for (int i = 0; i < 16; ++i) r += a[0][i];
          }
          r += __shfl_xor(r, 32, kWave);
          const float ninv = r > 0.f ? -1.f / r : -0.f;  // (as in finish_rows: the negated score is the key)
          top = 0u;
          marks[0] = marks[1] = 0u;
#pragma unroll 1
          for (int ct = 0; ct < kTiles; ++ct) {
            floatx16 one[1];
            scores(ct, one);
            floatx16 a = one[0];
            uint32_t mx = 0u;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int32_t c = 32 * ct + 8 * (i >> 2) + 4 * g + (i & 3);
              a[i] = c < ncnd ? a[i] * ninv : __uint_as_float(0x40000000u);
              mx = max(mx, __float_as_uint(a[i]));
            }
            const auto o = __builtin_amdgcn_permlane32_swap(mx, mx, false, false);
            mx = max(o[0], o[1]);
            if (mx > top) marks[0] = marks[1] = 0u;
            top = max(top, mx);
            const uint32_t w = mark_at_least(a, top, 0u) << (16 * (ct & 1));
            marks[0] |= ct < 2 ? w : 0u;
            marks[1] |= ct < 2 ? 0u : w;
          }
        }
      }
      // the lane's first marked column, and the row's
      const int32_t e = marks[0] ? __builtin_ctz(marks[0]) : 32 + __builtin_ctz(marks[1] | 0x80000000u);
      uint32_t col = 32 * (e >> 4) + 8 * ((e >> 2) & 3) + 4 * g + (e & 3);
      if ((marks[0] | marks[1]) == 0u) col = 0xffffu;
      const auto cc = __builtin_amdgcn_permlane32_swap(col, col, false, false);
      col = min(cc[0], cc[1]);
      if (counts && g == 0 && trow < s.T && col != 0xffffu) atomicAdd(&taken[col], 1);
      if (trow < s.T) {  // this lane's two words of the row
        const int32_t kw = (s.K + 31) >> 5;
        const uint32_t bit = 1u << (col & 31), at = col >> 5;
        uint32_t* mrow = mbits + (static_cast<int64_t>(head) * s.T + trow) * kw + 2 * g;
        const uint2 words = make_uint2(at == 2 * g ? bit : 0u, at == 2 * g + 1 ? bit : 0u);
        if (kw == 4) {
          *reinterpret_cast<uint2*>(mrow) = words;
        } else {
          mrow[0] = words.x;
          if (g == 0) mrow[1] = words.y;
        }
      }
    }
    first = end;
  }
  if (counts) {
    __syncthreads();
    if (lo < hi) hand_in((hi - 1) / tiles);
  }
}

int wlog_of(const Shape& s) {
  if (s.T % s.K != 0) return -1;
  const int32_t w = s.T / s.K;
  if ((w & (w - 1)) != 0) return -1;
  int l = 0;
  while ((1 << l) < w) ++l;
  return l;
}

}  // namespace

bool estimate_fused_supported(const Shape& s) {
  if (s.geometry != 0 || s.T > (1 << 24) || wlog_of(s) > 20) return false;
  if (s.m != 64 && s.m != 128 && s.m != 256) return false;
  if (s.K > 256) return false;
  return true;
}

namespace {
size_t up256(size_t b) { return (b + 255) & ~size_t(255); }
struct FusedWs {
  size_t state, pref, bsum_u, bsum_r, bpref, total;
};
// state | tile prefixes (causal; columns > 16: three bf16 planes; columns of any width: fp32) | for columns > 128: block sums, rounded block sums
// and block prefixes (the last two causal only)
FusedWs fused_layout(const Shape& s) {
  const int wl = wlog_of(s);
  const size_t N = static_cast<size_t>(s.N);
  FusedWs f{};
  size_t off = 0;
  f.state = off; off += up256(N * s.K * s.m * 2);
  f.pref = off;
  if (s.causal && wl < 0) off += up256(N * ((s.T + 15) / 16) * s.m * 4);
  if (s.causal && wl > 4) off += up256(N * (s.T / 16) * 3 * s.m * 2);
  f.bsum_u = off; if (wl > 7) off += up256(N * (s.T / 128) * s.m * 4);
  f.bsum_r = off; if (wl > 7 && s.causal) off += up256(N * (s.T / 128) * s.m * 4);
  f.bpref = off;  if (wl > 7 && s.causal) off += up256(N * (s.T / 128) * 3 * s.m * 2);
  f.total = off;
  return f;
}
}  // namespace

size_t estimate_fused_workspace(const Shape& s) { return fused_layout(s).total; }

namespace {

struct FusedPtrs {
  uint16_t* state;
  uint16_t* pref;
  float* bsum_u;
  float* bsum_r;
  uint16_t* bpref;
  int32_t* counts;    // rows per column (or nullptr): zeroed by the key kernels
  uint32_t ncounts;
};

template <int MC, int WLOG, int NCT>
void launch_rows(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* W, float* A_hat,
                 uint32_t* mbits, const FusedPtrs& f, float c_dot, float c_norm, int32_t gh, dim3 grid,
                 hipStream_t st) {
  if (s.causal)
    hipLaunchKernelGGL((estimate_rows_kernel<MC, true, WLOG, NCT>), grid, dim3(256), 0, st, s, Q, K, W, f.state,
                       f.pref, f.bpref, A_hat, mbits, c_dot, c_norm, gh, columns_of(s.T, s.K));
  else  // (a bidirectional row has no column of its own: any width will do)
    hipLaunchKernelGGL((estimate_rows_kernel<MC, false, kAnyWidth, NCT>), grid, dim3(256), 0, st, s, Q, K, W, f.state,
                       f.pref, f.bpref, A_hat, mbits, c_dot, c_norm, gh, columns_of(s.T, s.K));
}

template <int MC, int WLOG>
void launch_key(const Shape& s, const uint16_t* K, const uint16_t* W, const FusedPtrs& f, float c_dot,
                float c_norm, hipStream_t st) {
  constexpr int kKeyWaves = key_waves(WLOG);
  const uint32_t ktiles = (s.T + 16 * kKeyWaves - 1) / (16 * kKeyWaves);
  // Tiles per block: as many as make one round of blocks where a block is short (eight blocks of four waves on a CU, three of
  // eight: 12 heads of 131072 keys 60.6 -> 55.8 us against eight blocks per CU, 384 of 512 12.3 -> 11.4), two rounds and more
  // at m = 256, where the rows kernel then starts under the last blocks (32 heads of 32768 keys 80.1 against 83.4 us in
  // one round, 256 of 2048 40.9 / 42.7).
  constexpr int kPerCu = kKeyWaves == 8 && MC < 8 ? 3 : 8;
  const int64_t all = static_cast<int64_t>(s.N) * ktiles;
  const int32_t iters = static_cast<int32_t>(std::min<int64_t>(32, (all + 256 * kPerCu - 1) / (256 * kPerCu)));
  const uint32_t bph = (ktiles + iters - 1) / iters;
  hipLaunchKernelGGL((key_state_kernel<MC, WLOG>), dim3(static_cast<uint32_t>(s.N) * bph), dim3(64 * kKeyWaves), 0, st,
                     s, K, W, f.state, f.pref, f.bsum_u, f.bsum_r, c_dot, c_norm, iters, f.counts, f.ncounts);
}

// columns per block: about 256 keys, so that the 16 columns a product has room for are used where columns
// are narrow and wide columns still give many blocks
template <int MC>
void launch_key_columns(const Shape& s, const uint16_t* K, const uint16_t* W, const FusedPtrs& f, float c_dot,
                        float c_norm, hipStream_t st) {
  const int32_t w0 = s.T / s.K;
  const int32_t G = std::min(16, std::max(1, 256 / w0));
  const dim3 grid(static_cast<uint32_t>(s.N) * ((s.K + G - 1) / G));
  float* pref = reinterpret_cast<float*>(f.pref);
  const Columns cg = columns_of(s.T, s.K);
#define SEA_KEY_COLUMNS(CAUSAL_) \
  hipLaunchKernelGGL((key_columns_kernel<MC, CAUSAL_>), grid, dim3(256), 0, st, s, cg, K, W, f.state, pref, c_dot, c_norm, G, f.counts, \
                     f.ncounts)
  if (s.causal) SEA_KEY_COLUMNS(true);
  else SEA_KEY_COLUMNS(false);
#undef SEA_KEY_COLUMNS
}

template <int MC, int NCT, bool SCORES>
void launch_bidir(const Shape& s, const uint16_t* Q, const uint16_t* W, float* A_hat, uint32_t* mbits, const FusedPtrs& f,
                  float c_dot, float c_norm, hipStream_t st) {
  constexpr size_t lds = (static_cast<size_t>(32 * MC) * kWRow + static_cast<size_t>(16) * NCT * (32 * MC + 8)) * 2 +
                         (SCORES ? kBidirWaves * 32 * kPlaceRow * sizeof(float) : 0);
  static_assert(SCORES || lds <= (64u << 10), "no larger LDS has to be asked for");
  if (SCORES && hipFuncSetAttribute(reinterpret_cast<const void*>(&estimate_rows_bidir_kernel<MC, NCT, SCORES>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
    return;  // (the caller asks for the error)
  hipLaunchKernelGGL((estimate_rows_bidir_kernel<MC, NCT, SCORES>), dim3(SCORES ? kBidirBlocks / 2 : kBidirBlocks),
                     dim3(64 * kBidirWaves), lds, st, s, Q, W, f.state, A_hat, mbits, f.counts, c_dot, c_norm, columns_of(s.T, s.K));
}

template <int MC, int WLOG>
void launch_rows_k(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* W, float* A_hat,
                   uint32_t* mbits, const FusedPtrs& f, float c_dot, float c_norm, hipStream_t st) {
  const uint32_t tiles = (s.T + 63) / 64;
  const dim3 grid(static_cast<uint32_t>(s.N) * tiles);
  // heads whose state (K x m bf16 each) shares an XCD's L2 at one time: 2 MB worth
  const int64_t per_xcd = std::max<int64_t>(1, (int64_t(2) << 20) / (static_cast<int64_t>(s.K) * s.m * 2));
  const int32_t gh = static_cast<int32_t>(std::min<int64_t>(s.N, 8 * per_xcd));
  if (s.K <= 64)
    launch_rows<MC, WLOG, 4>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, gh, grid, st);
  else if (s.K <= 128)
    launch_rows<MC, WLOG, 8>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, gh, grid, st);
  else
    launch_rows<MC, WLOG, 16>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, gh, grid, st);
}

// Layers of the kernel for one column per row: from two groups of 128 rows per resident block on.  Layer with the other kernel /
// this one, us, m = K = 128: 32768 rows 26.1 / 27.0, 65536 32.7 / 31.3, 98304 40.0 / 38.7, 131072 45.6 / 42.2, 262144 68.4 / 63.7;
// K = 96 65536 89.5 / 88.8; m = 64, K = 100 65536 80.7 / 79.1.  (By these the line could lie at half of that.  It stays where it
// is: the two kernels add a row's scores up in different orders, so layers that change sides may take another of two columns
// whose scores are a unit in the last place apart.)
bool one_column_rows(const Shape& s) {
  const int64_t groups = (s.T + 16 * kBidirWaves - 1) / (16 * kBidirWaves) * s.N;
  return s.m <= 128 && !s.causal && !s.seq_len && s.k_hat == 1 && s.K > 64 && s.K <= 128 && groups >= 2 * kBidirBlocks && groups < (1ll << 28);
}

template <int MC>
void launch_w(const Shape& s, int wl, const uint16_t* Q, const uint16_t* K, const uint16_t* W, float* A_hat,
              uint32_t* mbits, const FusedPtrs& f, float c_dot, float c_norm, hipStream_t st) {
  {
    StageScope scope(SEA_STAGE_STATE, st);
    switch (wl) {
      case -1: launch_key_columns<MC>(s, K, W, f, c_dot, c_norm, st); break;
      case 0: launch_key<MC, 0>(s, K, W, f, c_dot, c_norm, st); break;
      case 1: launch_key<MC, 1>(s, K, W, f, c_dot, c_norm, st); break;
      case 2: launch_key<MC, 2>(s, K, W, f, c_dot, c_norm, st); break;
      case 3: launch_key<MC, 3>(s, K, W, f, c_dot, c_norm, st); break;
      case 4: launch_key<MC, 4>(s, K, W, f, c_dot, c_norm, st); break;
      case 5: launch_key<MC, 5>(s, K, W, f, c_dot, c_norm, st); break;
      case 6: launch_key<MC, 6>(s, K, W, f, c_dot, c_norm, st); break;
      default: launch_key<MC, 7>(s, K, W, f, c_dot, c_norm, st); break;
    }
    if (wl > 7)
      hipLaunchKernelGGL(wide_columns_kernel, dim3(static_cast<uint32_t>(s.N) * s.K), dim3(256), 0, st, s,
                         f.bsum_u, f.bsum_r, f.state, f.bpref, 1 << (wl - 7));
  }
  StageScope scope(SEA_STAGE_CONTRACT, st);
  if constexpr (MC <= 4) {
    if (one_column_rows(s))
      return A_hat ? launch_bidir<MC, 8, true>(s, Q, W, A_hat, mbits, f, c_dot, c_norm, st)
                   : launch_bidir<MC, 8, false>(s, Q, W, nullptr, mbits, f, c_dot, c_norm, st);
  }
  switch (wl) {
    case -1: launch_rows_k<MC, kAnyWidth>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
    case 0: launch_rows_k<MC, 0>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
    case 1: launch_rows_k<MC, 1>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
    case 2: launch_rows_k<MC, 2>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
    case 3: launch_rows_k<MC, 3>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
    case 4: launch_rows_k<MC, 4>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
    default: launch_rows_k<MC, 5>(s, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
  }
}

}  // namespace

BucketCounts estimate_counts_columns(const Shape& s) {
  if (!estimate_fused_supported(s)) return BucketCounts::none;
  return one_column_rows(s) ? BucketCounts::counted : BucketCounts::zeroed;
}

hipError_t launch_estimate_fused(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* W,
                                 float* A_hat, uint32_t* mbits, void* ws, hipStream_t st, int32_t* counts) {
  if (!estimate_fused_supported(s)) return hipErrorNotSupported;
  const int wl = wlog_of(s);
  const FusedWs lay = fused_layout(s);
  char* base = static_cast<char*>(ws);
  FusedPtrs f{};
  f.state = reinterpret_cast<uint16_t*>(base + lay.state);
  if (s.causal && (wl < 0 || wl > 4)) f.pref = reinterpret_cast<uint16_t*>(base + lay.pref);
  if (wl > 7) {
    f.bsum_u = reinterpret_cast<float*>(base + lay.bsum_u);
    if (s.causal) {
      f.bsum_r = reinterpret_cast<float*>(base + lay.bsum_r);
      f.bpref = reinterpret_cast<uint16_t*>(base + lay.bpref);
    }
  }
  if (counts) {
    f.counts = counts;
    f.ncounts = static_cast<uint32_t>(static_cast<int64_t>(s.N) * s.K);
  }
  const double l2e = 1.4426950408889634;
  const float c_dot = static_cast<float>(l2e * sqrt(static_cast<double>(s.scale)));
  const float c_norm = static_cast<float>(l2e * 0.5 * static_cast<double>(s.scale));
  switch (s.m) {
    case 64: launch_w<2>(s, wl, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
    case 128: launch_w<4>(s, wl, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
    default: launch_w<8>(s, wl, Q, K, W, A_hat, mbits, f, c_dot, c_norm, st); break;
  }
  return hipGetLastError();
}

}  // namespace sea
