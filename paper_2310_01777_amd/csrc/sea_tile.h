// Device helpers shared by the tiled attention kernels (32x32x16 bf16 matrix products with one
// query per lane and half-wave, K and V steps staged through LDS).
#pragma once
#include "sea_internal.h"
#include "sea_lds.h"

namespace sea {

#if defined(__HIPCC__)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// 64-bit LDS read with the 16-bit transpose across each group of 16 lanes (ds_read_b64_tr_b16)
__device__ __forceinline__ bf16x4 lds_transpose4(const uint16_t* p) {
  const shortx4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) shortx4*)(p));
  return __builtin_bit_cast(bf16x4, r);
}

// combine a value with the one held by the same lane of the other 32-lane half of the wave
__device__ __forceinline__ float half_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// largest of a lane's sixteen scores, NaNs left out.  (Written as the instruction: behind a branch the compiler
// does not know the scores for results of arithmetic and quiets them one by one first.)
__device__ __forceinline__ float max3(float a, float b, float c) {
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ float max_of(const float (&y)[16]) {
  float a = max3(y[0], y[1], y[2]), b = max3(y[3], y[4], y[5]);
  a = max3(a, y[6], y[7]);
  b = max3(b, y[8], y[9]);
  a = max3(a, y[10], y[11]);
  b = max3(b, y[12], y[13]);
  a = max3(a, y[14], y[15]);
  return max3(a, b, b);
}

// Running reference of a streaming softmax, log2 units: the largest score met when it was last moved.  It stays until a
// score exceeds it by kRefSlack.  Any reference gives the same weights up to a factor that the row sum takes out again,
// so it has to keep sums and products in range: a row's largest weight lies between 1 and 2^8, so values down to the
// smallest normal number keep their bits in its products, and sums of 2^14 such weights times values of 2^104 stay
// finite.  And it should be a score: that key's weight, mostly the row's largest, is then 1 and not rounded.
// References further up are moved less often but cost both.  32 above, moved after a rise of 48: c4 at T = 32768 and c2
// 2 % faster, error against 64 bits 2 % larger (c2 1.83e-3 -> 1.87e-3, weights of bf16), values below 2^-94 lost bits and
// those from about 2^106 on overflowed; 8 above, moved after 16: 1 % faster, the same loss of precision.  Weights kept to
// 24 bits lose more, because the argument of exp2 is rounded to its own last bit (rms 2^-21.8 -> 2^-20.4 of a row).
constexpr float kRefSlack = 8.f;

// O^T += V^T P^T for one 32-key sub-chunk with weights p = 2^y held in fp32: a weight enters the bf16 product
// as the sum of three bf16 values, its rounded value, the rounded remainder and what then remains.  Eight
// significant bits each, to nearest, cover the 24 of an fp32 number, so the products are those of the fp32
// weights (two values, 16 bits, left an error of 2^-18 of an output row's values against 2^-24).  Register
// order of y: key slot 8 (i / 4) + 4 g + i % 4 of register i; av = V^T fragments in that order.  Returns the
// sum of the weights.
struct MinusOnes {
  bf16x2 lo, hi;  // {-1, 0}, {0, -1}
};
// (kept in scalar registers: written as constants, the first is encoded as the inline operand -1.0, which
// the dot product reads as the fp32 pattern = {0, -1})
__device__ __forceinline__ MinusOnes minus_ones() {
  uint32_t lo = 0x0000bf80u, hi = 0xbf800000u;
  asm volatile("" : "+s"(lo), "+s"(hi));
  return {__builtin_bit_cast(bf16x2, lo), __builtin_bit_cast(bf16x2, hi)};
}
__device__ __forceinline__ bf16x8 join_pairs(const bf16x2* p) {
  const bf16x4 lo = __builtin_shufflevector(p[0], p[1], 0, 1, 2, 3);
  const bf16x4 hi = __builtin_shufflevector(p[2], p[3], 0, 1, 2, 3);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ float add_weighted_rows(const float (&y)[16], const bf16x8 (&av)[2][2], const MinusOnes& minus,
                                                   floatx16 (&oacc)[2]) {
  float sum = 0.f;
#pragma unroll
  for (int c2 = 0; c2 < 2; ++c2) {
    bf16x2 part[3][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      floatx2 f = {__builtin_amdgcn_exp2f(y[8 * c2 + 2 * e]), __builtin_amdgcn_exp2f(y[8 * c2 + 2 * e + 1])};
      sum += f[0];
      sum += f[1];
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        part[n][e] = __builtin_convertvector(f, bf16x2);
        if (n < 2)
          f = floatx2{__builtin_amdgcn_fdot2_f32_bf16(part[n][e], minus.lo, f[0], false),
                      __builtin_amdgcn_fdot2_f32_bf16(part[n][e], minus.hi, f[1], false)};
      }
    }
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      const bf16x8 p = join_pairs(part[n]);
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[mt][c2], p, oacc[mt], 0, 0, 0);
    }
  }
  return sum;
}

// Rows of a wave (one per lane and half-wave, bit r = row r) whose sum or accumulators are not finite
__device__ __forceinline__ uint32_t rows_not_finite(float l, const floatx16 (&oacc)[2]) {
  float zero = 0.f * l;  // NaN if anything is not finite
#pragma unroll
  for (int i = 0; i < 16; ++i) zero = fmaf(0.f, oacc[0][i], fmaf(0.f, oacc[1][i], zero));
  const uint64_t lanes = __ballot(zero != 0.f);
  return static_cast<uint32_t>(lanes | (lanes >> 32));
}

__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(byte_off), 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// Place in the longest-first order of a causal launch's blocks.  Where the whole launch is resident at once
// (per_cu blocks on each of 256 CUs, dealt in turn) every other round of 256 runs backwards, eight at a time (a head
// stays on its XCD), so that the CU with the longest block of one round gets the shortest of the next.  In longer
// launches a CU takes its next block when it is done with one.  Attention stage, us without / with: H = 32, T = 2048,
// B = 2, K = 256 (1024 blocks) 66.8 / 60.2, H = 12, T = 8192, whole columns (768) 192 / 172; c2 (768) 42.4 / 42.3;
// columns of any width, T = 1701, 64 heads 98.3 / 89.9.
// Three rounds are not evened out by one that runs backwards (c2: 46 to 56 steps of 64 keys per CU), but an order that does
// even them out, 50 or 52 steps everywhere, gives nothing that can be told from the spread of runs: attention stage without /
// with, least of sixty, 768 blocks 46.1 / 45.7, 704 45.1 / 44.9, 640 44.2 / 43.9, 576 37.5 / 37.4, of 4096 rows 640 82.2 / 81.6;
// columns of any width 768 72.1 / 73.2, 704 69.8 / 69.7.
// (Blocks with nothing but padding have to keep their turn there: they walk their steps without products, which costs
// little.  Where they return at once, the blocks behind them land on other CUs: B = 2, H = 32, T = 2048 padded by 0-25 %, K = 256,
// 60 -> 63 us.  Longer launches, where the next block takes their place: padding_returns.)
__device__ __forceinline__ bool padding_returns(uint32_t grid, uint32_t per_cu, bool causal) { return !causal || grid > 256u * per_cu; }
__device__ __forceinline__ uint32_t dealt_in_turn(uint32_t block, uint32_t grid, uint32_t per_cu, bool causal) {
  if (!causal || grid > 256u * per_cu || ((block >> 8) & 1u) == 0u) return block;
  const uint32_t lo = block & ~255u, n8 = min(256u, grid - lo) >> 3, at8 = (block - lo) >> 3;
  return at8 < n8 ? lo + 8u * (n8 - 1u - at8) + (block & 7u) : block;
}

#endif  // __HIPCC__

// heads whose row tiles are dealt out together, from a list of U keys each
int32_t group_heads_for(const Shape& s, int64_t U);

// A lane's half of its row of a result (O^T accumulators times inv), 8 bytes at a time
__device__ __forceinline__ void store_row(uint16_t* row, const floatx16 (&oacc)[2], float inv) {
  const int g = (threadIdx.x >> 5) & 1;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      // regs 4 q4 .. 4 q4 + 3 <-> d = 32 mt + 8 q4 + 4 g + 0..3
      const floatx2 f01 = {oacc[mt][4 * q4] * inv, oacc[mt][4 * q4 + 1] * inv};
      const floatx2 f23 = {oacc[mt][4 * q4 + 2] * inv, oacc[mt][4 * q4 + 3] * inv};
      const bf16x2 h01 = __builtin_convertvector(f01, bf16x2), h23 = __builtin_convertvector(f23, bf16x2);
      *reinterpret_cast<bf16x4*>(row + 32 * mt + 8 * q4 + 4 * g) = __builtin_shufflevector(h01, h23, 0, 1, 2, 3);
    }
}

// Rows of a result that lie past the sequence's end, by all threads of a block
template <int THREADS>
__device__ __forceinline__ void zero_rows(uint16_t* to, int32_t rows) {
  for (int32_t x = threadIdx.x; x < rows * (kHeadDim / 8); x += THREADS) reinterpret_cast<uint4*>(to)[x] = make_uint4(0u, 0u, 0u, 0u);
}

// The 32 rows of a wave's result (O^T accumulators times inv, a row's factor) to memory as whole lines: through the
// wave's 4 KB of LDS at `place`, piece p of row r at slot p ^ (r & 7), then eight lanes of 16 bytes per row.  dest(r) is
// row r's place in memory, or nullptr; rows of the mask `marked` are written as all ones.  (With store_row, whose
// instructions each touch 32 lines, us per attention stage: c5 42 against 39.4, c2 44.4 / 43.9.)
template <typename F>
__device__ __forceinline__ void store_rows(uint16_t* place, const floatx16 (&oacc)[2], float inv, uint32_t marked, F&& dest) {
  const int lane = threadIdx.x & 63, ql = lane & 31, g = lane >> 5, row = lane >> 3, part = lane & 7;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      // regs 4 q4 .. 4 q4 + 3 <-> d = 32 mt + 8 q4 + 4 g + 0..3
      const floatx2 f01 = {oacc[mt][4 * q4] * inv, oacc[mt][4 * q4 + 1] * inv};
      const floatx2 f23 = {oacc[mt][4 * q4 + 2] * inv, oacc[mt][4 * q4 + 3] * inv};
      const bf16x2 h01 = __builtin_convertvector(f01, bf16x2), h23 = __builtin_convertvector(f23, bf16x2);
      *reinterpret_cast<bf16x4*>(place + ql * kHeadDim + 8 * ((4 * mt + q4) ^ (ql & 7)) + 4 * g) = __builtin_shufflevector(h01, h23, 0, 1, 2, 3);
    }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = 8 * j + row;
    uint4 v = *reinterpret_cast<const uint4*>(place + r * kHeadDim + 8 * (part ^ row));
    if ((marked >> r) & 1u) v = make_uint4(~0u, ~0u, ~0u, ~0u);
    uint16_t* const at = dest(r);
    if (at) *reinterpret_cast<uint4*>(at + 8 * part) = v;
  }
  __builtin_amdgcn_wave_barrier();
}

// Partial result of a set of waves (O^T accumulators, row sum, reference maximum or -inf) in LDS, LANES lanes a
// set, and its log-sum-exp merge into the registers of the set that goes on.
constexpr int kPartFloats = 34;
template <int LANES>
__device__ __forceinline__ void store_part(float* p, const floatx16 (&oacc)[2], float l, float m) {
#pragma unroll
  for (int i = 0; i < 32; ++i) p[LANES * i] = oacc[i >> 4][i & 15];
  p[LANES * 32] = l;
  p[LANES * 33] = m;
}
template <int LANES>
__device__ __forceinline__ void merge_part(const float* p, floatx16 (&oacc)[2], float& l, float& m) {
  const float m_other = p[LANES * 33], m_new = fmaxf(m, m_other);
  const float f0 = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - m_new);
  const float f1 = m_other == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_other - m_new);
  l = l * f0 + p[LANES * 32] * f1;
#pragma unroll
  for (int i = 0; i < 32; ++i) oacc[i >> 4][i & 15] = oacc[i >> 4][i & 15] * f0 + p[LANES * i] * f1;
  m = m_new;
}

}  // namespace sea
