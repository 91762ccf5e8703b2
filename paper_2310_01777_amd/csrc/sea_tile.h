// Device helpers shared by the tiled attention kernels (32x32x16 bf16 matrix products with one
// query per lane and half-wave, K and V steps staged through LDS).
#pragma once
#include "sea_internal.h"

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

// raw buffer resource, word 3: 32-bit data format, no swizzle; loads past num_records return zero
constexpr int kBufferFlags = 0x00020000;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(byte_off), 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

#endif  // __HIPCC__

// heads whose keys and values (2 x U x 128 B each) share the L2s at one time
int32_t group_heads_for(int32_t N, int64_t U);

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
