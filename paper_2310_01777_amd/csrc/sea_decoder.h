// Device helpers and launchers shared by the decoder's translation units (bf16 operands of
// v_mfma_f32_16x16x32_bf16: lane l holds row / column l % 16 and the contraction elements
// 8 (l / 16) .. + 7 of a 32-wide step).
#pragma once
#include <algorithm>

#include "sea_internal.h"

namespace sea {

#if defined(__HIPCC__)
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 mfma16(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 load8(const uint16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }
__device__ __forceinline__ bf16x8 zero8() {
  const uint4 z = {0u, 0u, 0u, 0u};
  return __builtin_bit_cast(bf16x8, z);
}
__device__ __forceinline__ bf16x8 pack8(floatx4 lo, floatx4 hi) {
  uint4 u;
  u.x = pack_bf16(lo[0], lo[1]);
  u.y = pack_bf16(lo[2], lo[3]);
  u.z = pack_bf16(hi[0], hi[1]);
  u.w = pack_bf16(hi[2], hi[3]);
  return __builtin_bit_cast(bf16x8, u);
}
__device__ __forceinline__ floatx4 relu4(floatx4 x) {
  return floatx4{fmaxf(x[0], 0.f), fmaxf(x[1], 0.f), fmaxf(x[2], 0.f), fmaxf(x[3], 0.f)};
}
#endif

// C_perf = FAVOR+(Q, K, [V_I; V]), normalised: [N][T][128] bf16; `state` is dec_linattn_state_bytes() of scratch
size_t dec_linattn_state_bytes(const Shape& s);
hipError_t launch_dec_linattn(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* V, const uint16_t* W,
                              uint16_t* Cp, void* state, float c_dot, float c_norm, hipStream_t st);
// mu, nu and the scalers on rows [C_perf; V]: the CNN's input image [B][T][K / 2][4 H], s_mix, s_prob [B][H][T]
hipError_t launch_dec_mlp(const Shape& s, const sea_decoder_weights& wt, const uint16_t* Cp, const uint16_t* V,
                          uint16_t* img, float* s_mix, float* s_prob, hipStream_t st);

// a 3x3 layer on a channels-last image [B][Tin][X][Cin], weights [Cout][3][3][Cin]; the columns keep their
// number, rows i stride_t - pad_top .. + 2 make output row i, zeros outside
struct DecConv {
  const uint16_t* in;
  const uint16_t* w;
  const float* bias;
  int32_t B, Tin, X, Cin, Tout, Cout, stride_t, pad_top;
};
// conv 1 and 2 with ReLU, bf16 [B][Tout][X][Cout]
hipError_t launch_dec_conv(const DecConv& c, uint16_t* out, hipStream_t st);
// conv 3 on the image resized (nearest) to Tv x 2 X, and the softmax of its rows: A [B][Cout][Tout][2 X] fp32,
// rows at or past seq_len zero
hipError_t launch_dec_conv_softmax(const DecConv& c, int32_t Tv, float* A, const int32_t* seq_len, hipStream_t st);
// all three layers of a causal image [B][T][X][4 H] in one launch; w, bias: the layers' in order
struct DecChain {
  const uint16_t* in;
  const uint16_t* w[3];
  const float* bias[3];
  int32_t B, T, X, H;
};
hipError_t launch_dec_chain(const DecChain& c, float* A, const int32_t* seq_len, hipStream_t st);

}  // namespace sea
