// Column ranges of a sequence of T keys spread over K columns when K need not divide T: column c holds
// keys ceil(c T / K) .. ceil((c + 1) T / K) - 1.  With T = w0 K + rm its first key is
// c w0 + ceil(c rm / K), and c rm < K^2 <= 2^20 divides by K exactly in fp32.
#pragma once
#include "sea_internal.h"

namespace sea {

struct Columns {
  int32_t K, w0, rm;
  float invK;   // 1 / K
  float ratio;  // K / T
};
inline Columns columns_of(int32_t T, int32_t K) {
  Columns c{};
  c.K = K;
  c.w0 = T / K;
  c.rm = T % K;
  c.invK = 1.0f / static_cast<float>(K);
  c.ratio = static_cast<float>(static_cast<double>(K) / static_cast<double>(T));
  return c;
}

#if defined(__HIPCC__)
// floor(x / n) for 0 <= x < 2^21, inv = 1 / n rounded to fp32: x + 1/2 is at least 1 / (2 n) away from the
// next multiple of n (in quotients), and the fused product is off by less than x / n 2^-23 < 1 / (4 n)
__device__ __forceinline__ int32_t div_small(int32_t x, float inv) {
  return static_cast<int32_t>(fmaf(static_cast<float>(x), inv, 0.5f * inv));
}
__device__ __forceinline__ int32_t column_start(const Columns& g, int32_t c) {
  return c * g.w0 + div_small(c * g.rm + g.K - 1, g.invK);
}
// column of key j, 0 <= j < T <= 2^24: the fp32 product is off by less than one column, and the
// exact column starts decide
__device__ __forceinline__ int32_t column_of(const Columns& g, int32_t j) {
  int32_t c = static_cast<int32_t>(static_cast<float>(j) * g.ratio);
  if (column_start(g, c + 1) <= j) ++c;
  if (column_start(g, c) > j) --c;
  return c;
}
#endif

}  // namespace sea
