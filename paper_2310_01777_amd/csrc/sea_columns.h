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

struct ColumnList {
  Columns cg;
  int32_t r;   // keys per column, 0 = whole columns
  float invr;  // 1 / r
  int32_t U;   // length of the list
};
// A selected column emits min(w, cap) of its w keys, and a cap between the two widths of a ragged split cannot
// occur: the cap is then reached in both.  div_small needs r (w + 1) < 2^21.
inline bool column_list_supported(const Shape& s) {
  if (s.geometry != 0 || s.T > (1 << 24)) return false;
  const int32_t w0 = s.T / s.K;
  return s.rep_cap > w0 || static_cast<int64_t>(s.rep_cap) * (w0 + 1) < (1 << 21);
}
inline ColumnList column_list(const Shape& s) {
  ColumnList g{};
  g.cg = columns_of(s.T, s.K);
  g.r = s.rep_cap > g.cg.w0 ? 0 : s.rep_cap;
  g.invr = g.r == 0 ? 0.f : 1.0f / static_cast<float>(g.r);
  g.U = g.r == 0 ? s.T : s.K * g.r;
  return g;
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

// The keys a head's rows can use, as one list ascending in position: all keys (r = 0: whole columns are
// emitted) or r keys start + floor(i w / r) of every column.
__device__ __forceinline__ int32_t entry_offset(const ColumnList& g, int32_t i, int32_t w) { return div_small(i * w, g.invr); }
__device__ __forceinline__ int32_t entry_pos(const ColumnList& g, int32_t c, int32_t i) {
  const int32_t s0 = column_start(g.cg, c), w = column_start(g.cg, c + 1) - s0;
  return s0 + entry_offset(g, i, w);
}
// number of list entries with position <= jmax
__device__ __forceinline__ int32_t list_count(const ColumnList& g, int32_t jmax) {
  if (jmax < 0) return 0;
  if (g.r == 0) return jmax + 1;
  const int32_t col = column_of(g.cg, jmax);
  const int32_t s0 = column_start(g.cg, col), w = column_start(g.cg, col + 1) - s0;
  return col * g.r + min(g.r, ((jmax - s0 + 1) * g.r + w - 1) / w);
}
#endif

}  // namespace sea
