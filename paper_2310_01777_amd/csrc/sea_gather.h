// Attention of one query row by one wavefront, its keys read one by one (Sec. 3.1.1: rho, sigma, A* V fused).
//
// A key (or value) row of d = 64 elements is 128 B in bf16 (8 lanes x 16 B) or 256 B in fp32 (16 lanes x 16 B),
// so one 128-bit load per lane fetches 8 (bf16) or 4 (fp32) gathered rows per wave instruction, each row
// contiguous across its lane group.  The softmax is the streaming (running max / running sum) form held in
// registers.  Keys the row does not use are never part of its arithmetic.
//
// Where the keys come from is a type: n slots, taken in order, kGatherUnroll G at a time, by
// next<G>(g, j, ok): slot u G + g of the batch is key j[u] if ok[u]; else j[u] is an address that may be read
// (a key of the row where it has one, so that a weight of zero never meets what the row does not use).
#pragma once
#include "sea_columns.h"
#include "sea_internal.h"
#include "sea_tile.h"

namespace sea {
#if defined(__HIPCC__)

constexpr int kGatherUnroll = 4;

// n entries at p, each a key plus `base`; entries outside [0, T) are ignored
struct ListKeys {
  const int32_t* p;
  int32_t n, base, T;
  int32_t k0 = 0;
  template <int G>
  __device__ __forceinline__ void next(int g, int32_t (&j)[kGatherUnroll], bool (&ok)[kGatherUnroll]) {
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) {
      const int32_t at = k0 + u * G + g;
      // the index is read unconditionally (a slot past the list re-reads its last entry and is
      // then discarded): a load behind `at < n` would be waited for before the next slot's is issued
      const int32_t v = p[min(at, n - 1)] - base;
      const bool in = static_cast<uint32_t>(v) < static_cast<uint32_t>(T);
      ok[u] = in && at < n;
      j[u] = in ? v : 0;
    }
    k0 += kGatherUnroll * G;
  }
};

// The keys of a row's selected columns up to position jmax (sea_columns.h; the order of the list).  Lane l works
// out the position of every 64th slot; a batch takes its slots from the lanes that hold them.
struct ColumnKeys {
  ColumnList g;
  const uint16_t* cols;  // the row's columns, ascending: K halfwords of LDS that belong to this wave
  int32_t n;             // slots: columns times `per` (a whole column may leave its last slot empty)
  int32_t ncols, per, jmax, first, q64, r64;
  int32_t ci, i, at, key;

  // mrow: the row's mask words (global memory); the whole wave calls
  __device__ __forceinline__ ColumnKeys(const ColumnList& list, const uint32_t* mrow, int32_t KW, int32_t jmax_,
                                        uint16_t* place)
      : g(list), cols(place), jmax(jmax_) {
    const int lane = threadIdx.x & 63;
    uint32_t w = lane < KW ? mrow[lane] : 0u;  // KW <= 32
    const int32_t left = g.cg.K - 32 * lane;
    if (left < 32) w &= left > 0 ? (1u << left) - 1u : 0u;  // bits that are no column
    int32_t upto = __popc(w);
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
      const int32_t below = __shfl_up(upto, off, kWave);
      if (lane >= off) upto += below;
    }
    ncols = __builtin_amdgcn_readlane(upto, 31);
    __builtin_amdgcn_wave_barrier();
    for (int32_t e = upto - __popc(w); w != 0u; w &= w - 1u, ++e)
      place[e] = static_cast<uint16_t>(32 * lane + __ffs(static_cast<int>(w)) - 1);
    __builtin_amdgcn_wave_barrier();
    per = g.r != 0 ? g.r : g.cg.w0 + (g.cg.rm > 0 ? 1 : 0);
    n = ncols * per;
    first = ncols > 0 ? column_start(g.cg, cols[0]) : 0;
    ci = lane / per;
    i = lane - ci * per;
    q64 = kWave / per;
    r64 = kWave - q64 * per;
    at = kWave;
  }
  __device__ __forceinline__ void refill() {
    const int32_t c = cols[min(ci, ncols - 1)];
    const int32_t s0 = column_start(g.cg, c), w = column_start(g.cg, c + 1) - s0;
    const int32_t pos = s0 + (g.r == 0 ? i : entry_offset(g, i, w));
    const bool ok = ci < ncols && (g.r != 0 || i < w) && pos <= jmax;
    key = ok ? pos : ~first;
    ci += q64;
    i += r64;
    if (i >= per) {
      i -= per;
      ++ci;
    }
    at = 0;
  }
  template <int G>
  __device__ __forceinline__ void next(int g8, int32_t (&j)[kGatherUnroll], bool (&ok)[kGatherUnroll]) {
    static_assert(kWave % (kGatherUnroll * G) == 0, "whole batches");
    if (at == kWave) refill();
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) {
      const int32_t k = __shfl(key, at + u * G + g8, kWave);
      ok[u] = k >= 0;
      j[u] = k >= 0 ? k : ~k;
    }
    at += kGatherUnroll * G;
  }
};

// bf16: fp32 logits (f q.k, f = scale log2(e)), weights and accumulators; O rounded once
template <typename Keys>
__device__ __forceinline__ void gather_row_bf16(Keys keys, float f, const uint16_t* __restrict__ Qr,
                                                const uint16_t* __restrict__ Kh, const uint16_t* __restrict__ Vh,
                                                uint16_t* __restrict__ Or) {
  const int lane = threadIdx.x & 63;
  const int g = lane >> 3;   // which of the 8 rows of a wave load
  const int c8 = lane & 7;   // which 16-byte chunk of the row

  // q stays in bf16 pairs: q.k is four packed dot-product instructions per lane (exact products,
  // fp32 sums); the logit scale is applied to the finished dot product
  const uint4 qv = *reinterpret_cast<const uint4*>(Qr + c8 * 8);
  const uint32_t qw[4] = {qv.x, qv.y, qv.z, qv.w};
  const int32_t n = keys.n;

  float m_run = -INFINITY, l_run = 0.f;
  float o[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = 0.f;

  for (int32_t k0 = 0; k0 < n; k0 += 8 * kGatherUnroll) {
    uint4 kv[kGatherUnroll], vv[kGatherUnroll];
    int32_t j[kGatherUnroll];
    bool ok[kGatherUnroll];
    keys.template next<8>(g, j, ok);
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) {
      kv[u] = *reinterpret_cast<const uint4*>(Kh + static_cast<int64_t>(j[u]) * kHeadDim + c8 * 8);
      vv[u] = *reinterpret_cast<const uint4*>(Vh + static_cast<int64_t>(j[u]) * kHeadDim + c8 * 8);
    }
    float sc[kGatherUnroll];
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) {
      const uint32_t w[4] = {kv[u].x, kv[u].y, kv[u].z, kv[u].w};
      float a = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, qw[i]), __builtin_bit_cast(bf16x2, w[i]), a, false);
      a += __shfl_xor(a, 1, kWave);
      a += __shfl_xor(a, 2, kWave);
      a += __shfl_xor(a, 4, kWave);
      sc[u] = ok[u] ? a * f : -INFINITY;
      mx = fmaxf(mx, sc[u]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 8, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    const float m_new = fmaxf(m_run, mx);
    if (m_new == -INFINITY) continue;  // nothing valid yet (uniform across the wave)
    const float corr = exp2f(m_run - m_new);  // exp2(-inf) = 0 on the first valid batch
    m_run = m_new;
    l_run *= corr;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] *= corr;
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) {
      const float pj = exp2f(sc[u] - m_new);  // 0 for masked entries
      l_run += pj;
      const uint32_t w[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        o[2 * i] = fmaf(pj, bf16lo_to_f32(w[i]), o[2 * i]);
        o[2 * i + 1] = fmaf(pj, bf16hi_to_f32(w[i]), o[2 * i + 1]);
      }
    }
  }
  // combine the 8 row groups
#pragma unroll
  for (int mask = 8; mask <= 32; mask <<= 1) {
    l_run += __shfl_xor(l_run, mask, kWave);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] += __shfl_xor(o[e], mask, kWave);
  }
  if (g == 0) {
    const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
    uint4 out;
    out.x = pack_bf16(o[0] * inv, o[1] * inv);
    out.y = pack_bf16(o[2] * inv, o[3] * inv);
    out.z = pack_bf16(o[4] * inv, o[5] * inv);
    out.w = pack_bf16(o[6] * inv, o[7] * inv);
    *reinterpret_cast<uint4*>(Or + c8 * 8) = out;
  }
}

// fp32: f q.k with fp64 sums, so that logits of magnitude ~40 still leave the probabilities accurate to ~1e-7;
// weights and accumulators in fp32
template <typename Keys>
__device__ __forceinline__ void gather_row_f32(Keys keys, double f, const float* __restrict__ Qr,
                                               const float* __restrict__ Kh, const float* __restrict__ Vh,
                                               float* __restrict__ Or) {
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4;    // which of the 4 rows of a wave load
  const int c16 = lane & 15;  // which 16-byte chunk of the row

  const float4 q4 = *reinterpret_cast<const float4*>(Qr + c16 * 4);
  const double qd[4] = {q4.x, q4.y, q4.z, q4.w};
  const int32_t n = keys.n;

  double m_run = -INFINITY;
  float l_run = 0.f;
  float o[4] = {0.f, 0.f, 0.f, 0.f};

  for (int32_t k0 = 0; k0 < n; k0 += 4 * kGatherUnroll) {
    float4 kv[kGatherUnroll], vv[kGatherUnroll];
    bool ok[kGatherUnroll];
    int32_t j[kGatherUnroll];
    keys.template next<4>(g, j, ok);
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) {
      kv[u] = *reinterpret_cast<const float4*>(Kh + static_cast<int64_t>(j[u]) * kHeadDim + c16 * 4);
      vv[u] = *reinterpret_cast<const float4*>(Vh + static_cast<int64_t>(j[u]) * kHeadDim + c16 * 4);
    }
    double sc[kGatherUnroll];
    double mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) {
      double a = qd[0] * kv[u].x;
      a = fma(qd[1], static_cast<double>(kv[u].y), a);
      a = fma(qd[2], static_cast<double>(kv[u].z), a);
      a = fma(qd[3], static_cast<double>(kv[u].w), a);
      a += __shfl_xor(a, 1, kWave);
      a += __shfl_xor(a, 2, kWave);
      a += __shfl_xor(a, 4, kWave);
      a += __shfl_xor(a, 8, kWave);
      sc[u] = ok[u] ? a * f : -INFINITY;
      mx = fmax(mx, sc[u]);
    }
    mx = fmax(mx, __shfl_xor(mx, 16, kWave));
    mx = fmax(mx, __shfl_xor(mx, 32, kWave));
    const double m_new = fmax(m_run, mx);
    if (m_new == -INFINITY) continue;
    const float corr = exp2f(static_cast<float>(m_run - m_new));
    m_run = m_new;
    l_run *= corr;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] *= corr;
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) {
      const float pj = exp2f(static_cast<float>(sc[u] - m_new));
      l_run += pj;
      o[0] = fmaf(pj, vv[u].x, o[0]);
      o[1] = fmaf(pj, vv[u].y, o[1]);
      o[2] = fmaf(pj, vv[u].z, o[2]);
      o[3] = fmaf(pj, vv[u].w, o[3]);
    }
  }
#pragma unroll
  for (int mask = 16; mask <= 32; mask <<= 1) {
    l_run += __shfl_xor(l_run, mask, kWave);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] += __shfl_xor(o[e], mask, kWave);
  }
  if (g == 0) {
    float4 out = {0.f, 0.f, 0.f, 0.f};
    if (l_run > 0.f) out = {o[0] / l_run, o[1] / l_run, o[2] / l_run, o[3] / l_run};
    *reinterpret_cast<float4*>(Or + c16 * 4) = out;
  }
}

#endif  // __HIPCC__
}  // namespace sea
