// The decoder's Performer step (Sec. 3.1 "CNN Decoder"): C_perf = FAVOR+(Q, K, [V_I; V]) in linear time,
// normalised rows of 128 bf16 values.  V_I is the T x 64 nearest-neighbour stretch of the identity.
//
// A block takes 64-token chunks of one head; nothing but Q, K, V, W is read and nothing but C_perf and the
// segment states is written.  Eight waves, three barriers per chunk:
//   features  waves 0..3 phi(Q), waves 4..7 phi(K) of 16 tokens each (C[feature][token] = W X^T); phi(Q) goes to LDS as
//             operand fragments, phi(K) and V as rows
//   products  wave v owns the 16 value columns 16 v .. (V_I: 0..3, V: 4..7) and their m x 16 state S in registers:
//             O^T = S^T phi(Q)^T; causal: the ten lower-triangular 16 x 16 tiles of P^T = phi(K) phi(Q)^T are shared
//             out among the waves and meet in LDS; then S += phi(K)^T U, the token-major operands coming from the rows
//             through the LDS transpose read
//   outputs   O^T += U^T P^T, the normaliser passes through LDS, C_perf leaves as bf16 under the next chunk's products
//             (at once, the next chunk's features waited for the stores)
// Every key lies in exactly one column of V_I, so a row's normaliser is the sum of its V_I outputs; and a wave of V_I's has
// values at a quarter of the tokens only: chunks and segments without any are left out of its products and sums.
// Products contract over features in the order of packed accumulators (slot 8 g + e of a 32-feature step =
// feature 16 (e / 4) + 4 g + e % 4) and over tokens in the same order, so accumulators are operands as they
// stand.  phi(Q) is scaled per row by a power of two, which cancels in the normaliser.
//
// For parallelism the sequence is cut into G segments: a first launch (MODE 0) leaves each segment's
// state, the second starts from the sum of the earlier ones (causal) or of all (bidirectional).
// Bound: LDS (450 KB of operands per chunk) and the vector pipe, each a third of the time and one after the other between
// the barriers.  B = 4, H = 12, T = 2048, m = 128: 20.3 + 44.6 -> 16.5 + 38.0 us with a ninth wave for the normaliser
// (and the stores, the zero products of V_I) gone.  Two blocks per CU with half the chunks each take 16 + 44.
// The estimator's scores against 64 bits (relative 2-norm, 12 heads of 512 rows, three seeds) with a normaliser of its own, whose
// state was rounded apart from the outputs', and so: causal 2.59, 3.22, 2.87e-3 -> 2.56, 3.20, 2.84e-3, bidirectional 2.53, 3.13,
// 2.77e-3 -> 2.49, 3.11, 2.74e-3.
#include "sea_decoder.h"
#include "sea_rowlanes.h"

namespace sea {
namespace {

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
// 64-bit LDS read with the 16-bit transpose across each group of 16 lanes (ds_read_b64_tr_b16): lane i of a
// group receives element i % 4 of the 8 bytes that lanes 4 e + i / 4, e = 0..3, of the group point at
__device__ __forceinline__ bf16x4 lds_transpose4(const uint16_t* p) {
  return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)(p)));
}
__device__ __forceinline__ bf16x8 join(bf16x4 lo, bf16x4 hi) { return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7); }

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

constexpr int kLinWaves = 8, kLinThreads = 64 * kLinWaves;
constexpr int kTok = 64;   // tokens per chunk
constexpr int kVRow = 80;  // halfwords per staged V row: the rows of a transpose read on distinct banks

// MODE 0 leaves the states of the segments, 1 emits the rows of bidirectional layers, 2 those of causal ones.
template <int MC, int MODE>
__global__ __launch_bounds__(kLinThreads, 2) void dec_linattn_kernel(Shape s, int32_t G, int32_t cps,
                                                                     const uint16_t* __restrict__ Q,
                                                                     const uint16_t* __restrict__ K,
                                                                     const uint16_t* __restrict__ V,
                                                                     const uint16_t* __restrict__ W,
                                                                     uint16_t* __restrict__ Cp,
                                                                     float4* __restrict__ seg_state, float c_dot,
                                                                     float c_norm) {
  constexpr int m = 32 * MC;
  constexpr bool EMIT = MODE != 0, CAUSAL = MODE == 2, KEYS = MODE != 1;
  constexpr int kKRow = m + 16;  // halfwords per staged phi(K) row (+ 32 B: as above)
  extern __shared__ __attribute__((aligned(16))) uint16_t lin_lds[];
  uint4* Wf = reinterpret_cast<uint4*>(lin_lds);               // [2 MC tiles][2 halves][64]: W rows as operands
  uint4* Qf = Wf + 2 * MC * 2 * 64;                             // [4 token tiles][MC][64]
  uint16_t* Ks = reinterpret_cast<uint16_t*>(Qf + (EMIT ? 4 * MC * 64 : 0));  // [64][kKRow]
  uint16_t* Vs = Ks + kTok * kKRow;                             // [64][kVRow]
  uint4* Ps = reinterpret_cast<uint4*>(Vs + kTok * kVRow);      // [2 key pairs][4 query tiles][64]
  float* den = reinterpret_cast<float*>(Ps + (EMIT ? 8 * 64 : 0));  // [4 waves][64 queries]
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t seg = static_cast<int32_t>(blockIdx.x % static_cast<uint32_t>(G));
  const int64_t head = blockIdx.x / static_cast<uint32_t>(G);
  const int32_t b = static_cast<int32_t>(head / s.H);
  const int32_t len = s.seq_len ? min(max(s.seq_len[b], 0), s.T) : s.T;
  const int32_t nchunks = (s.T + kTok - 1) / kTok;
  const int32_t c_begin = min(nchunks, seg * cps), c_end = min(nchunks, c_begin + cps);
  if (!EMIT && s.causal && seg == G - 1) return;  // nothing comes after the last segment (block-uniform)

  // the chunk's rows on their way: waves 0..3 the queries, 4..7 the keys of their 16 tokens (MODE 0: all eight the
  // keys, half of the features each), and a piece of a value row per thread
  const bool is_q = EMIT && wid < 4;
  bf16x8 r0 = zero8(), r1 = zero8();
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 vreg = {0u, 0u, 0u, 0u};
  auto request = [&](int32_t c) __attribute__((always_inline)) {
    if (is_q || KEYS) {
      const uint16_t* X = (is_q ? Q : K) + (head * s.T + min(kTok * c + 16 * (wid & 3) + lr, s.T - 1)) * kHeadDim;
      r0 = load8(X + 8 * lg);
      r1 = load8(X + 32 + 8 * lg);
    }
    if (KEYS) vreg = *reinterpret_cast<const u32x4*>(V + (head * s.T + min(kTok * c + (tid >> 3), s.T - 1)) * kHeadDim + 8 * (tid & 7));
  };
  request(c_begin);
  uint4 wreg[MC / 2];
#pragma unroll
  for (int e = 0; e < MC / 2; ++e) {
    const int id = tid + kLinThreads * e, fl = id & 63, half = (id >> 6) & 1, ft = id >> 7;
    wreg[e] = *reinterpret_cast<const uint4*>(W + (16 * ft + (fl & 15)) * kHeadDim + 32 * half + 8 * (fl >> 4));
  }

  // this wave's value columns: V_I[j][v] = 1 for vi_lo <= j < vi_hi, i.e. floor(j 64 / T) == v; a wave of V_I's has
  // values at tokens own_lo .. own_hi - 1 only
  const int32_t vcol = 16 * wid + lr;
  auto vi_first = [&](int32_t v) { return min(s.T, static_cast<int32_t>((static_cast<int64_t>(v) * s.T + kHeadDim - 1) / kHeadDim)); };
  const int32_t vi_lo = vi_first(vcol), vi_hi = vi_first(vcol + 1);
  const int32_t own_lo = wid < 4 ? vi_first(16 * wid) : 0, own_hi = wid < 4 ? vi_first(16 * wid + 16) : s.T;
  auto has_values = [&](int32_t from, int32_t to) { return from < own_hi && to > own_lo; };
  // values of tokens t0 + 32 p + {4 lg .. + 3, 16 + 4 lg .. + 3} in this lane's column
  auto value_frag = [&](int32_t t0, int p) -> bf16x8 {
    if (wid >= 4) {
      const uint16_t* r = Vs + (32 * p + 4 * lg + (lr >> 2)) * kVRow + 16 * (wid - 4) + 4 * (lr & 3);
      return join(lds_transpose4(r), lds_transpose4(r + 16 * kVRow));
    }
    uint32_t w[4];
    const int32_t j0 = t0 + 32 * p + 4 * lg;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int32_t j = j0 + (e < 2 ? 2 * e : 12 + 2 * e);
      w[e] = (j >= vi_lo && j < vi_hi ? 0x3f80u : 0u) | (j + 1 >= vi_lo && j + 1 < vi_hi ? 0x3f800000u : 0u);
    }
    const uint4 u = {w[0], w[1], w[2], w[3]};
    return __builtin_bit_cast(bf16x8, u);
  };

  auto features = [&](int32_t c) __attribute__((always_inline)) {
    // (every way through here has the rows: where one way left them pending, the next request would wait for whatever
    // is on its way, the stores of the chunk before among it)
    asm volatile("" : "+v"(r0), "+v"(r1), "+v"(vreg));
    if (KEYS) {
      const bool in = kTok * c + (tid >> 3) < len;
      *reinterpret_cast<u32x4*>(Vs + (tid >> 3) * kVRow + 8 * (tid & 7)) = in ? vreg : u32x4{0u, 0u, 0u, 0u};
    }
    if (!is_q && !KEYS) return;
    const float bias = c_norm * rows_sum(sumsq8(r0) + sumsq8(r1));
    const bool active = kTok * c + 16 * (wid & 3) + lr < len;
    auto project = [&](int ft) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = mfma16(__builtin_bit_cast(bf16x8, Wf[(2 * ft) * 64 + lane]), r0, acc);
      acc = mfma16(__builtin_bit_cast(bf16x8, Wf[(2 * ft + 1) * 64 + lane]), r1, acc);
      return floatx4{fmaf(c_dot, acc[0], -bias), fmaf(c_dot, acc[1], -bias), fmaf(c_dot, acc[2], -bias), fmaf(c_dot, acc[3], -bias)};
    };
    auto exps = [&](floatx4 a, float shift) {
      return floatx4{active ? __builtin_amdgcn_exp2f(a[0] - shift) : 0.f, active ? __builtin_amdgcn_exp2f(a[1] - shift) : 0.f,
                     active ? __builtin_amdgcn_exp2f(a[2] - shift) : 0.f, active ? __builtin_amdgcn_exp2f(a[3] - shift) : 0.f};
    };
    if (is_q) {
      floatx4 arg[2 * MC];
      float amax = -INFINITY;
#pragma unroll
      for (int ft = 0; ft < 2 * MC; ++ft) {
        arg[ft] = project(ft);
#pragma unroll
        for (int i = 0; i < 4; ++i) amax = fmaxf(amax, arg[ft][i]);
      }
      const float shift = ceilf(rows_max(amax));
#pragma unroll
      for (int kc = 0; kc < MC; ++kc)
        Qf[((wid & 3) * MC + kc) * 64 + lane] = __builtin_bit_cast(uint4, pack8(exps(arg[2 * kc], shift), exps(arg[2 * kc + 1], shift)));
    } else {
      const int kc0 = EMIT ? 0 : (wid >> 2) * (MC / 2);
#pragma unroll
      for (int k = 0; k < (EMIT ? MC : MC / 2); ++k) {
        const int kc = kc0 + k;
        const floatx4 lo = project(2 * kc), hi = project(2 * kc + 1);
        const uint4 f = __builtin_bit_cast(uint4, pack8(exps(lo, 0.f), exps(hi, 0.f)));
        uint16_t* row = Ks + (16 * (wid & 3) + lr) * kKRow + 32 * kc + 4 * lg;
        *reinterpret_cast<uint2*>(row) = make_uint2(f.x, f.y);
        *reinterpret_cast<uint2*>(row + 16) = make_uint2(f.z, f.w);
      }
    }
  };
  // phi(K) of 16 keys as an operand with the keys as rows
  auto key_frag = [&](int jt, int kc) {
    const uint16_t* r = Ks + (16 * jt + lr) * kKRow + 32 * kc + 4 * lg;
    const uint2 a = *reinterpret_cast<const uint2*>(r), c = *reinterpret_cast<const uint2*>(r + 16);
    const uint4 u = {a.x, a.y, c.x, c.y};
    return __builtin_bit_cast(bf16x8, u);
  };

  floatx4 S[2 * MC];
#pragma unroll
  for (int x = 0; x < 2 * MC; ++x) S[x] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int64_t hs = head * kLinWaves + wid;  // (head, value tile)
  if (EMIT) {
    const int32_t upto = CAUSAL ? seg : G;
    const float4* st = seg_state + hs * G * (2 * MC * 64) + lane;
#pragma unroll 2
    for (int32_t q = 0; q < upto; ++q) {
      if (!has_values(kTok * cps * q, kTok * cps * (q + 1))) continue;
#pragma unroll
      for (int x = 0; x < 2 * MC; ++x) {
        const float4 v = st[(static_cast<int64_t>(q) * 2 * MC + x) * 64];
        S[x][0] += v.x; S[x][1] += v.y; S[x][2] += v.z; S[x][3] += v.w;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < MC / 2; ++e) Wf[tid + kLinThreads * e] = wreg[e];
  __syncthreads();  // W is parked
  uint2 out[4];  // a chunk's results; they leave while the next chunk's products run
  auto store = [&](int32_t t0) __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < 4; ++qt) {
      const int32_t t = t0 + 16 * qt + lr;
      if (t < s.T) *reinterpret_cast<uint2*>(Cp + (head * s.T + t) * 128 + 16 * wid + 4 * lg) = out[qt];
    }
  };
  for (int32_t c = c_begin; c < c_end; ++c) {
    const int32_t t0 = kTok * c;
    features(c);
    __syncthreads();
    if (EMIT && c > c_begin) store(t0 - kTok);
    request(c + 1);
    floatx4 OT[4];
    bf16x8 U[2];
    if (EMIT) {
      if (CAUSAL) {
        // tile id = (query tile qt, key tile jt <= qt); V_I's waves, which have less to do, take two each, two others one
#pragma unroll 1
        for (int id = wid < 4 ? wid : wid + 4; id < (wid < 4 ? 8 : 10); id += 4) {
          const int qt = id < 1 ? 0 : (id < 3 ? 1 : (id < 6 ? 2 : 3)), jt = id - (qt * (qt + 1)) / 2;
          floatx4 P = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kc = 0; kc < MC; ++kc) P = mfma16(key_frag(jt, kc), __builtin_bit_cast(bf16x8, Qf[(qt * MC + kc) * 64 + lane]), P);
          // rows = keys 4 lg + i, column = query lr
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (jt == qt && 4 * lg + i > lr) P[i] = 0.f;
          uint2* dst = reinterpret_cast<uint2*>(&Ps[((jt >> 1) * 4 + qt) * 64 + lane]);
          dst[jt & 1] = make_uint2(pack_bf16(P[0], P[1]), pack_bf16(P[2], P[3]));
          if (jt == qt && (jt & 1) == 0) dst[1] = make_uint2(0u, 0u);  // the pair's other tile lies above the diagonal
        }
      }
#pragma unroll
      for (int qt = 0; qt < 4; ++qt) OT[qt] = floatx4{0.f, 0.f, 0.f, 0.f};
      if (!CAUSAL || own_lo < t0)  // (else there is no state yet)
#pragma unroll
      for (int kc = 0; kc < MC; ++kc) {
        const bf16x8 sf = pack8(S[2 * kc], S[2 * kc + 1]);
#pragma unroll
        for (int qt = 0; qt < 4; ++qt) OT[qt] = mfma16(sf, __builtin_bit_cast(bf16x8, Qf[(qt * MC + kc) * 64 + lane]), OT[qt]);
      }
    }
    const bool here = has_values(t0, t0 + kTok);  // wave-uniform
    if (KEYS && here) {
      U[0] = value_frag(t0, 0);
      U[1] = value_frag(t0, 1);
      if (!EMIT || c + 1 < c_end) {  // the state after the last emitted chunk is not used
#pragma unroll
        for (int x = 0; x < 2 * MC; ++x)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const uint16_t* r = Ks + (32 * p + 4 * lg + (lr >> 2)) * kKRow + 16 * x + 4 * (lr & 3);
            S[x] = mfma16(join(lds_transpose4(r), lds_transpose4(r + 16 * kKRow)), U[p], S[x]);
          }
      }
    }
    if (EMIT) {
      if (CAUSAL) {
        __syncthreads();  // P is there
        if (here)
#pragma unroll
        for (int qt = 0; qt < 4; ++qt)
#pragma unroll
          for (int p = 0; p <= qt / 2; ++p) OT[qt] = mfma16(U[p], __builtin_bit_cast(bf16x8, Ps[(p * 4 + qt) * 64 + lane]), OT[qt]);
      }
      if (wid < 4)  // every key lies in one column of V_I: a row's normaliser is the sum of its outputs there
#pragma unroll
        for (int qt = 0; qt < 4; ++qt) {
          const float d = rows_sum((OT[qt][0] + OT[qt][1]) + (OT[qt][2] + OT[qt][3]));
          if (lg == 0) den[64 * wid + 16 * qt + lr] = d;
        }
    }
    __syncthreads();  // the chunk's rows are no longer read; the normaliser is there
    if (EMIT) {
#pragma unroll
      for (int qt = 0; qt < 4; ++qt) {
        const float d = (den[16 * qt + lr] + den[64 + 16 * qt + lr]) + (den[128 + 16 * qt + lr] + den[192 + 16 * qt + lr]);
        const float inv = d > 0.f ? 1.f / d : 0.f;
        out[qt] = make_uint2(pack_bf16(OT[qt][0] * inv, OT[qt][1] * inv), pack_bf16(OT[qt][2] * inv, OT[qt][3] * inv));
      }
    }
  }
  if (EMIT && c_begin < c_end) store(kTok * (c_end - 1));
  if (!EMIT && has_values(kTok * c_begin, kTok * c_end)) {
    float4* my = seg_state + (hs * G + seg) * (2 * MC * 64) + lane;
#pragma unroll
    for (int x = 0; x < 2 * MC; ++x) my[x * 64] = make_float4(S[x][0], S[x][1], S[x][2], S[x][3]);
  }
}

// segments per sequence: blocks for every CU (one block each), at least two chunks per segment
int32_t segments(const Shape& s) {
  const int32_t nchunks = (s.T + kTok - 1) / kTok;
  return std::max(1, std::min({16, 256 / s.N, nchunks / 2}));
}

template <int MC, int MODE>
hipError_t start(const Shape& s, int32_t G, int32_t cps, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                 const uint16_t* W, uint16_t* Cp, float4* seg, float c_dot, float c_norm, hipStream_t st) {
  constexpr int m = 32 * MC;
  const size_t lds = static_cast<size_t>(2 * MC * 2 * 64 + (MODE ? 4 * MC * 64 + 8 * 64 : 0)) * 16 +
                     static_cast<size_t>(kTok) * (m + 16 + kVRow) * 2 + (MODE ? 4 * kTok * 4 : 0);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dec_linattn_kernel<MC, MODE>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((dec_linattn_kernel<MC, MODE>), dim3(static_cast<uint32_t>(s.N) * G), dim3(kLinThreads), lds, st, s, G, cps,
                     Q, K, V, W, Cp, seg, c_dot, c_norm);
  return hipGetLastError();
}

template <int MC>
hipError_t start_both(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* V, const uint16_t* W, uint16_t* Cp,
                      float4* seg, float c_dot, float c_norm, hipStream_t st) {
  const int32_t nchunks = (s.T + kTok - 1) / kTok, most = segments(s), cps = (nchunks + most - 1) / most, G = (nchunks + cps - 1) / cps;
  if (G > 1 || !s.causal) {
    const hipError_t e = start<MC, 0>(s, G, cps, Q, K, V, W, Cp, seg, c_dot, c_norm, st);
    if (e != hipSuccess) return e;
  }
  return s.causal ? start<MC, 2>(s, G, cps, Q, K, V, W, Cp, seg, c_dot, c_norm, st)
                  : start<MC, 1>(s, G, cps, Q, K, V, W, Cp, seg, c_dot, c_norm, st);
}

}  // namespace

size_t dec_linattn_state_bytes(const Shape& s) {
  return static_cast<size_t>(s.N) * kLinWaves * segments(s) * s.m * 16 * sizeof(float);
}

hipError_t launch_dec_linattn(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* V, const uint16_t* W,
                              uint16_t* Cp, void* state, float c_dot, float c_norm, hipStream_t st) {
  float4* seg = static_cast<float4*>(state);
  switch (s.m) {
    case 64: return start_both<2>(s, Q, K, V, W, Cp, seg, c_dot, c_norm, st);
    case 128: return start_both<4>(s, Q, K, V, W, Cp, seg, c_dot, c_norm, st);
    default: return start_both<8>(s, Q, K, V, W, Cp, seg, c_dot, c_norm, st);
  }
}

}  // namespace sea
