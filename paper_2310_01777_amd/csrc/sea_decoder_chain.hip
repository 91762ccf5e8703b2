// The decoder's three 3x3 convolutions (Sec. 3.1 "CNN Decoder", App. A.5.1) of a causal layer in one launch, with the softmax
// of the last one's rows.  Causal layers read rows t - 2 .. t of the layer before, so a block walks down a strip of
// rows and keeps the last rows of each image in LDS: what the layers hand to each other never leaves the chip.  One
// launch per layer wrote and read it (50 MB each way and layer at H = 12, K = 128, T = 2048, B = 4).
//
// Two sets of four waves share the matrix cores, one wave of each on every SIMD.  Each wave keeps the weights of its
// layer in registers (168 at 48 channels; conv 1's last eight fragments in LDS), so an operand tile of 16 pixels read from
// LDS feeds every output channel: 64 clocks of LDS for the 96 that a step's products take.  With the weights in LDS it
// would be the other way round.  A step is four rows of every layer, one per wave: while conv 1 is on rows 4 j, conv 2 is on
// the four before and conv 3 on the four before those.  Two barriers a step: everything is read, then the new rows replace
// the oldest.  A strip's first rows are those that its second and third layer look back to (four of conv 1, two of conv 2).
//
// H = 12, K = 128, T = 2048, B = 4: 59 us where the three launches took 102 (33 + 34 + 33 and two gaps); T = 512 27 against 38,
// T = 256, B = 1 17.5 against 26; K = 64, T = 1365, B = 8 44 against 79.  A step takes 10.9 thousand clocks of 1.9 GHz, 6.3
// of them products: the waves of conv 1 and 3 are the longer chain (products of conv 3 1.4, softmax 3.3, products of conv 1
// 4.0, stores and barriers 1.7), in which the softmax waits on itself.
#include "sea_decoder.h"
#include "sea_lds.h"
#include "sea_rowlanes.h"

namespace sea {
namespace {

constexpr int kImgRows = 10, kMidRows = 6;  // rows in LDS: six that a step reads and, of the input, the next step's four
constexpr int kBack = 6;                    // input rows in front of a strip that its rows depend on

// fragments of conv 1's weights that stay in LDS: its waves take conv 3 too and need registers for that one's sums
constexpr int chain_lds_fragments(int P) { return P == 6 ? 8 : 0; }

// a wait the compiler knows of: it would otherwise wait for the weights inside the loop, where later loads are on their way
__device__ __forceinline__ void weights_here() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

struct ChainArgs {
  DecChain c;
  int32_t rows, strips;  // rows per strip (a multiple of four), strips per sequence
};

// where a lane finds unit 4 ks + lg of a contraction whose rows hold W units each; past the third row (zero weights) the first
// unit again
__device__ __forceinline__ const uint4* unit_at(const uint4* const (&row)[3], int W, int ks, int lg) {
  const int lo = 4 * ks / W, next = W * (lo + 1) - 4 * ks;  // lane groups from `next` on are in the row after
  const uint4* p = row[lo] + (4 * ks - lo * W) + lg;
  if (next < 4) {
    const uint4* o = lo + 1 < 3 ? row[lo + 1] + (4 * ks - (lo + 1) * W) + lg : row[0];
    p = lg >= next ? o : p;
  }
  return p;
}

// channel of row r of output tile nt: a lane holds rows 4 lg .. + 3 of each tile, and those of two tiles are eight channels in
// a row, one store of 16 bytes; a last odd tile keeps its order
__device__ __forceinline__ constexpr int channel(int NT, int nt, int r) {
  return (nt | 1) < NT ? 32 * (nt / 2) + r / 4 * 8 + nt % 2 * 4 + r % 4 : 16 * nt + r;
}

// One row of conv 1 or 2: the first FR fragments of the weights in registers, the others at wl (LDS, this lane's).  Pixels
// are requested two steps ahead of their products, in pairs of tiles (the compiler, left alone, asks for them one step at a
// time and waits).
template <int P, int NP, int FR>
__device__ __forceinline__ void conv_row(const bf16x8 (&wf)[FR], const uint4* wl, const uint4* const (&row)[3], int lg,
                                         const float* bias, uint2 (&res)[2 * NP][P / 2]) {
  constexpr int NT = P / 2, KS = (9 * P + 3) / 4, FL = KS * NT - FR;
  bf16x8 x[3][2], wx[FL > 0 ? FL : 1];
  floatx4 acc[NT][2];
  auto pixels = [&](int i) {
    const uint4* p = unit_at(row, 3 * P, i % KS, lg) + i / KS * 32 * P;
    x[i % 3][0] = __builtin_bit_cast(bf16x8, p[0]);
    x[i % 3][1] = __builtin_bit_cast(bf16x8, p[16 * P]);
  };
  pixels(0);
  pixels(1);
#pragma unroll
  for (int i = 0; i < NP * KS; ++i) {
    const int ks = i % KS;
    if (ks == 0) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const float4 bv = *reinterpret_cast<const float4*>(bias + channel(NT, nt, 4 * lg));
        acc[nt][0] = acc[nt][1] = floatx4{bv.x, bv.y, bv.z, bv.w};
      }
    }
    if (ks == FR / NT - 2) {
#pragma unroll
      for (int e = 0; e < FL; ++e) wx[e] = __builtin_bit_cast(bf16x8, wl[e * 64]);
    }
    if (i + 2 < NP * KS) pixels(i + 2);
    __builtin_amdgcn_sched_barrier(0x6);  // (arithmetic may pass: one pair's rounding goes under the next one's products)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int e = ks * NT + nt;
      const bf16x8 f = e < FR ? wf[e < FR ? e : 0] : wx[e < FR ? 0 : e - FR];
      acc[nt][0] = mfma16(f, x[i % 3][0], acc[nt][0]);
      acc[nt][1] = mfma16(f, x[i % 3][1], acc[nt][1]);
    }
    if (ks == KS - 1) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const floatx4 v = relu4(acc[nt][h]);
          uint2& r = res[2 * (i / KS) + h][nt];
          r = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
          if (i == NP * KS - 1) asm volatile("" : "+v"(r.x), "+v"(r.y));  // (here, not behind the barrier that the results wait for)
        }
    }
  }
}

// fragment e = (step ks, tile nt of the output channels) of a layer's weights [C][9 C]: channels 8 u .. + 7 of the contraction for output row lr
template <int P>
__device__ __forceinline__ bf16x8 weights_at(const uint16_t* w, int e, int lr, int lg) {
  const int ks = e / (P / 2), nt = e - ks * (P / 2), u = 4 * ks + lg;
  const bf16x8 v = load8(w + channel(P / 2, nt, lr) * (72 * P) + 8 * min(u, 9 * P - 1));
  return u < 9 * P ? v : zero8();
}

// The end of conv 3 for one image row and the head of a lane's column (l % 16): from D[k][mt][i], the products of tap column k
// with stored pixel s = 16 mt + 4 (l / 16) + i (D[1] holds the bias too), to the logits of the row resized to twice its width,
//   out[2 s] = D_0[s - 1] + D_1[s] + D_2[s],   out[2 s + 1] = D_0[s] + D_1[s] + D_2[s + 1],
// their softmax and the stores.  Pixels in the registers, heads in the lanes: three of four neighbours are the lane's own,
// a row's sums take two steps across lanes, and there is one division (280 vector instructions a row; 460 with the pixels
// in the lanes).  o: the head's row, if `exists`.
template <int MT>
__device__ __forceinline__ void finish_row(const floatx4 (&D)[3][MT], int lane, bool valid, float* __restrict__ o, bool exists) {
  typedef float float4_at __attribute__((ext_vector_type(4), aligned(8)));  // (rows of A may start between 16-byte words)
  const int lg = lane >> 4;
  auto put = [&](int mt, const float (&e)[8]) {
    float* p = o + 2 * (16 * mt + 4 * lg);
    *reinterpret_cast<float4_at*>(p) = float4_at{e[0], e[1], e[2], e[3]};
    *reinterpret_cast<float4_at*>(p + 4) = float4_at{e[4], e[5], e[6], e[7]};
  };
  if (!valid) {  // (uniform) a row past the sequence's end
    const float e[8] = {};
    if (exists) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) put(mt, e);
    }
    return;
  }
  // neighbours of a lane's outer pixels: the lane groups before and after, whose outermost hand on the next tile's
  auto from = [&](int other, float v) { return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * other, __float_as_int(v))); };
  float before[MT], after[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    before[mt] = from((lane - 16) & 63, lg == 3 ? (mt > 0 ? D[0][mt > 0 ? mt - 1 : 0][3] : 0.f) : D[0][mt][3]);
    after[mt] = from((lane + 16) & 63, lg == 0 ? (mt + 1 < MT ? D[2][mt + 1 < MT ? mt + 1 : mt][0] : 0.f) : D[2][mt][0]);
  }
  float x[MT][8], part[MT];  // (a tile's maximum, then its sum)
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    part[mt] = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[mt][2 * i] = D[1][mt][i] + D[2][mt][i] + (i > 0 ? D[0][mt][i > 0 ? i - 1 : 0] : before[mt]);
      x[mt][2 * i + 1] = D[0][mt][i] + D[1][mt][i] + (i < 3 ? D[2][mt][i < 3 ? i + 1 : 3] : after[mt]);
      part[mt] = fmaxf(fmaxf(part[mt], x[mt][2 * i]), x[mt][2 * i + 1]);
    }
  }
  float mx = part[0];
#pragma unroll
  for (int mt = 1; mt < MT; ++mt) mx = fmaxf(mx, part[mt]);
  mx = rows_max(mx);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    part[mt] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      x[mt][e] = __expf(x[mt][e] - mx);
      x[mt][e + 1] = __expf(x[mt][e + 1] - mx);
      part[mt] += x[mt][e] + x[mt][e + 1];
    }
  }
  float sum = part[0];
#pragma unroll
  for (int mt = 1; mt < MT; ++mt) sum += part[mt];
  const float inv = 1.f / rows_sum(sum);
  if (exists) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[mt][e] *= inv;
      put(mt, x[mt]);
    }
  }
}

// P = 16-byte units per pixel (8 channels each), NP = pairs of 16-pixel tiles per row
template <int P, int NP>
__global__ __launch_bounds__(512, 2) void dec_conv_chain_kernel(ChainArgs g, float* __restrict__ A,
                                                                const int32_t* __restrict__ seq_len) {
  constexpr int X = 32 * NP, C = 8 * P, NT = C / 16, KS = (9 * P + 3) / 4, K3 = (3 * P + 3) / 4;
  constexpr int FL = chain_lds_fragments(P), FR = KS * NT - FL;  // conv 1's fragments in LDS, in registers
  constexpr int kRow = (X + 2) * P;      // units of a row in LDS: a pixel of zeros on either side
  constexpr int kLoads = X * P / 64;     // wave-wide loads per row
  static_assert(C % 16 == 0 && X * P % 64 == 0, "whole operand tiles and loads");
  extern __shared__ __attribute__((aligned(16))) uint4 chain_lds[];
  uint4* const img = chain_lds;
  uint4* const y1 = img + kImgRows * kRow;
  uint4* const y2 = y1 + kMidRows * kRow;
  uint4* const w3 = y2 + kMidRows * kRow;                       // [K3][3][64]
  uint4* const wl = w3 + K3 * 3 * 64;                           // conv 1: [FL][64]
  float* const bias_s = reinterpret_cast<float*>(wl + FL * 64);  // conv 1, 2 and 3 (16)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int32_t T = g.c.T, H = g.c.H;
  const int32_t b = static_cast<int32_t>(blockIdx.x / static_cast<uint32_t>(g.strips));
  const int32_t t0 = (static_cast<int32_t>(blockIdx.x) - b * g.strips) * g.rows;
  const int32_t nblk = 1 + (min(g.rows, T - t0) + 3) / 4;  // steps of one layer
  // row q of the strip's count is image row t0 - kBack + q
  const int32_t first = max(t0 - kBack, 0);
  const u32x4 src = buffer_words(g.c.in + (static_cast<int64_t>(b) * T + first) * X * C,
                                 static_cast<uint32_t>(min(g.rows + kBack, T - first)) * (X * C * 2));
  auto request = [&](int32_t q0, int32_t n, int32_t id, int32_t waves) {
    for (; id < n * kLoads; id += waves) {
      const int32_t r = id / kLoads, part = id - r * kLoads, q = q0 + r, t = t0 - kBack + q;
      uint4* at = img + (q % kImgRows) * kRow + P + 64 * part;
      if (t >= 0 && t < T) {
        buffer_load_lds16(src, reinterpret_cast<uint16_t*>(at), static_cast<uint32_t>(t - first) * (X * C * 2) + 1024 * part + 16 * lane);
      } else {
        at[lane] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
  };
  // What passes through registers on its way to LDS is asked for together and first, the first rows and each wave's weights together
  // behind it: two waits for memory.
  {
    static_assert(FL <= 8, "one fragment per wave");
    constexpr int kW3 = (K3 * 3 * 64 + 511) / 512;
    bf16x8 l = zero8(), v[kW3];
    if (FL > 0) l = weights_at<P>(g.c.w[0], FR + min(wid, FL - 1), lr, lg);
    auto where = [&](int e, int32_t* ky, int32_t* co) {
      const int32_t id = tid + 512 * e, fl = id & 63, q = id >> 6, ks = q / 3, kx = q - 3 * ks, u = 4 * ks + (fl >> 4);
      *ky = u / P;
      *co = fl & 15;
      return (min(*co, H - 1) * 9 + 3 * min(*ky, 2) + kx) * C + 8 * (u - *ky * P);
    };
    int32_t ky, co;
#pragma unroll
    for (int e = 0; e < kW3; ++e) v[e] = load8(g.c.w[2] + where(e, &ky, &co));
    const float bias = *(tid < C ? g.c.bias[0] + tid : tid < 2 * C ? g.c.bias[1] + (tid - C) : g.c.bias[2] + min(tid - 2 * C, H - 1));
    __builtin_amdgcn_sched_barrier(0);
    if (wid < FL) wl[64 * wid + lane] = __builtin_bit_cast(uint4, l);
#pragma unroll
    for (int e = 0; e < kW3; ++e) {
      where(e, &ky, &co);
      if (tid + 512 * e < K3 * 3 * 64) w3[tid + 512 * e] = __builtin_bit_cast(uint4, ky < 3 && co < H ? v[e] : zero8());
    }
    if (tid < 2 * C + 16) bias_s[tid] = tid < 2 * C + H ? bias : 0.f;
  }
  request(0, 6, wid, 8);
  for (int32_t id = tid; id < (kImgRows + 2 * kMidRows) * 2 * P; id += 512) {
    const int32_t row = id / (2 * P), u = id - row * (2 * P);
    img[row * kRow + (u < P ? u : kRow - 2 * P + u)] = make_uint4(0u, 0u, 0u, 0u);  // (the three images lie one after the other)
  }
  const int32_t len = seq_len ? min(max(seq_len[b], 0), T) : T;

  // what the steps derive from the lane they derive anew: kept through the loop it would be spilled
  auto this_lane = [&]() {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  // rows q .. q + 2 of an image, pixel lr
  auto rows_at = [&](const uint4* ring, int32_t M, int32_t q, int lr, const uint4* (&row)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) row[k] = ring + ((q + k) % M) * kRow + lr * P;
  };
  // row q + 2 of block jb, computed before the barrier and stored behind it
  auto store = [&](uint4* ring, int32_t q, const uint2 (&res)[2 * NP][NT]) {
    const int l = this_lane(), lr = l & 15, lg = l >> 4;
    uint4* const out = ring + ((q + 2) % kMidRows) * kRow + (lr + 1) * P;
#pragma unroll
    for (int mt = 0; mt < 2 * NP; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; nt += 2) {
        uint4* const o = out + mt * 16 * P + 2 * nt;
        if (nt + 1 < NT) {
          o[lg] = make_uint4(res[mt][nt].x, res[mt][nt].y, res[mt][nt + 1 < NT ? nt + 1 : nt].x, res[mt][nt + 1 < NT ? nt + 1 : nt].y);
        } else {
          reinterpret_cast<uint2*>(o)[lg] = res[mt][nt];
        }
      }
  };
  auto clear = [&](uint2 (&res)[2 * NP][NT]) {  // in front of the sequence: zeros, not what a layer makes of zeros
#pragma unroll
    for (int mt = 0; mt < 2 * NP; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) res[mt][nt] = make_uint2(0u, 0u);
  };

  // the two sets of waves: the same steps and the same barriers
  if (wid < 4) {
    bf16x8 wf[FR];
#pragma unroll
    for (int e = 0; e < FR; ++e) wf[e] = weights_at<P>(g.c.w[0], e, lr, lg);
    lds_loads_done();
    weights_here();
    __syncthreads();
    for (int32_t j = 0; j < nblk + 2; ++j) {
      const uint4* row[3];
      if (j >= 3) {
        const int32_t q = 4 * (j - 2) + wid, t = t0 - kBack + q + 2;
        if (t < T) {
          const int l = this_lane(), lr = l & 15, lg = l >> 4;
          rows_at(y2 + P, kMidRows, q, lr, row);
          floatx4 D[3][2 * NP];
          const float b3 = bias_s[2 * C + lr];
#pragma unroll
          for (int mt = 0; mt < 2 * NP; ++mt) {
            D[0][mt] = D[2][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
            D[1][mt] = floatx4{b3, b3, b3, b3};
          }
          // weights a step ahead, pixels a pair of tiles
          bf16x8 kf[2][3], xf[2][2];
          auto weights = [&](int ks) {
#pragma unroll
            for (int k = 0; k < 3; ++k) kf[ks % 2][k] = __builtin_bit_cast(bf16x8, w3[(ks * 3 + k) * 64 + l]);
          };
          auto pixels = [&](int i) {
            const uint4* p = unit_at(row, P, i / NP, lg) + i % NP * 32 * P;
            xf[i % 2][0] = __builtin_bit_cast(bf16x8, p[0]);
            xf[i % 2][1] = __builtin_bit_cast(bf16x8, p[16 * P]);
          };
          weights(0);
          pixels(0);
#pragma unroll
          for (int i = 0; i < K3 * NP; ++i) {
            const int ks = i / NP, pr = i % NP;
            if (pr == 0 && ks + 1 < K3) weights(ks + 1);
            if (i + 1 < K3 * NP) pixels(i + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
              for (int h = 0; h < 2; ++h) D[k][2 * pr + h] = mfma16(xf[i % 2][h], kf[ks % 2][k], D[k][2 * pr + h]);
          }
          finish_row<2 * NP>(D, l, t < len, A + ((static_cast<int64_t>(b) * H + lr) * T + t) * (2 * X), lr < H);
        }
      }
      const int32_t q = 4 * j + wid;
      uint2 res[2 * NP][NT];
      if (j < nblk && t0 - kBack + q + 2 >= 0) {
        const int l = this_lane();
        rows_at(img, kImgRows, q, l & 15, row);
        conv_row<P, NP, FR>(wf, wl + l, row, l >> 4, bias_s, res);
      } else {
        clear(res);
      }
      __syncthreads();  // everything is read
      if (j < nblk) store(y1, q, res);
      __syncthreads();  // (no wait for memory: the loads are the other set's, this one only stores A)
    }
  } else {
    bf16x8 wf[KS * NT];
#pragma unroll
    for (int e = 0; e < KS * NT; ++e) wf[e] = weights_at<P>(g.c.w[1], e, lr, lg);
    lds_loads_done();
    weights_here();
    __syncthreads();
    for (int32_t j = 0; j < nblk + 2; ++j) {
      if (j + 1 < nblk) request(4 * j + 6, 4, wid - 4, 4);  // (the other set's chain is the longer one)
      const bool busy = j >= 1 && j <= nblk;
      const int32_t q = 4 * (j - 1) + wid - 4;
      uint2 res[2 * NP][NT];
      if (busy && t0 - kBack + q + 2 >= 0) {
        const uint4* row[3];
        const int l = this_lane();
        rows_at(y1, kMidRows, q, l & 15, row);
        conv_row<P, NP, KS * NT>(wf, nullptr, row, l >> 4, bias_s + C, res);
      } else {
        clear(res);
      }
      __syncthreads();
      if (busy) store(y2, q, res);
      lds_loads_done();
      __syncthreads();
    }
  }
}

template <int P, int NP>
hipError_t start_chain(const ChainArgs& g, float* A, const int32_t* seq_len, hipStream_t st) {
  constexpr size_t lds = ((kImgRows + 2 * kMidRows) * static_cast<size_t>((32 * NP + 2) * P) + (3 * P + 3) / 4 * 3 * 64 +
                          chain_lds_fragments(P) * 64) * 16 + (16 * P + 16) * 4;
  static_assert(lds <= (160 << 10), "one block per CU");
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dec_conv_chain_kernel<P, NP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((dec_conv_chain_kernel<P, NP>), dim3(static_cast<uint32_t>(g.c.B * g.strips)), dim3(512), lds, st, g, A, seq_len);
  return hipGetLastError();
}

}  // namespace

// hipErrorNotSupported: no instance for these layers; the caller has a kernel for each.  Heads: 4 H channels, whole tiles of 16, and
// at most 48, whose weights fit a wave's registers.  Rows: whole pairs of 16-pixel tiles (K = 32 stores 16 pixels).  Wider rows than
// 64 pixels would fit in LDS with 8 heads to K = 192 (148 KB) and with 4 to K = 256 (96 KB), with 12 not (K = 192: 207 KB); no instances
// are built.  Where it fits it is the faster one at every size measured, layers of one short sequence (estimate, three launches /
// this: H = 4, K = 64, T = 64 31.6 / 23.1 us, H = 12, T = 256 49.3 / 42.3) to 16 rounds of a CU (the convolutions, T = 4096, B = 4 182 / 108); fewer
// channels gain as much (H = 4 47 / 24 at T = 2048, B = 4, H = 8 70 / 38).
hipError_t launch_dec_chain(const DecChain& c, float* A, const int32_t* seq_len, hipStream_t st) {
  if ((c.H != 4 && c.H != 8 && c.H != 12) || (c.X != 32 && c.X != 64)) return hipErrorNotSupported;
  if (c.T > 1 << 19) return hipErrorNotSupported;  // (32-bit offsets into a strip)
  ChainArgs g{};
  g.c = c;
  // strips: as many as fill the CUs once, or a few times if the last round would be short; a strip costs three steps
  // beside its own.  (One block per CU; of four heads, with 86 or 122 registers, a second one would fit: not tried)
  const int64_t quads = (static_cast<int64_t>(c.T) + 3) / 4;
  int64_t best = 0;
  for (int64_t n = 1; n <= 4; ++n) {
    const int64_t want = std::max<int64_t>(1, 256 * n / c.B), per = (quads + want - 1) / want, strips = (quads + per - 1) / per;
    const int64_t cost = (c.B * strips + 255) / 256 * (per + 3);
    if (best == 0 || cost < best) {
      best = cost;
      g.rows = static_cast<int32_t>(4 * per);
      g.strips = static_cast<int32_t>(strips);
    }
  }
  const bool wide = c.X == 64;
  if (c.H == 4) return wide ? start_chain<2, 2>(g, A, seq_len, st) : start_chain<2, 1>(g, A, seq_len, st);
  if (c.H == 8) return wide ? start_chain<4, 2>(g, A, seq_len, st) : start_chain<4, 1>(g, A, seq_len, st);
  return wide ? start_chain<6, 2>(g, A, seq_len, st) : start_chain<6, 1>(g, A, seq_len, st);
}

}  // namespace sea
