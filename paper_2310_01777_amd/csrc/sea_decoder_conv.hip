// The decoder's 3x3 convolutions (Sec. 3.1 "CNN Decoder", App. A.5.1) for images of up to 64 channels
// (conv 1 and 2) and, for the last layer, up to 128 with rows of at most 128 stored pixels, whose softmax is
// taken on the spot.  Channels-last bf16 images, fp32 sums, products transposed: C[channel][pixel] =
// weights x pixels^T.
//
// Both kernels keep all weights of their channel slab in LDS, in operand-fragment order, and stay on
// their CU: a block takes tile after tile, and the next tile's input window is on its way to registers
// while the current one, parked in LDS, is multiplied.  The contraction runs over (tap, 8-channel
// unit) pairs; where a lane finds its unit inside the window is the same for every tile and pixel, so
// offsets taken once (a register or a table word per step) replace the index arithmetic, which is what
// bound the chunked kernel of sea_decoder.hip on these sizes (about 100 vector instructions against 12
// matrix products per step).
#include "sea_decoder.h"

namespace sea {
namespace {

constexpr int kMaxPieces = 8;  // 16-byte pieces of the window a thread moves per tile

struct ConvTile {
  const uint16_t* in;
  const uint16_t* w;  // [Cout][3][3][Cin]
  const float* bias;
  int32_t B, Tin, Xin, Cin, Tout, Xout, Cout, stride_t, pad_top, relu;
  int32_t Tv;         // rows of the (nearest) resized image the taps read; columns are as stored
  int32_t P, pxu;     // 16-byte units per pixel, and their odd stride in LDS
  int32_t ksteps;
  int32_t cw_log, rows_out, halo_rows, halo_cols, tiles_t, tiles_x;
  float invP, inv_cols;
};

// element `id` of a tile's window: pixel and unit
struct Piece {
  int32_t hr, hc, unit;
};
__device__ __forceinline__ Piece piece_of(const ConvTile& g, int32_t id) {
  const int32_t px = static_cast<int32_t>((static_cast<float>(id) + 0.5f) * g.invP);
  const int32_t hr = static_cast<int32_t>((static_cast<float>(px) + 0.5f) * g.inv_cols);
  return {hr, px - hr * g.halo_cols, id - px * g.P};
}

// conv 1 and 2, 8 P channels in and out.  Block = 8 waves; wave = 16 MT pixels of the tile x all channels.
template <int P, int MT>
__global__ __launch_bounds__(512, 2) void dec_conv_tile_kernel(ConvTile g, uint16_t* __restrict__ out) {
  constexpr int NT = (P + 1) / 2, KS = (9 * P + 3) / 4, pxu = P | 1;
  extern __shared__ __attribute__((aligned(16))) uint4 conv_lds[];
  uint4* halo = conv_lds;                                     // [halo_rows][halo_cols][pxu]
  uint4* wts = halo + g.halo_rows * g.halo_cols * pxu;        // [KS][NT][64]
  float* bias_s = reinterpret_cast<float*>(wts + KS * NT * 64);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  for (int32_t id = tid; id < KS * NT * 64; id += 512) {
    const int32_t fl = id & 63, q = id >> 6, ks = q / NT, nt = q - ks * NT;
    const int32_t u = 4 * ks + (fl >> 4), tap = u / P, cu = u - tap * P;
    const int32_t co = 16 * nt + (fl & 15);
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (tap < 9 && co < g.Cout) v = *reinterpret_cast<const uint4*>(g.w + static_cast<int64_t>(co * 9 + tap) * g.Cin + 8 * cu);
    wts[id] = v;
  }
  // where this lane's unit of each step lies in a pixel's window (a step's units past the ninth tap meet
  // zero weights: any place will do)
  int32_t offs[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int32_t u = 4 * ks + lg, tap = u / P, cu = u - tap * P, ky = tap / 3, kx = tap - 3 * ky;
    offs[ks] = tap < 9 ? (ky * g.halo_cols + kx) * pxu + cu : 0;
  }
  if (tid < 16 * NT) bias_s[tid] = tid < g.Cout ? g.bias[tid] : 0.f;

  const int32_t npiece = g.halo_rows * g.halo_cols * P;
  uint4 held[kMaxPieces];
  auto place = [&](int64_t tile, int64_t* b, int32_t* t0, int32_t* x0) {
    const int64_t q = tile / g.tiles_x;
    *x0 = static_cast<int32_t>(tile - q * g.tiles_x) << g.cw_log;
    *b = q / g.tiles_t;
    *t0 = static_cast<int32_t>(q - *b * g.tiles_t) * g.rows_out;
  };
  auto request = [&](int64_t tile) {
    int64_t b;
    int32_t t0, x0;
    place(tile, &b, &t0, &x0);
    const uint16_t* img = g.in + b * g.Tin * static_cast<int64_t>(g.Xin) * g.Cin;
#pragma unroll
    for (int e = 0; e < kMaxPieces; ++e) {
      if (512 * e >= npiece) break;
      const Piece p = piece_of(g, min(tid + 512 * e, npiece - 1));
      const int32_t tv = t0 * g.stride_t - g.pad_top + p.hr, xv = x0 - 1 + p.hc;
      const bool ok = static_cast<uint32_t>(tv) < static_cast<uint32_t>(g.Tin) && static_cast<uint32_t>(xv) < static_cast<uint32_t>(g.Xin);
      // (unconditional load from a clamped address, cleared afterwards: no load behind a branch)
      const int32_t tc = min(max(tv, 0), g.Tin - 1), xc = min(max(xv, 0), g.Xin - 1);
      const uint4 v = *reinterpret_cast<const uint4*>(img + (static_cast<int64_t>(tc) * g.Xin + xc) * g.Cin + 8 * p.unit);
      held[e] = ok ? v : make_uint4(0u, 0u, 0u, 0u);
    }
  };
  auto park = [&]() {
#pragma unroll
    for (int e = 0; e < kMaxPieces; ++e) {
      const int32_t id = tid + 512 * e;
      if (id >= npiece) break;
      const Piece p = piece_of(g, id);
      halo[(p.hr * g.halo_cols + p.hc) * pxu + p.unit] = held[e];
    }
  };
  int32_t base[MT], prow[MT], pcol[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int32_t pidx = (wid * MT + mt) * 16 + lr;
    prow[mt] = pidx >> g.cw_log;
    pcol[mt] = pidx & ((1 << g.cw_log) - 1);
    base[mt] = (prow[mt] * g.stride_t * g.halo_cols + pcol[mt]) * pxu;
  }
  const int64_t ntile = static_cast<int64_t>(g.B) * g.tiles_t * g.tiles_x;
  int64_t tile = blockIdx.x;
  if (tile < ntile) request(tile);
  for (; tile < ntile; tile += gridDim.x) {
    __syncthreads();  // the previous window is no longer read (first round: weights and table are there)
    park();
    __syncthreads();
    if (tile + gridDim.x < ntile) request(tile + gridDim.x);
    floatx4 acc[NT][MT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const float4 bv = *reinterpret_cast<const float4*>(bias_s + 16 * nt + 4 * lg);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = floatx4{bv.x, bv.y, bv.z, bv.w};
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int32_t o = offs[ks];
      bf16x8 xf[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xf[mt] = __builtin_bit_cast(bf16x8, halo[base[mt] + o]);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const bf16x8 wf = __builtin_bit_cast(bf16x8, wts[(ks * NT + nt) * 64 + lane]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = mfma16(wf, xf[mt], acc[nt][mt]);
      }
    }
    int64_t b;
    int32_t t0, x0;
    place(tile, &b, &t0, &x0);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int32_t t = t0 + prow[mt], x = x0 + pcol[mt];
      if (t >= g.Tout || x >= g.Xout) continue;
      uint16_t* o = out + ((b * g.Tout + t) * g.Xout + x) * g.Cout + 4 * lg;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        if (16 * nt + 4 * lg >= g.Cout) continue;
        floatx4 v = acc[nt][mt];
        if (g.relu) v = relu4(v);
        *reinterpret_cast<uint2*>(o + 16 * nt) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
      }
    }
  }
}

// conv 3 on the image resized to T x 2 Wd (nearest), and the softmax over the 2 Wd outputs of a (head, row).
// The resize doubles every stored pixel, so the three taps of an output column read two stored pixels:
// with D_k[s] = the products of tap column k (all three rows) with stored pixel s,
//   out[2 s] = D_0[s - 1] + D_1[s] + D_2[s],   out[2 s + 1] = D_0[s] + D_1[s] + D_2[s + 1]
// -- the same products, taken once per stored pixel instead of once per output (half the pixel operands
// and less than half the steps), and added in fp32.  Wave = one image row of up to 16 MT stored pixels x
// 16 heads (blockIdx.y: which 16); lane l % 16 is the pixel, so neighbours are lane rotations and a row's
// softmax stays inside the wave.
template <int MT, int NW>
__global__ __launch_bounds__(64 * NW, 2) void dec_conv_softmax_kernel(ConvTile g, float* __restrict__ A,
                                                                      const int32_t* __restrict__ seq_len) {
  extern __shared__ __attribute__((aligned(16))) uint4 conv_lds[];
  constexpr int kThreads = 64 * NW;
  uint4* halo = conv_lds;                                            // [NW + 2 rows][Xin][pxu]
  uint4* wts = halo + g.halo_rows * g.halo_cols * g.pxu;             // [kstep][3][64]
  int32_t* offs = reinterpret_cast<int32_t*>(wts + g.ksteps * 3 * 64);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int32_t cout0 = 16 * blockIdx.y;
  for (int32_t id = tid; id < g.ksteps * 3 * 64; id += kThreads) {
    const int32_t fl = id & 63, q = id >> 6, ks = q / 3, kx = q - 3 * ks;
    const int32_t u = 4 * ks + (fl >> 4);
    const int32_t ky = static_cast<int32_t>((static_cast<float>(u) + 0.5f) * g.invP), cu = u - ky * g.P;
    const int32_t co = cout0 + (fl & 15);
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (ky < 3 && co < g.Cout) v = *reinterpret_cast<const uint4*>(g.w + static_cast<int64_t>(co * 9 + 3 * ky + kx) * g.Cin + 8 * cu);
    wts[id] = v;
  }
  if (tid < 4 * g.ksteps) {
    const int32_t ky = tid / g.P, cu = tid - ky * g.P;
    offs[tid] = ky < 3 ? ky * g.halo_cols * g.pxu + cu : 0;
  }
  float bv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) bv[i] = cout0 + 4 * lg + i < g.Cout ? g.bias[cout0 + 4 * lg + i] : 0.f;

  const int32_t npiece = g.halo_rows * g.halo_cols * g.P;
  uint4 held[kMaxPieces];
  auto request = [&](int64_t tile) {
    const int64_t b = tile / g.tiles_t;
    const int32_t t0 = static_cast<int32_t>(tile - b * g.tiles_t) * NW;
    const uint16_t* img = g.in + b * g.Tin * static_cast<int64_t>(g.Xin) * g.Cin;
#pragma unroll
    for (int e = 0; e < kMaxPieces; ++e) {
      if (kThreads * e >= npiece) break;
      const Piece p = piece_of(g, min(tid + kThreads * e, npiece - 1));
      const int32_t tv = t0 - g.pad_top + p.hr;
      const bool ok = static_cast<uint32_t>(tv) < static_cast<uint32_t>(g.Tv);
      const int32_t tc = min(max(tv, 0), g.Tv - 1);
      const int32_t ts = g.Tv == g.Tin ? tc : static_cast<int32_t>((static_cast<int64_t>(tc) * g.Tin) / g.Tv);
      const uint4 v = *reinterpret_cast<const uint4*>(img + (static_cast<int64_t>(ts) * g.Xin + p.hc) * g.Cin + 8 * p.unit);
      held[e] = ok ? v : make_uint4(0u, 0u, 0u, 0u);
    }
  };
  auto park = [&]() {
#pragma unroll
    for (int e = 0; e < kMaxPieces; ++e) {
      const int32_t id = tid + kThreads * e;
      if (id >= npiece) break;
      const Piece p = piece_of(g, id);
      halo[(p.hr * g.halo_cols + p.hc) * g.pxu + p.unit] = held[e];
    }
  };
  int32_t base[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) base[mt] = (wid * g.halo_cols + min(16 * mt + lr, g.Xin - 1)) * g.pxu;

  const int64_t ntile = static_cast<int64_t>(g.B) * g.tiles_t;
  int64_t tile = blockIdx.x;
  if (tile < ntile) request(tile);
  for (; tile < ntile; tile += gridDim.x) {
    __syncthreads();
    park();
    __syncthreads();
    if (tile + gridDim.x < ntile) request(tile + gridDim.x);
    floatx4 D[3][MT];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) D[k][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int32_t ks = 0; ks < g.ksteps; ++ks) {
      const int32_t o = offs[4 * ks + lg];
      bf16x8 wf[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) wf[k] = __builtin_bit_cast(bf16x8, wts[(ks * 3 + k) * 64 + lane]);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const bf16x8 xf = __builtin_bit_cast(bf16x8, halo[base[mt] + o]);
#pragma unroll
        for (int k = 0; k < 3; ++k) D[k][mt] = mfma16(wf[k], xf, D[k][mt]);
      }
    }
    const int64_t b = tile / g.tiles_t;
    const int32_t t = static_cast<int32_t>(tile - b * g.tiles_t) * NW + wid;
    if (t >= g.Tout) continue;  // (wave-uniform; the barriers are at the loop's head)
    const int32_t len = seq_len ? min(max(seq_len[b], 0), g.Tout) : g.Tout;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // lane rotations inside the 16 pixels of a tile: left[mt] = D_0 of the pixel before, right[mt] = D_2
      // of the pixel after (tile borders take the neighbouring tile's, the image's border is zero)
      float ev[MT], od[MT];
      float rot_prev = 0.f;  // D_0 of the tile before, rotated
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float d0 = D[0][mt][i];
        const float rot = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(d0), 0x121, 0xf, 0xf, false));  // row_ror:1
        const float left = lr == 0 ? rot_prev : rot;
        rot_prev = rot;
        ev[mt] = left + (D[1][mt][i] + D[2][mt][i]) + bv[i];
        od[mt] = d0 + D[1][mt][i] + bv[i];
      }
      float rot_next = 0.f;  // D_2 of the tile after, rotated
#pragma unroll
      for (int mt = MT - 1; mt >= 0; --mt) {
        const bool last = 16 * mt + lr == g.Xin - 1;
        const float rot = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(D[2][mt][i]), 0x12F, 0xf, 0xf, false));  // row_ror:15
        const float right = lr == 15 ? rot_next : rot;
        rot_next = rot;
        od[mt] += last ? 0.f : right;
      }
      // softmax over the row's 2 Xin values
      float mx = -INFINITY;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const bool in = 16 * mt + lr < g.Xin;
        ev[mt] = in ? ev[mt] : -INFINITY;
        od[mt] = in ? od[mt] : -INFINITY;
        mx = fmaxf(mx, fmaxf(ev[mt], od[mt]));
      }
      mx = fmaxf(mx, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mx), 0xB1, 0xf, 0xf, false)));
      mx = fmaxf(mx, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mx), 0x4E, 0xf, 0xf, false)));
      mx = fmaxf(mx, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mx), 0x141, 0xf, 0xf, false)));
      mx = fmaxf(mx, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mx), 0x140, 0xf, 0xf, false)));
      float sum = 0.f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        ev[mt] = __expf(ev[mt] - mx);
        od[mt] = __expf(od[mt] - mx);
        sum += ev[mt] + od[mt];
      }
      sum += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(sum), 0xB1, 0xf, 0xf, false));
      sum += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(sum), 0x4E, 0xf, 0xf, false));
      sum += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(sum), 0x141, 0xf, 0xf, false));
      sum += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(sum), 0x140, 0xf, 0xf, false));
      const float inv = t < len ? 1.f / sum : 0.f;
      const int32_t h = cout0 + 4 * lg + i;
      if (h < g.Cout) {
        float* o = A + ((b * g.Cout + h) * g.Tout + t) * g.Xout;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          if (16 * mt + lr < g.Xin) {
            const float e0 = t < len ? ev[mt] * inv : 0.f, e1 = t < len ? od[mt] * inv : 0.f;
            *reinterpret_cast<float2*>(o + 2 * (16 * mt + lr)) = make_float2(e0, e1);
          }
      }
    }
  }
}

constexpr size_t kLdsMax = 160 << 10;

template <int P, int MT>
hipError_t start_conv(const ConvTile& g, size_t lds, uint16_t* out, hipStream_t st) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dec_conv_tile_kernel<P, MT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  const int64_t ntile = static_cast<int64_t>(g.B) * g.tiles_t * g.tiles_x;
  const uint32_t per_cu = lds <= kLdsMax / 2 && MT == 1 ? 2 : 1;  // (more pixels per wave: registers for one block)
  hipLaunchKernelGGL((dec_conv_tile_kernel<P, MT>), dim3(static_cast<uint32_t>(std::min<int64_t>(ntile, 256 * per_cu))), dim3(512),
                     lds, st, g, out);
  return hipGetLastError();
}
template <int MT>
hipError_t start_conv_p(const ConvTile& g, size_t lds, uint16_t* out, hipStream_t st) {
  switch (g.P) {
    case 1: return start_conv<1, MT>(g, lds, out, st);
    case 2: return start_conv<2, MT>(g, lds, out, st);
    case 3: return start_conv<3, MT>(g, lds, out, st);
    case 4: return start_conv<4, MT>(g, lds, out, st);
    case 5: return start_conv<5, MT>(g, lds, out, st);
    case 6: return start_conv<6, MT>(g, lds, out, st);
    case 7: return start_conv<7, MT>(g, lds, out, st);
    default: return start_conv<8, MT>(g, lds, out, st);
  }
}
template <int MT, int NW>
hipError_t start_softmax(const ConvTile& g, size_t lds, float* A, const int32_t* seq_len, hipStream_t st) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dec_conv_softmax_kernel<MT, NW>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  const int64_t ntile = static_cast<int64_t>(g.B) * g.tiles_t;
  const uint32_t per_cu = lds <= kLdsMax / 2 && NW == 4 ? 2 : 1;
  hipLaunchKernelGGL((dec_conv_softmax_kernel<MT, NW>),
                     dim3(static_cast<uint32_t>(std::min<int64_t>(ntile, 256 * per_cu)), static_cast<uint32_t>((g.Cout + 15) / 16)),
                     dim3(64 * NW), lds, st, g, A, seq_len);
  return hipGetLastError();
}

}  // namespace

// hipErrorNotSupported: the layer does not fit (more than 64 channels); the caller has another kernel
hipError_t launch_dec_conv(const DecConv& c, uint16_t* out, hipStream_t st) {
  if (c.Cin % 8 != 0 || c.Cout != c.Cin || c.Cin > 64) return hipErrorNotSupported;
  ConvTile g{};
  g.in = c.in; g.w = c.w; g.bias = c.bias; g.B = c.B; g.Tin = g.Tv = c.Tin; g.Xin = g.Xout = c.X; g.Cin = c.Cin;
  g.Tout = c.Tout; g.Cout = c.Cout; g.stride_t = c.stride_t; g.pad_top = c.pad_top; g.relu = 1;
  g.P = c.Cin / 8; g.pxu = g.P | 1; g.ksteps = (9 * g.P + 3) / 4; g.invP = 1.0f / static_cast<float>(g.P);
  const int nt = (c.Cout + 15) / 16;
  g.cw_log = c.X <= 16 ? 4 : (c.X <= 32 ? 5 : 6);
  g.tiles_x = (c.X + (1 << g.cw_log) - 1) >> g.cw_log;
  g.halo_cols = (1 << g.cw_log) + 2;
  g.inv_cols = 1.0f / static_cast<float>(g.halo_cols);
  // pixels per wave: the largest whose window fits next to the weights, smaller where that leaves CUs idle
  for (int mt = 4; mt >= 1; mt /= 2) {
    g.rows_out = (8 * 16 * mt) >> g.cw_log;
    if (g.rows_out < 1) break;
    g.halo_rows = (g.rows_out - 1) * g.stride_t + 3;
    g.tiles_t = (c.Tout + g.rows_out - 1) / g.rows_out;
    const size_t lds = static_cast<size_t>(g.halo_rows * g.halo_cols * g.pxu + g.ksteps * nt * 64) * 16 + 64 * 4;
    if (lds > kLdsMax || g.halo_rows * g.halo_cols * g.P > 512 * kMaxPieces) continue;
    if (mt > 1 && static_cast<int64_t>(g.B) * g.tiles_t * g.tiles_x < 256) continue;
    if (mt == 4) return start_conv_p<4>(g, lds, out, st);
    if (mt == 2) return start_conv_p<2>(g, lds, out, st);
    return start_conv_p<1>(g, lds, out, st);
  }
  return hipErrorNotSupported;
}

hipError_t launch_dec_conv_softmax(const DecConv& c, int32_t Tv, float* A, const int32_t* seq_len, hipStream_t st) {
  if (c.Cin % 8 != 0 || c.X > 128) return hipErrorNotSupported;
  ConvTile g{};
  g.in = c.in; g.w = c.w; g.bias = c.bias; g.B = c.B; g.Tin = c.Tin; g.Tv = Tv; g.Xin = c.X; g.Xout = 2 * c.X; g.Cin = c.Cin;
  g.Tout = c.Tout; g.Cout = c.Cout; g.stride_t = 1; g.pad_top = c.pad_top;
  g.P = c.Cin / 8; g.pxu = g.P | 1; g.ksteps = (3 * g.P + 3) / 4; g.invP = 1.0f / static_cast<float>(g.P);
  g.halo_cols = c.X;
  g.inv_cols = 1.0f / static_cast<float>(g.halo_cols);
  for (int nw = 8; nw >= 4; nw /= 2) {
    g.rows_out = nw;
    g.halo_rows = nw + 2;
    g.tiles_t = (c.Tout + nw - 1) / nw;
    const size_t lds = static_cast<size_t>(g.halo_rows * g.halo_cols * g.pxu + g.ksteps * 3 * 64) * 16 + 4 * g.ksteps * 4;
    if (lds > kLdsMax || g.halo_rows * g.halo_cols * g.P > 64 * nw * kMaxPieces) continue;
    if (nw > 4 && static_cast<int64_t>(g.B) * g.tiles_t < 256 && c.Tout > 4) continue;
    if (nw == 8) {
      if (c.X <= 32) return start_softmax<2, 8>(g, lds, A, seq_len, st);
      if (c.X <= 64) return start_softmax<4, 8>(g, lds, A, seq_len, st);
      return start_softmax<8, 8>(g, lds, A, seq_len, st);
    }
    if (c.X <= 32) return start_softmax<2, 4>(g, lds, A, seq_len, st);
    if (c.X <= 64) return start_softmax<4, 4>(g, lds, A, seq_len, st);
    return start_softmax<8, 4>(g, lds, A, seq_len, st);
  }
  return hipErrorNotSupported;
}

}  // namespace sea
