// SEA's decoder path (Sec. 3.1 "CNN Decoder", App. A.5.1 "Attention Estimator CNN") with
// caller-supplied weights: the Performer output on the concatenated values [V_I; V], the MLPs mu
// and nu, the three-layer CNN (nearest resize before its last layer) and the final softmax that
// yields the compressed attention matrix A_hat, plus the scalers s_mix, s_prob of Sec. 3.1.1
// "Output Calculation".  bf16 tensors, fp32 accumulation, every contraction on the matrix cores
// (v_mfma_f32_16x16x32_bf16) with operand fragments loaded straight from memory: lane l of a wave
// holds row / column l % 16 and the contraction elements 8 (l / 16) .. + 7 of a 32-wide step, and
// an accumulator tile (lane = column l % 16, registers = rows 4 (l / 16) + i) can be packed and
// fed back as an operand fragment of the next product without leaving the registers.
//
// Kernels, in the order a call runs them:
//   dec_linattn_kernel    C_perf from Q, K, V (sea_decoder_linattn.hip)
//   dec_mlp_kernel        mu, nu, s_mix, s_prob (sea_decoder_mlp.hip)
//   dec_conv_chain_kernel all three convolutions and the final softmax of causal layers with rows of 32 or 64 stored pixels
//                         and 4, 8 or 12 heads (sea_decoder_chain.hip); others:
//   dec_conv_tile_kernel, dec_conv_softmax_kernel
//                         the convolutions of images with up to 64 channels and the final softmax
//                         (sea_decoder_conv.hip); wider layers:
//   dec_conv3_kernel, dec_conv_lds_kernel, dec_conv_kernel
//                         implicit GEMM on channels-last images, optional nearest resize on the read
//   dec_softmax_kernel    softmax over the K columns of a row, rows past the sequence end zeroed
#include "sea_decoder.h"

namespace sea {
namespace {

constexpr int kCs = 2;       // width reduction of the CNN's hidden image (c_s)
constexpr int kCh = 4;       // channel expansion (c_h)

// ------------------------------------------------------------------------------------------
// implicit GEMM: out[pixel][cout] = act(bias[cout] + sum over (tap, c) in[pixel + tap][c] w[cout][tap][c]).
// A 3x3 convolution on a channels-last image [B][Tin][Xin][Cin], read through an optional nearest
// resize to Tv x Xv (source index floor(v * size / vsize)); zero outside the (virtual) image.  Computed transposed,
// C[cout][pixel] = W x X^T: the lane is the pixel, a lane holds four consecutive output channels.
// Wide layers (dec_conv_lds_kernel): block = 4 waves, wave = 64 pixels x up to 128 output channels
// (blockIdx.y picks the channel slab); the weights of the block's channels go through LDS in slabs of
// 128 contraction elements (fetched into registers one slab ahead), the pixels' operand fragments
// come straight from memory.
// ------------------------------------------------------------------------------------------
struct ConvArgs {
  const uint16_t* in;
  const uint16_t* w;     // [Cout][3][3][Cin]
  const float* bias;     // [Cout]
  void* out;
  int32_t B, Tin, Xin, Cin, Tv, Xv, Tout, Xout, Cout, stride_t, pad_top, relu;
  int32_t mode;          // 0: bf16 channels-last; 2: fp32 planes
};

constexpr int kSlabK = 128;            // contraction elements of the weights staged per step
constexpr int kSlabRow = kSlabK + 8;   // halfwords per staged weight row (+16 B: b128 reads spread over the banks)

__global__ __launch_bounds__(256, 2) void dec_conv_lds_kernel(ConvArgs a) {
  // weights of the block's 128 output channels for one slab of the contraction, shared by the four waves
  __shared__ __attribute__((aligned(16))) uint16_t Wsl[128 * kSlabRow];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int64_t npix = static_cast<int64_t>(a.B) * a.Tout * a.Xout;
  const int64_t pix0 = (static_cast<int64_t>(blockIdx.x) * 4 + wid) * 64;  // may lie past the end: the wave then only stages
  const int32_t cout0 = blockIdx.y * 128;
  const int32_t ntiles = min(8, (a.Cout - cout0 + 15) / 16);
  const int32_t ktot = 9 * a.Cin;
  const int32_t nslabs = (ktot + kSlabK - 1) / kSlabK;
  // this lane's four pixels (operand columns)
  int32_t pb[4], pt[4], px[4];
  bool pok[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    const int64_t p = pix0 + 16 * mt + lr;
    pok[mt] = p < npix;
    const int64_t pc = pok[mt] ? p : npix - 1;
    px[mt] = static_cast<int32_t>(pc % a.Xout);
    pt[mt] = static_cast<int32_t>((pc / a.Xout) % a.Tout);
    pb[mt] = static_cast<int32_t>(pc / (static_cast<int64_t>(a.Xout) * a.Tout));
  }
  floatx4 acc[8][4];
#pragma unroll
  for (int nt = 0; nt < 8; ++nt)
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

  // staging role: 16-byte piece (tid & 15) of rows (tid >> 4) + 16 q, q < 8
  const int srow = tid >> 4, spart = tid & 15;
  uint4 wreg[8];
  auto fetch = [&](int32_t slab) {
    const int32_t k = slab * kSlabK + 8 * spart;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int32_t co = cout0 + srow + 16 * q;
      wreg[q] = (co < a.Cout && k < ktot) ? *reinterpret_cast<const uint4*>(a.w + static_cast<int64_t>(co) * ktot + k)
                                          : make_uint4(0u, 0u, 0u, 0u);
    }
  };
  auto park = [&]() {
#pragma unroll
    for (int q = 0; q < 8; ++q) *reinterpret_cast<uint4*>(&Wsl[(srow + 16 * q) * kSlabRow + 8 * spart]) = wreg[q];
  };
  fetch(0);
  park();
  __syncthreads();
  for (int32_t slab = 0; slab < nslabs; ++slab) {
    if (slab + 1 < nslabs) fetch(slab + 1);
    if (pix0 < npix) {
#pragma unroll
      for (int ks = 0; ks < kSlabK / 32; ++ks) {
        const int32_t kbase = slab * kSlabK + 32 * ks;
        if (kbase >= ktot) break;
        const int32_t k0 = kbase + 8 * lg;
        const bool kok = k0 < ktot;
        const int32_t tap = kok ? k0 / a.Cin : 0, c0 = kok ? k0 - tap * a.Cin : 0;
        const int32_t ky = tap / 3, kx = tap - 3 * ky;
        bf16x8 xf[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const int32_t tv = pt[mt] * a.stride_t + ky - a.pad_top;
          const int32_t xv = px[mt] + kx - 1;
          const bool ok = kok && pok[mt] && tv >= 0 && tv < a.Tv && xv >= 0 && xv < a.Xv;
          if (ok) {
            const int32_t ts = a.Tv == a.Tin ? tv : static_cast<int32_t>((static_cast<int64_t>(tv) * a.Tin) / a.Tv);
            const int32_t xs = a.Xv == a.Xin ? xv : static_cast<int32_t>((static_cast<int64_t>(xv) * a.Xin) / a.Xv);
            xf[mt] = load8(a.in + ((static_cast<int64_t>(pb[mt]) * a.Tin + ts) * a.Xin + xs) * a.Cin + c0);
          } else {
            xf[mt] = zero8();
          }
        }
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
          if (nt < ntiles) {
            const bf16x8 wf = *reinterpret_cast<const bf16x8*>(&Wsl[(16 * nt + lr) * kSlabRow + 32 * ks + 8 * lg]);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = mfma16(wf, xf[mt], acc[nt][mt]);
          }
        }
      }
    }
    __syncthreads();  // every wave is done with the slab
    if (slab + 1 < nslabs) {
      park();
      __syncthreads();
    }
  }
  if (pix0 >= npix) return;
  // epilogue: tile (nt, mt): rows = output channels cout0 + 16 nt + 4 lg + i, column = pixel lr of tile mt
#pragma unroll
  for (int nt = 0; nt < 8; ++nt) {
    if (nt >= ntiles) continue;
    const int32_t co = cout0 + 16 * nt + 4 * lg;
    if (co >= a.Cout) continue;
    float bv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bv[i] = co + i < a.Cout ? a.bias[co + i] : 0.f;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      if (!pok[mt]) continue;
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = acc[nt][mt][i] + bv[i];
        if (a.relu) v[i] = fmaxf(v[i], 0.f);
      }
      const int64_t p = pix0 + 16 * mt + lr;
      if (a.mode == 0) {
        uint2 pk = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + p * a.Cout + co) = pk;
      } else {
        float* o = static_cast<float*>(a.out);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (co + i < a.Cout)
            o[((static_cast<int64_t>(pb[mt]) * a.Cout + co + i) * a.Tout + pt[mt]) * a.Xout + px[mt]] = v[i];
      }
    }
  }
}

// The same product for few output channels or a short contraction: wave = 32 pixels, every operand
// fragment straight from memory (the weights stay in the caches), no barriers.
__global__ __launch_bounds__(256) void dec_conv_kernel(ConvArgs a) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int64_t npix = static_cast<int64_t>(a.B) * a.Tout * a.Xout;
  const int64_t pix0 = (static_cast<int64_t>(blockIdx.x) * 4 + wid) * 32;
  if (pix0 >= npix) return;
  const int32_t cout0 = blockIdx.y * 128;
  const int32_t ntiles = min(8, (a.Cout - cout0 + 15) / 16);
  const int32_t ktot = 9 * a.Cin;
  // this lane's two pixels (operand columns)
  int32_t pb[2], pt[2], px[2];
  bool pok[2];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    const int64_t p = pix0 + 16 * mt + lr;
    pok[mt] = p < npix;
    const int64_t pc = pok[mt] ? p : npix - 1;
    px[mt] = static_cast<int32_t>(pc % a.Xout);
    pt[mt] = static_cast<int32_t>((pc / a.Xout) % a.Tout);
    pb[mt] = static_cast<int32_t>(pc / (static_cast<int64_t>(a.Xout) * a.Tout));
  }
  floatx4 acc[8][2];
#pragma unroll
  for (int nt = 0; nt < 8; ++nt) acc[nt][0] = acc[nt][1] = floatx4{0.f, 0.f, 0.f, 0.f};

  for (int32_t k0 = 8 * lg; k0 - 8 * lg < ktot; k0 += 32) {
    const bool kok = k0 < ktot;
    const int32_t tap = kok ? k0 / a.Cin : 0, c0 = kok ? k0 - tap * a.Cin : 0;
    const int32_t ky = tap / 3, kx = tap - 3 * ky;
    bf16x8 xf[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      const int32_t tv = pt[mt] * a.stride_t + ky - a.pad_top;
      const int32_t xv = px[mt] + kx - 1;
      const bool ok = kok && pok[mt] && tv >= 0 && tv < a.Tv && xv >= 0 && xv < a.Xv;
      if (ok) {
        const int32_t ts = a.Tv == a.Tin ? tv : static_cast<int32_t>((static_cast<int64_t>(tv) * a.Tin) / a.Tv);
        const int32_t xs = a.Xv == a.Xin ? xv : static_cast<int32_t>((static_cast<int64_t>(xv) * a.Xin) / a.Xv);
        xf[mt] = load8(a.in + ((static_cast<int64_t>(pb[mt]) * a.Tin + ts) * a.Xin + xs) * a.Cin + c0);
      } else {
        xf[mt] = zero8();
      }
    }
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
      if (nt < ntiles) {
        const int32_t co = cout0 + 16 * nt + lr;
        const bf16x8 wf = (kok && co < a.Cout) ? load8(a.w + static_cast<int64_t>(co) * ktot + k0) : zero8();
        acc[nt][0] = mfma16(wf, xf[0], acc[nt][0]);
        acc[nt][1] = mfma16(wf, xf[1], acc[nt][1]);
      }
    }
  }
  // epilogue: tile (nt, mt): rows = output channels cout0 + 16 nt + 4 lg + i, column = pixel lr of tile mt
#pragma unroll
  for (int nt = 0; nt < 8; ++nt) {
    if (nt >= ntiles) continue;
    const int32_t co = cout0 + 16 * nt + 4 * lg;
    if (co >= a.Cout) continue;
    float bv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bv[i] = co + i < a.Cout ? a.bias[co + i] : 0.f;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      if (!pok[mt]) continue;
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = acc[nt][mt][i] + bv[i];
        if (a.relu) v[i] = fmaxf(v[i], 0.f);
      }
      const int64_t p = pix0 + 16 * mt + lr;
      if (a.mode == 0) {
        uint2 pk = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + p * a.Cout + co) = pk;
      } else {
        float* o = static_cast<float*>(a.out);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (co + i < a.Cout)
            o[((static_cast<int64_t>(pb[mt]) * a.Cout + co + i) * a.Tout + pt[mt]) * a.Xout + px[mt]] = v[i];
      }
    }
  }
}

// softmax over the K entries of each row [B][H][T][K] in place; rows at or past seq_len -> 0
__global__ __launch_bounds__(256) void dec_softmax_kernel(float* __restrict__ A, const int32_t* __restrict__ seq_len,
                                                          int64_t rows, int32_t H, int32_t T, int32_t K) {
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int32_t t = static_cast<int32_t>(row % T);
  const int32_t b = static_cast<int32_t>(row / (static_cast<int64_t>(T) * H));
  const int32_t len = seq_len ? min(max(seq_len[b], 0), T) : T;
  float* r = A + row * K;
  if (t >= len) {
    for (int32_t c = lane; c < K; c += 64) r[c] = 0.f;
    return;
  }
  float mx = -INFINITY;
  for (int32_t c = lane; c < K; c += 64) mx = fmaxf(mx, r[c]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  float sum = 0.f;
  for (int32_t c = lane; c < K; c += 64) sum += __expf(r[c] - mx);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  const float inv = 1.f / sum;
  for (int32_t c = lane; c < K; c += 64) r[c] = __expf(r[c] - mx) * inv;
}

size_t up256(size_t b) { return (b + 255) & ~size_t(255); }

struct DecWs {
  size_t seg, Cp, img, y1, y2, total;
  int32_t T1, Wd, C;
};
DecWs dec_layout(const Shape& s) {
  DecWs w{};
  const size_t N = static_cast<size_t>(s.N), T = static_cast<size_t>(s.T), B = N / s.H;
  w.T1 = s.causal ? s.T : (s.T + kCs - 1) / kCs;
  w.Wd = s.K / kCs;
  w.C = s.H * kCh;
  size_t off = 0;
  w.seg = off; off += up256(dec_linattn_state_bytes(s));
  w.Cp = off; off += up256(N * T * 128 * 2);
  w.img = off; off += up256(B * T * w.Wd * w.C * 2);
  w.y1 = off; off += up256(B * static_cast<size_t>(w.T1) * w.Wd * w.C * 2);
  w.y2 = off; off += up256(B * static_cast<size_t>(w.T1) * w.Wd * w.C * 2);
  w.total = off;
  return w;
}

// ------------------------------------------------------------------------------------------
// 3x3 convolutions with the input window in LDS.  A block of eight waves computes a tile of output
// pixels (each wave 64 of them: RW rows x CW columns, RW CW = 64) for a slab of up to 16 NT output
// channels.  The tile's input halo -- every (virtual, i.e. resized) pixel any of its taps touches,
// zeros outside the image -- and the slab's weights are parked in LDS once per channel chunk, the
// weights in operand-fragment order, the pixels with an odd number of 16-byte units per pixel so
// that the 16 pixels of an operand tile hit different banks.  Each input pixel is then read from
// memory once per tile instead of once per tap.  The contraction runs over (tap, channel) of the
// chunk flattened in units of 8 channels, one unit per lane group and step; a lane advances its own
// (tap, unit) position without divisions.
// ------------------------------------------------------------------------------------------
struct Conv3Args {
  ConvArgs a;
  int32_t t_shift, x_shift;      // log2 of the nearest-resize ratios (virtual / stored size)
  int32_t CK, nchunk, P, pp_log; // channels per chunk, chunks, 16-byte units per pixel and chunk, log2 of P rounded up
  int32_t ksteps;                // contraction steps per chunk
  int32_t cw_log;                // log2 of the columns a wave covers (4..6); rows per wave = 64 >> cw_log
  int32_t rows_out, cols_out, halo_rows, halo_cols, px_units;  // tile geometry; px_units odd
  int32_t tiles_t, tiles_x;
};
constexpr int kConv3Waves = 8;

template <int NT>
__global__ __launch_bounds__(64 * kConv3Waves) void dec_conv3_kernel(Conv3Args g) {
  extern __shared__ __attribute__((aligned(16))) uint4 lds3[];
  const ConvArgs& a = g.a;
  uint4* halo = lds3;                                                        // [halo_rows][halo_cols][px_units]
  uint4* wts = lds3 + static_cast<int64_t>(g.halo_rows) * g.halo_cols * g.px_units;  // [kstep][NT][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  uint32_t bid = blockIdx.x;
  const int32_t tx = static_cast<int32_t>(bid % static_cast<uint32_t>(g.tiles_x)); bid /= static_cast<uint32_t>(g.tiles_x);
  const int32_t tt = static_cast<int32_t>(bid % static_cast<uint32_t>(g.tiles_t));
  const int64_t b = bid / static_cast<uint32_t>(g.tiles_t);
  const int32_t t0 = tt * g.rows_out, x0 = tx * g.cols_out;     // first output pixel of the tile
  const int32_t tv0 = t0 * a.stride_t - a.pad_top, xv0 = x0 - 1;  // first virtual input pixel of the halo
  const int32_t cout0 = blockIdx.y * (16 * NT);
  const int32_t ktot = 9 * a.Cin;
  const uint16_t* img = a.in + b * a.Tin * a.Xin * a.Cin;

  floatx4 acc[NT][4];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  // this lane's pixel in each of the wave's four operand tiles: row and column inside the output tile
  const int rw = 64 >> g.cw_log, ctiles = (1 << g.cw_log) >> 4;  // rows per wave, 16-pixel tiles per row
  int32_t prow[4], pcol[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    prow[mt] = wid * rw + mt / ctiles;
    pcol[mt] = (mt % ctiles) * 16 + lr;
  }

  for (int32_t ch = 0; ch < g.nchunk; ++ch) {
    if (ch > 0) __syncthreads();  // the previous chunk is no longer read
    const int32_t cbase = ch * g.CK;
    // halo: thread = (pixel, 16-byte unit); units past P idle
    {
      const int32_t unit = tid & ((1 << g.pp_log) - 1);
      const int32_t npx = g.halo_rows * g.halo_cols;
      for (int32_t px = tid >> g.pp_log; px < npx; px += (64 * kConv3Waves) >> g.pp_log) {
        if (unit >= g.P) continue;
        const int32_t hr = px / g.halo_cols, hc = px - hr * g.halo_cols;
        const int32_t tv = tv0 + hr, xv = xv0 + hc;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (static_cast<uint32_t>(tv) < static_cast<uint32_t>(a.Tv) && static_cast<uint32_t>(xv) < static_cast<uint32_t>(a.Xv)) {
          const int32_t ts = tv >> g.t_shift, xs = xv >> g.x_shift;
          v = *reinterpret_cast<const uint4*>(img + (static_cast<int64_t>(ts) * a.Xin + xs) * a.Cin + cbase + 8 * unit);
        }
        halo[static_cast<int64_t>(px) * g.px_units + unit] = v;
      }
    }
    // weights of the chunk: fragment (step, tile, lane) = channels cbase + 8 cu .. + 7 of tap `tap` for
    // output channel cout0 + 16 nt + lane % 16, with (tap, cu) = unit 4 step + lane / 16 of the chunk
    for (int32_t id = tid; id < g.ksteps * NT * 64; id += 64 * kConv3Waves) {
      const int32_t fl = id & 63, q = id >> 6, nt = q % NT, ks = q / NT;
      const int32_t u = 4 * ks + (fl >> 4), tap = u / g.P, cu = u - tap * g.P;
      const int32_t co = cout0 + 16 * nt + (fl & 15);
      uint4 v = make_uint4(0u, 0u, 0u, 0u);
      if (tap < 9 && co < a.Cout)
        v = *reinterpret_cast<const uint4*>(a.w + static_cast<int64_t>(co) * ktot + tap * a.Cin + cbase + 8 * cu);
      wts[id] = v;
    }
    __syncthreads();
    int32_t tap = 0, cu = lg;
    while (cu >= g.P) { cu -= g.P; ++tap; }
    for (int32_t ks = 0; ks < g.ksteps; ++ks) {
      const bool valid = tap < 9;
      const int32_t ky = (tap * 11) >> 5, kx = tap - 3 * ky;  // tap / 3 and tap % 3 for tap <= 8
      bf16x8 xf[4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int32_t hr = prow[mt] * a.stride_t + ky, hc = pcol[mt] + kx;
        const uint4 v = halo[valid ? (static_cast<int64_t>(hr) * g.halo_cols + hc) * g.px_units + cu : 0];
        xf[mt] = valid ? __builtin_bit_cast(bf16x8, v) : zero8();
      }
      const uint4* wk = wts + (static_cast<int64_t>(ks) * NT) * 64 + lane;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const bf16x8 wf = __builtin_bit_cast(bf16x8, wk[nt * 64]);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = mfma16(wf, xf[mt], acc[nt][mt]);
      }
      cu += 4;
      while (cu >= g.P) { cu -= g.P; ++tap; }
    }
  }
  // epilogue: tile (nt, mt): rows = output channels cout0 + 16 nt + 4 lg + i, column = this lane's pixel of tile mt
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int32_t co = cout0 + 16 * nt + 4 * lg;
    if (co >= a.Cout) continue;
    float bv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bv[i] = co + i < a.Cout ? a.bias[co + i] : 0.f;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const int32_t t = t0 + prow[mt], x = x0 + pcol[mt];
      if (prow[mt] >= g.rows_out || pcol[mt] >= g.cols_out || t >= a.Tout || x >= a.Xout) continue;
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = acc[nt][mt][i] + bv[i];
        if (a.relu) v[i] = fmaxf(v[i], 0.f);
      }
      if (a.mode == 0) {
        const uint2 pk = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + ((b * a.Tout + t) * a.Xout + x) * a.Cout + co) = pk;
      } else {
        float* o = static_cast<float*>(a.out);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (co + i < a.Cout) o[((b * a.Cout + co + i) * a.Tout + t) * a.Xout + x] = v[i];
      }
    }
  }
}

// log2 of virtual / stored size when that ratio is a power of two, else -1
int32_t resize_shift(int32_t vsize, int32_t size) {
  for (int32_t sh = 0; sh < 16; ++sh)
    if ((static_cast<int64_t>(size) << sh) == vsize) return sh;
  return -1;
}

// Geometry of the LDS-window kernel for one layer; false when the layer does not fit it (then the
// direct kernels run).  The channel chunk is the largest divisor of Cin (in units of 8 channels)
// whose halo and weights fit the LDS budget.
constexpr size_t kConv3LdsBudget = 72 << 10;  // two blocks per CU overlap one block's staging with the other's products
bool conv3_plan(const ConvArgs& a, Conv3Args* g, int32_t* nt_out, size_t* lds_out) {
  if (a.Cin % 8 != 0) return false;
  if (a.mode == 0 && a.Cout % 4 != 0) return false;
  const int32_t ts = resize_shift(a.Tv, a.Tin), xs = resize_shift(a.Xv, a.Xin);
  if (ts < 0 || xs < 0) return false;
  const int32_t slab = a.Cout < 128 ? a.Cout : 128;
  const int32_t nt = (slab + 15) / 16;
  int32_t cw_log = 6;
  while (cw_log > 4 && (1 << (cw_log - 1)) >= a.Xout) --cw_log;
  const int32_t rows_out = kConv3Waves * (64 >> cw_log), cols_out = 1 << cw_log;
  const int32_t halo_rows = (rows_out - 1) * a.stride_t + 3, halo_cols = cols_out + 2;
  const int32_t units = a.Cin / 8;
  for (int32_t nchunk = 1; nchunk <= units; ++nchunk) {
    if (units % nchunk != 0) continue;
    const int32_t P = units / nchunk;
    const int32_t px_units = P | 1;
    const int32_t ksteps = (9 * P + 3) / 4;
    const size_t lds = (static_cast<size_t>(halo_rows) * halo_cols * px_units + static_cast<size_t>(ksteps) * nt * 64) * 16;
    if (lds > kConv3LdsBudget) continue;
    int32_t pp_log = 0;
    while ((1 << pp_log) < P) ++pp_log;
    g->a = a; g->t_shift = ts; g->x_shift = xs; g->CK = 8 * P; g->nchunk = nchunk; g->P = P; g->pp_log = pp_log;
    g->ksteps = ksteps; g->cw_log = cw_log; g->rows_out = rows_out; g->cols_out = cols_out;
    g->halo_rows = halo_rows; g->halo_cols = halo_cols; g->px_units = px_units;
    g->tiles_t = (a.Tout + rows_out - 1) / rows_out; g->tiles_x = (a.Xout + cols_out - 1) / cols_out;
    *nt_out = nt; *lds_out = lds;
    return true;
  }
  return false;
}

// a failed attribute call stays the runtime's last error, which the caller reports
template <int NT>
void launch_conv3(const Conv3Args& g, uint32_t slabs, size_t lds, hipStream_t st) {
  if (lds > (64u << 10) &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(&dec_conv3_kernel<NT>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
    return;
  const uint32_t blocks = static_cast<uint32_t>(g.a.B) * g.tiles_t * g.tiles_x;
  hipLaunchKernelGGL(dec_conv3_kernel<NT>, dim3(blocks, slabs), dim3(64 * kConv3Waves), lds, st, g);
}

void launch_conv(const ConvArgs& a, hipStream_t st) {
  const int64_t npix = static_cast<int64_t>(a.B) * a.Tout * a.Xout;
  Conv3Args g{};
  int32_t nt = 0;
  size_t lds = 0;
  if (conv3_plan(a, &g, &nt, &lds)) {
    const uint32_t slabs3 = static_cast<uint32_t>((a.Cout + 16 * nt - 1) / (16 * nt));
    switch (nt) {
      case 1: launch_conv3<1>(g, slabs3, lds, st); break;
      case 2: launch_conv3<2>(g, slabs3, lds, st); break;
      case 3: launch_conv3<3>(g, slabs3, lds, st); break;
      case 4: launch_conv3<4>(g, slabs3, lds, st); break;
      case 5: launch_conv3<5>(g, slabs3, lds, st); break;
      case 6: launch_conv3<6>(g, slabs3, lds, st); break;
      case 7: launch_conv3<7>(g, slabs3, lds, st); break;
      default: launch_conv3<8>(g, slabs3, lds, st); break;
    }
    return;
  }
  const uint32_t slabs = static_cast<uint32_t>((a.Cout + 127) / 128);
  if (a.Cout >= 96 && 9 * a.Cin >= 512) {
    hipLaunchKernelGGL(dec_conv_lds_kernel, dim3(static_cast<uint32_t>((npix + 255) / 256), slabs), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL(dec_conv_kernel, dim3(static_cast<uint32_t>((npix + 127) / 128), slabs), dim3(256), 0, st, a);
  }
}

}  // namespace

namespace {
// conv 1 or 2: the kernel with all weights in LDS where the layer fits it, else the channel-chunked one
hipError_t conv_layer(const DecConv& c, uint16_t* out, hipStream_t st) {
  const hipError_t e = launch_dec_conv(c, out, st);
  if (e != hipErrorNotSupported) return e;
  ConvArgs a{};
  a.in = c.in; a.w = c.w; a.bias = c.bias; a.out = out; a.B = c.B; a.Cin = c.Cin; a.Cout = c.Cout;
  a.Tin = a.Tv = c.Tin; a.Tout = c.Tout; a.Xin = a.Xv = a.Xout = c.X;
  a.stride_t = c.stride_t; a.pad_top = c.pad_top; a.relu = 1; a.mode = 0;
  launch_conv(a, st);
  return hipGetLastError();
}
}  // namespace

bool decoder_supported(const Shape& s, sea_dtype dt) {
  if (dt != SEA_BF16) return false;
  if (s.m != 64 && s.m != 128 && s.m != 256) return false;
  if (s.K % kCs != 0 || s.K > 1024) return false;
  if ((s.H * kCh) % 8 != 0) return false;  // operand fragments are 8 channels
  if (s.geometry != 0) return false;
  return true;
}

size_t decoder_workspace(const Shape& s) { return dec_layout(s).total; }

hipError_t launch_decoder_estimate(const Shape& s, const sea_decoder_weights& wt, const uint16_t* Q, const uint16_t* K,
                                   const uint16_t* V, const uint16_t* W, float* A_hat, float* s_mix, float* s_prob,
                                   void* ws, hipStream_t st) {
  if (!decoder_supported(s, SEA_BF16)) return hipErrorNotSupported;
  if (static_cast<int64_t>(s.N) * s.T >> 32) return hipErrorNotSupported;  // (Q, K and V of so many rows are 1.6 TB)
  const DecWs lay = dec_layout(s);
  char* base = static_cast<char*>(ws);
  auto u16 = [&](size_t off) { return reinterpret_cast<uint16_t*>(base + off); };
  const double l2e = 1.4426950408889634;
  const float c_dot = static_cast<float>(l2e * sqrt(static_cast<double>(s.scale)));
  const float c_norm = static_cast<float>(l2e * 0.5 * static_cast<double>(s.scale));
  const int32_t B = s.N / s.H;
  const int64_t rows = static_cast<int64_t>(s.N) * s.T;
  hipError_t e;
  {
    StageScope scope(SEA_STAGE_STATE, st);
    e = launch_dec_linattn(s, Q, K, V, W, u16(lay.Cp), base + lay.seg, c_dot, c_norm, st);
    if (e != hipSuccess) return e;
  }
  StageScope scope(SEA_STAGE_CONTRACT, st);
  // mu, nu and the scalers: rows [C_perf; V] -> the CNN's input image [B][T][Wd][C], channels h c_h + ch
  e = launch_dec_mlp(s, wt, u16(lay.Cp), V, u16(lay.img), s_mix, s_prob, st);
  if (e != hipSuccess) return e;
  if (s.causal) {  // (the strips of the one launch look back only)
    DecChain n{};
    n.in = u16(lay.img);
    n.w[0] = static_cast<const uint16_t*>(wt.conv1_w); n.bias[0] = wt.conv1_b;
    n.w[1] = static_cast<const uint16_t*>(wt.conv2_w); n.bias[1] = wt.conv2_b;
    n.w[2] = static_cast<const uint16_t*>(wt.conv3_w); n.bias[2] = wt.conv3_b;
    n.B = B; n.T = s.T; n.X = lay.Wd; n.H = s.H;
    if ((e = launch_dec_chain(n, A_hat, s.seq_len, st)) != hipErrorNotSupported) return e;
  }
  // conv 1: [B][T][Wd][C] -> [B][T1][Wd][C], ReLU.  Causal: rows t-2..t; else stride c_s, rows i c_s - 1 .. + 1
  DecConv c{};
  c.in = u16(lay.img); c.w = static_cast<const uint16_t*>(wt.conv1_w); c.bias = wt.conv1_b;
  c.B = B; c.Tin = s.T; c.X = lay.Wd; c.Cin = c.Cout = lay.C; c.Tout = lay.T1;
  c.stride_t = s.causal ? 1 : kCs; c.pad_top = s.causal ? 2 : 1;
  if ((e = conv_layer(c, u16(lay.y1), st)) != hipSuccess) return e;
  // conv 2
  c.in = u16(lay.y1); c.w = static_cast<const uint16_t*>(wt.conv2_w); c.bias = wt.conv2_b;
  c.Tin = lay.T1; c.stride_t = 1;
  if ((e = conv_layer(c, u16(lay.y2), st)) != hipSuccess) return e;
  // conv 3 on the image resized to T x K (nearest, on the read) and the softmax of its rows
  c.in = u16(lay.y2); c.w = static_cast<const uint16_t*>(wt.conv3_w); c.bias = wt.conv3_b;
  c.Tout = s.T; c.Cout = s.H;
  e = launch_dec_conv_softmax(c, s.T, A_hat, s.seq_len, st);
  if (e != hipErrorNotSupported) return e;
  ConvArgs a{};
  a.in = c.in; a.w = c.w; a.bias = c.bias; a.out = A_hat; a.B = B; a.Cin = lay.C; a.Cout = s.H;
  a.Tin = lay.T1; a.Xin = lay.Wd; a.Tv = a.Tout = s.T; a.Xv = a.Xout = s.K;
  a.stride_t = 1; a.pad_top = c.pad_top; a.relu = 0; a.mode = 2;
  launch_conv(a, st);
  hipLaunchKernelGGL(dec_softmax_kernel, dim3(static_cast<uint32_t>((rows + 3) / 4)), dim3(256), 0, st, A_hat, s.seq_len,
                     rows, s.H, s.T, s.K);
  return hipGetLastError();
}

}  // namespace sea
