// The decoder's MLPs in one kernel (Sec. 3.1 "CNN Decoder": mu on [C_perf; V], nu on mu's output; and the
// scalers s_mix, s_prob of Sec. 3.1.1 "Output Calculation"): a wave takes 32 rows through
//   Z = relu(mu_w [C_perf; V] + mu_b), (s_mix, s_prob) = sigmoid(w . Z + b), hidden = relu(nu1_w Z + nu1_b),
//   image = nu2_w hidden + nu2_b
// without leaving its registers.  Every product is taken transposed, C[channel][row] = weights x rows^T, so
// an accumulator tile (lane = row l % 16, registers = channels 4 (l / 16) + i) packed in pairs is the
// operand of the next layer, with contraction slot 8 g + e of a 32-channel step meaning channel
// 16 (e / 4) + 4 g + e % 4; the weights of nu are parked in that order.  All weights live in LDS (148 KB for
// K = 128: one block of twelve waves per CU); more than 256 outputs of nu go through in slabs.
// Z and the hidden layer are rounded to bf16 as the layers are defined.
//
// Bound: memory latency (reads 2 x 192, writes 8 K / 2 bytes per row; 3 TB/s are moved).  B = 4, H = 12, T = 2048, K = 128:
// 0.14 -> 0.04 ms; before, the concatenated rows, Z and the hidden layer made a round trip each and the scalers read Z again.
// Twelve waves with a CU's neighbouring tiles dealt to them, the next tile's rows requested into the registers that the
// first layer has just read, against eight with a register set of their own for the next tile: 37.6 -> 31.7 us there (12
// tiles per CU: one round instead of a full and a half one).  Tiles dealt over all blocks instead: 34.7, and the
// convolution that follows waits for lines written by several XCDs (bidirectional layer 152 -> 158 us).
// The weights a block stages are asked for in whole lines and all at once, before most rows: 30.3 -> 27.2 us there, K = 256 48 -> 42,
// K = 64, T = 256, B = 1 13.2 -> 12.2 (before, a loop of one piece per thread after the other; with the rows of all waves in front,
// the barrier behind the weights waits for those too).
#include "sea_decoder.h"

namespace sea {
namespace {

constexpr int kCpDim = 128;   // [V_I; V] through the Performer: two value widths
constexpr int kMlpWaves = 12, kMlpThreads = 64 * kMlpWaves;
constexpr int kEarly = 4;                      // waves that ask for their rows in front of the weights: as many as do not hold those up
constexpr int kMuSteps = 6, kHidSteps = 4;     // contraction steps of 32: 192 and 128 channels
constexpr int kNu1Tiles = 9;                   // 128 outputs + one tile for the scalers
constexpr int kSlabTiles = 16;                 // 256 outputs of nu's last layer per slab

struct MlpArgs {
  const uint16_t* Cp;   // C_perf rows, kCpDim wide
  const uint16_t* V;    // value rows, kHeadDim wide
  const uint16_t *mu_w, *nu1_w, *nu2_w, *mix_w, *prob_w;
  const float *mu_b, *nu1_b, *nu2_b, *mix_b, *prob_b;
  uint16_t* img;        // [B][T][Wd][C]
  float *s_mix, *s_prob;
  const int32_t* seq_len;
  int32_t H, T, Wd, C;
  int64_t rows;         // B T H
  int32_t out2;         // outputs of nu's last layer, 4 Wd
  int64_t per_block;    // 32-row tiles of a block, neighbours
};

__global__ __launch_bounds__(kMlpThreads, 3) void dec_mlp_kernel(MlpArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint4 mlp_lds[];
  uint4* w_mu = mlp_lds;                                  // [6][8][64]
  uint4* w_nu1 = w_mu + kMuSteps * 8 * 64;                // [4][9][64]
  float* b_mu = reinterpret_cast<float*>(w_nu1 + kHidSteps * kNu1Tiles * 64);  // biases: 128, 128, 16 per tile of the slab
  float* b_nu1 = b_mu + 128;
  float* b_nu2 = b_nu1 + 128;
  uint4* w_nu2 = reinterpret_cast<uint4*>(b_nu2 + 16 * kSlabTiles);            // [4][tiles][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int32_t slabs = (a.out2 + 16 * kSlabTiles - 1) / (16 * kSlabTiles);
  const int32_t slab_tiles = min(kSlabTiles, (a.out2 + 15) / 16);
  float* b_sc = reinterpret_cast<float*>(w_nu2 + kHidSteps * slab_tiles * 64);  // the scalers'

  // Weights are read as they lie, a kilobyte of whole lines per wave (sixteen rows' 64-byte pieces at a time cost 80 clocks a load,
  // with every CU at the same lines), all of them asked for before any is waited for, and take their order on the way to LDS.
  // nu's rows of 128 channels in the order of packed accumulators: 16 bytes are the halves of two operands.
  auto park_nu = [&](uint4* w, int32_t tiles, int32_t piece, uint4 v) __attribute__((always_inline)) {
    const int32_t row = piece >> 4, p = piece & 15, half = (p >> 1) & 1;
    uint2* const at = reinterpret_cast<uint2*>(w + ((p >> 2) * tiles + (row >> 4)) * 64 + 32 * (p & 1) + (row & 15)) + half;
    at[0] = make_uint2(v.x, v.y);
    at[32] = make_uint2(v.z, v.w);
  };
  auto nu2_piece = [&](int32_t slab, int32_t piece) __attribute__((always_inline)) {
    const int32_t co = slab * 16 * kSlabTiles + (piece >> 4);
    const uint4 v = reinterpret_cast<const uint4*>(a.nu2_w)[static_cast<int64_t>(min(co, a.out2 - 1)) * 16 + (piece & 15)];
    return co < a.out2 ? v : make_uint4(0u, 0u, 0u, 0u);
  };
  auto nu2_bias = [&](int32_t slab) { return a.nu2_b[min(slab * 16 * kSlabTiles + min(tid, 16 * slab_tiles - 1), a.out2 - 1)]; };
  auto stage_nu2 = [&](int32_t slab) {
    for (int32_t id = tid; id < 256 * slab_tiles; id += kMlpThreads) park_nu(w_nu2, slab_tiles, id, nu2_piece(slab, id));
    if (tid < 16 * slab_tiles) b_nu2[tid] = nu2_bias(slab);
  };

  const int64_t first = blockIdx.x * a.per_block, end = min(first + a.per_block, (a.rows + 31) / 32);
  // rows in the order (b, t, h), heads fastest: a wave's stores lie next to each other in the image.  Their numbers are split in
  // 32 bits, which the caller has seen to (a 64-bit division is a hundred instructions)
  auto split = [&](int64_t at, int32_t* h, int32_t* t, int32_t* b) {
    const uint32_t pp = static_cast<uint32_t>(at), H = static_cast<uint32_t>(a.H), T = static_cast<uint32_t>(a.T), q = pp / H;
    *h = static_cast<int32_t>(pp - q * H);
    *b = static_cast<int32_t>(q / T);
    *t = static_cast<int32_t>(q - static_cast<uint32_t>(*b) * T);
  };
  bf16x8 xf[kMuSteps][2];
  auto request = [&](int64_t tile) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      int32_t h, t, b;
      split(min(tile * 32 + 16 * mt + lr, a.rows - 1), &h, &t, &b);
      const int64_t r = (static_cast<int64_t>(b) * a.H + h) * a.T + t;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) xf[ks][mt] = load8(a.Cp + r * kCpDim + 32 * ks + 8 * lg);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) xf[4 + ks][mt] = load8(a.V + r * kHeadDim + 32 * ks + 8 * lg);
    }
  };
  const int64_t tile0 = first + wid;
  if (wid < kEarly && tile0 < end) request(tile0);
  {
    constexpr int kMu = 128 * 24 / kMlpThreads, kNu1 = (128 * 16 + kMlpThreads - 1) / kMlpThreads;
    constexpr int kNu2 = (16 * kSlabTiles * 16 + kMlpThreads - 1) / kMlpThreads;
    static_assert(kMu * kMlpThreads == 128 * 24, "whole rounds");
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 mu[kMu];  // (an array of uint4 that is only copied ends up in scratch memory)
    uint4 nu1[kNu1], nu2[kNu2];
#pragma unroll
    for (int e = 0; e < kMu; ++e) mu[e] = reinterpret_cast<const u32x4*>(a.mu_w)[static_cast<uint32_t>(tid + kMlpThreads * e)];
#pragma unroll
    for (int e = 0; e < kNu1; ++e) nu1[e] = reinterpret_cast<const uint4*>(a.nu1_w)[static_cast<uint32_t>(min(tid + kMlpThreads * e, 128 * 16 - 1))];
#pragma unroll
    for (int e = 0; e < kNu2; ++e) nu2[e] = nu2_piece(0, min(tid + kMlpThreads * e, 256 * slab_tiles - 1));
    // the scalers' vectors, whose alignment is only that of a pair: rows 0 and 1 of nu1's ninth tile
    const uint32_t* const sv = reinterpret_cast<const uint32_t*>(lr & 1 ? a.prob_w : a.mix_w) + 16 * (wid & 3) + 2 * lg;
    const uint4 sc = make_uint4(sv[0], sv[1], sv[8], sv[9]);
    const float* const bp = tid < 128 ? a.mu_b + tid : (tid < 256 ? a.nu1_b + tid - 128 : (tid == 256 ? a.mix_b : a.prob_b));
    const float bias = *bp, bias2 = nu2_bias(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < kMu; ++e) {
      const int32_t id = tid + kMlpThreads * e, row = id / 24, p = id - row * 24;
      reinterpret_cast<u32x4*>(w_mu)[((p >> 2) * 8 + (row >> 4)) * 64 + 16 * (p & 3) + (row & 15)] = mu[e];
    }
#pragma unroll
    for (int e = 0; e < kNu1; ++e)
      if (tid + kMlpThreads * e < 128 * 16) park_nu(w_nu1, kNu1Tiles, tid + kMlpThreads * e, nu1[e]);
    if (wid < 4) w_nu1[(wid * kNu1Tiles + 8) * 64 + lane] = lr < 2 ? sc : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int e = 0; e < kNu2; ++e)
      if (tid + kMlpThreads * e < 256 * slab_tiles) park_nu(w_nu2, slab_tiles, tid + kMlpThreads * e, nu2[e]);
    if (tid < 258) (tid < 256 ? b_mu : b_sc - 256)[tid] = bias;  // (nu1's follow mu's)
    if (tid < 16 * slab_tiles) b_nu2[tid] = bias2;
  }
  __syncthreads();
  if (wid >= kEarly && tile0 < end) request(tile0);
  // with one slab the loop has no barrier and a wave without a tile leaves it; with several, every wave of
  // the block stays for the barriers of the staging (the first wave's tile is the smallest)
  for (int64_t tile = tile0; slabs == 1 ? tile < end : tile - wid < end; tile += kMlpWaves) {
    const bool on = tile < end;  // wave-uniform
    bf16x8 zf[kHidSteps][2];
    int64_t orow[2];
    bool live[2], exists[2];
    if (on) {
      // mu, two 16-channel tiles at a time
#pragma unroll
      for (int kc = 0; kc < kHidSteps; ++kc) {
        floatx4 acc[2][2];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const float4 bv = *reinterpret_cast<const float4*>(b_mu + 16 * (2 * kc + hf) + 4 * lg);
          acc[hf][0] = acc[hf][1] = floatx4{bv.x, bv.y, bv.z, bv.w};
        }
#pragma unroll
        for (int ks = 0; ks < kMuSteps; ++ks)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            const bf16x8 wf = __builtin_bit_cast(bf16x8, w_mu[(ks * 8 + 2 * kc + hf) * 64 + lane]);
            acc[hf][0] = mfma16(wf, xf[ks][0], acc[hf][0]);
            acc[hf][1] = mfma16(wf, xf[ks][1], acc[hf][1]);
          }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) zf[kc][mt] = pack8(relu4(acc[0][mt]), relu4(acc[1][mt]));
      }
      int32_t hh[2], tt[2], bb[2], lens[2];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        split(min(tile * 32 + 16 * mt + lr, a.rows - 1), &hh[mt], &tt[mt], &bb[mt]);
        lens[mt] = a.seq_len ? a.seq_len[bb[mt]] : a.T;
      }
      if (tile + kMlpWaves < end) request(tile + kMlpWaves);  // the rows have left their registers
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const int64_t pp = tile * 32 + 16 * mt + lr;
        const int32_t h = hh[mt], t = tt[mt], b = bb[mt], len = min(max(lens[mt], 0), a.T);
        exists[mt] = pp < a.rows;
        live[mt] = t < len;
        orow[mt] = (static_cast<int64_t>(b) * a.T + t) * a.Wd * a.C + h * 4;
        // the scalers: rows 0 and 1 of nu1's ninth tile
        floatx4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < kHidSteps; ++kc)
          sc = mfma16(__builtin_bit_cast(bf16x8, w_nu1[(kc * kNu1Tiles + 8) * 64 + lane]), zf[kc][mt], sc);
        if (lg == 0 && exists[mt]) {
          const int64_t r = (static_cast<int64_t>(b) * a.H + h) * a.T + t;
          if (a.s_mix) a.s_mix[r] = live[mt] ? 1.f / (1.f + __expf(-(sc[0] + b_sc[0]))) : 0.f;
          if (a.s_prob) a.s_prob[r] = live[mt] ? 1.f / (1.f + __expf(-(sc[1] + b_sc[1]))) : 0.f;
        }
      }
      // nu, first layer
      bf16x8 hf8[kHidSteps][2];
#pragma unroll
      for (int kc = 0; kc < kHidSteps; ++kc) {
        floatx4 acc[2][2];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const float4 bv = *reinterpret_cast<const float4*>(b_nu1 + 16 * (2 * kc + hf) + 4 * lg);
          acc[hf][0] = acc[hf][1] = floatx4{bv.x, bv.y, bv.z, bv.w};
        }
#pragma unroll
        for (int ks = 0; ks < kHidSteps; ++ks)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            const bf16x8 wf = __builtin_bit_cast(bf16x8, w_nu1[(ks * kNu1Tiles + 2 * kc + hf) * 64 + lane]);
            acc[hf][0] = mfma16(wf, zf[ks][0], acc[hf][0]);
            acc[hf][1] = mfma16(wf, zf[ks][1], acc[hf][1]);
          }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) hf8[kc][mt] = pack8(relu4(acc[0][mt]), relu4(acc[1][mt]));
      }
#pragma unroll
      for (int kc = 0; kc < kHidSteps; ++kc) { zf[kc][0] = hf8[kc][0]; zf[kc][1] = hf8[kc][1]; }
    }
    // nu, last layer: outputs 4 x .. 4 x + 3 of a row are the row's head's channels of image column x
    for (int32_t slab = 0; slab < slabs; ++slab) {
      if (slabs > 1) {
        __syncthreads();
        stage_nu2(slab);
        __syncthreads();
      }
      if (!on) continue;
      for (int32_t nt = 0; nt < slab_tiles; ++nt) {
        const int32_t co = (slab * kSlabTiles + nt) * 16 + 4 * lg;
        const float4 bv = *reinterpret_cast<const float4*>(b_nu2 + 16 * nt + 4 * lg);
        floatx4 acc[2];
        acc[0] = acc[1] = floatx4{bv.x, bv.y, bv.z, bv.w};
#pragma unroll
        for (int ks = 0; ks < kHidSteps; ++ks) {
          const bf16x8 wf = __builtin_bit_cast(bf16x8, w_nu2[(ks * slab_tiles + nt) * 64 + lane]);
          acc[0] = mfma16(wf, zf[ks][0], acc[0]);
          acc[1] = mfma16(wf, zf[ks][1], acc[1]);
        }
        if (co >= a.out2) continue;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          uint2 pk = {pack_bf16(acc[mt][0], acc[mt][1]), pack_bf16(acc[mt][2], acc[mt][3])};
          if (!live[mt]) pk = make_uint2(0u, 0u);
          if (exists[mt]) *reinterpret_cast<uint2*>(a.img + orow[mt] + static_cast<int64_t>(co >> 2) * a.C) = pk;
        }
      }
    }
  }
}

}  // namespace

hipError_t launch_dec_mlp(const Shape& s, const sea_decoder_weights& wt, const uint16_t* Cp, const uint16_t* V,
                          uint16_t* img, float* s_mix, float* s_prob, hipStream_t st) {
  MlpArgs a{};
  auto u16 = [](const void* p) { return static_cast<const uint16_t*>(p); };
  a.Cp = Cp; a.V = V;
  a.mu_w = u16(wt.mu_w); a.nu1_w = u16(wt.nu1_w); a.nu2_w = u16(wt.nu2_w); a.mix_w = u16(wt.mix_w); a.prob_w = u16(wt.prob_w);
  a.mu_b = wt.mu_b; a.nu1_b = wt.nu1_b; a.nu2_b = wt.nu2_b; a.mix_b = wt.mix_b; a.prob_b = wt.prob_b;
  a.img = img; a.s_mix = s_mix; a.s_prob = s_prob; a.seq_len = s.seq_len;
  a.H = s.H; a.T = s.T; a.Wd = s.K / 2; a.C = 4 * s.H; a.rows = static_cast<int64_t>(s.N) * s.T; a.out2 = 4 * a.Wd;
  const int32_t slab_tiles = std::min(kSlabTiles, (a.out2 + 15) / 16);
  const size_t lds = static_cast<size_t>(kMuSteps * 8 + kHidSteps * kNu1Tiles + kHidSteps * slab_tiles) * 1024 +
                     (256 + 16 * kSlabTiles + 2) * sizeof(float);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dec_mlp_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  // an equal share of the tiles for each CU: small launches use all of them, with few waves each
  const int64_t tiles = (a.rows + 31) / 32;
  a.per_block = (tiles + 255) / 256;
  hipLaunchKernelGGL(dec_mlp_kernel, dim3(static_cast<uint32_t>((tiles + a.per_block - 1) / a.per_block)), dim3(kMlpThreads), lds, st, a);
  return hipGetLastError();
}

}  // namespace sea
