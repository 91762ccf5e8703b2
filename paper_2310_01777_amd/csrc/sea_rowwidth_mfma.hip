// Per-row width estimate for bf16 tensors on the bf16 matrix cores (App. A.4: a causal row t is
// resized to its own width, so its column c holds the keys [ceil(c (t+1) / K), ceil((c+1)(t+1) / K));
// Sec. 3 "Performer (FAVOR+)", Sec. 3.1 "Attention Matrix Estimation").
//
//   A^[t][c] = sum over the keys j of row t's column c of  phi~(q_t) . phi~(k_j),  then / row sum
//
// with phi~ the features rounded to bf16 (queries after a power-of-two row shift).  The products
// a_tj of 32 query rows x 32 keys are a tile of phi~(K) phi~(Q)^T (v_mfma_f32_32x32x16_bf16,
// fp32 accumulation); every a_tj is then added to the bin of its column floor(j K / (t + 1)) in LDS.
// Nothing is differenced, so there is no cancellation, and no prefix state exists.  The bins are
// fp64: the LDS adds 64 doubles in about 11 clocks but needs about 170 for 64 floats (measured,
// ds_add_f64 against ds_add_f32; with fp32 bins nothing else bounded this kernel).  Bound: key features from the
// L2, products and binning take turns in a wave (B = 4, H = 12, T = 2048, m = K = 128 with the selection: vector pipe
// 50 %, matrix pipe 13 %, LDS 15 % busy, 2.8 waves per SIMD).
//
//   rw_features_kernel   phi~(Q), phi~(K) -> HBM, already in the order the tile kernel's lanes
//                        consume them: [head][32-token chunk][step][lane][8 features], so every
//                        operand load of the tile kernel is one contiguous 1 KB piece
//   rw_tiles_mfma_kernel one wavefront per (head, 32 or 64 query rows, column part): walks the 32-key
//                        chunks its columns cover, bins, normalises, writes fp32 A^
//
// Column parts: a wave keeps the bins of at most 32 columns ([32 rows][<= 32] fp64 = 9 KB), so that
// a CU holds sixteen waves, four per SIMD; the ceil(K / 32) parts of a row tile are taken by the (at
// most eight) waves of one block, which meet only for the row sums.  The columns of a row are monotone in the key index, so part p walks only the keys of its
// own columns: the work is split, not repeated.
#include <algorithm>

#include "sea_columns.h"
#include "sea_internal.h"
#include "sea_select.h"

namespace sea {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kWRow = 72;      // halfwords per staged W row (128 B + 16 B pad): conflict-free b128 reads
constexpr int kChunk = 32;     // tokens per feature chunk = keys per step of the tile kernel
constexpr int kPartCols = 32;  // columns whose bins one wavefront keeps

__device__ __forceinline__ floatx4 mfma16(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx16 mfma32(bf16x8 a, bf16x8 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
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

// ------------------------------------------------------------------------------------------
// Features.  The projection is taken transposed, C[feature][token] = W X^T (v_mfma_f32_16x16x32_bf16):
// lane l owns token l % 16 and, per 16-feature tile ft, the features 16 ft + 4 (l / 16) + i.  Two
// consecutive tiles give a lane 8 rounded values = one 16-byte piece; piece (kc, lg) of a token
// becomes contraction step 2 kc + lg / 2, lane half lg % 2 of the tile kernel's operands.  Which
// feature sits in which contraction slot is irrelevant as long as queries and keys agree.
//
// Operand row of a token within its 32-token chunk: queries keep their order (row = token).  Keys
// are permuted so that result register i of lane half h' is key 16 h' + i of the chunk: key
// 16 h' + 4 a + b sits in operand row 8 a + 4 h' + b.
//
// grid (N * blocks per head, 2): y = 0 queries, y = 1 keys.  A block parks W once and takes
// `iters` consecutive 64-token tiles.
// ------------------------------------------------------------------------------------------
template <int MC>  // m / 32
__global__ __launch_bounds__(256) void rw_features_kernel(Shape s, const uint16_t* __restrict__ Q,
                                                          const uint16_t* __restrict__ K,
                                                          const uint16_t* __restrict__ W, uint4* __restrict__ phiQ,
                                                          uint4* __restrict__ phiK, float c_dot, float c_norm,
                                                          int32_t iters) {
  constexpr int m = 32 * MC;
  constexpr int MS = 2 * MC;  // contraction steps of the tile kernel
  __shared__ __attribute__((aligned(16))) uint16_t Ws[m * kWRow];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const bool keys = blockIdx.y != 0;
  const uint32_t nch = (s.T + kChunk - 1) / kChunk;
  const uint32_t tiles = (nch + 1) / 2;
  const uint32_t bph = (tiles + iters - 1) / iters;
  const int64_t head = blockIdx.x / bph;
  const uint32_t first = (blockIdx.x % bph) * iters;
  for (int x = tid; x < m * 8; x += 256) {
    const int r = x >> 3, part = x & 7;
    *reinterpret_cast<uint4*>(&Ws[r * kWRow + part * 8]) = *reinterpret_cast<const uint4*>(W + r * kHeadDim + part * 8);
  }
  __syncthreads();
  const int32_t b = static_cast<int32_t>(head / s.H);
  const int32_t len = s.seq_len ? min(max(s.seq_len[b], 0), s.T) : s.T;
  const uint16_t* src = keys ? K : Q;
  uint4* dst = keys ? phiK : phiQ;
  for (uint32_t tile = first; tile < min(first + static_cast<uint32_t>(iters), tiles); ++tile) {
    const uint32_t chunk = 2 * tile + (wid >> 1);
    if (chunk >= nch) continue;  // wave-uniform
    const int32_t kappa = 16 * (wid & 1) + lr;
    const int32_t tok = static_cast<int32_t>(chunk) * kChunk + kappa;
    const uint16_t* X = src + (head * s.T + min(tok, s.T - 1)) * kHeadDim;
    const bf16x8 x0 = *reinterpret_cast<const bf16x8*>(X + 8 * lg);
    const bf16x8 x1 = *reinterpret_cast<const bf16x8*>(X + 32 + 8 * lg);
    float nx = sumsq8(x0) + sumsq8(x1);
    nx += __shfl_xor(nx, 16, kWave);
    nx += __shfl_xor(nx, 32, kWave);  // |x|^2 of token lr, in every lane group
    floatx4 dots[2 * MC];
#pragma unroll
    for (int ft = 0; ft < 2 * MC; ++ft) {
      const uint16_t* w = &Ws[(ft * 16 + lr) * kWRow + 8 * lg];
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = mfma16(*reinterpret_cast<const bf16x8*>(w), x0, acc);
      dots[ft] = mfma16(*reinterpret_cast<const bf16x8*>(w + 32), x1, acc);
    }
    // Exponent offset (log2 units).  Keys: the norm term alone.  Queries: also minus the row's
    // largest argument rounded up, a power-of-two row scale that commutes with the bf16 rounding
    // and cancels in the row normalisation.  Tokens past the sequence end: all-zero features.
    float off = -(c_norm * nx);
    if (!keys) {
      float dmax = -INFINITY;
#pragma unroll
      for (int ft = 0; ft < 2 * MC; ++ft)
#pragma unroll
        for (int i = 0; i < 4; ++i) dmax = fmaxf(dmax, dots[ft][i]);
      dmax = fmaxf(dmax, __shfl_xor(dmax, 16, kWave));
      dmax = fmaxf(dmax, __shfl_xor(dmax, 32, kWave));
      off -= ceilf(fmaf(c_dot, dmax, off));
    }
    if (tok >= len) off = -INFINITY;
    const int32_t row = keys ? 8 * ((kappa & 15) >> 2) + 4 * (kappa >> 4) + (kappa & 3) : kappa;
    uint4* out = dst + ((head * nch + chunk) * MS + (lg >> 1)) * 64 + 32 * (lg & 1) + row;
#pragma unroll
    for (int kc = 0; kc < MC; ++kc) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = __builtin_amdgcn_exp2f(fmaf(c_dot, dots[2 * kc][i], off));
        v[4 + i] = __builtin_amdgcn_exp2f(fmaf(c_dot, dots[2 * kc + 1][i], off));
      }
      uint4 u;
      u.x = pack_bf16(v[0], v[1]);
      u.y = pack_bf16(v[2], v[3]);
      u.z = pack_bf16(v[4], v[5]);
      u.w = pack_bf16(v[6], v[7]);
      out[2 * kc * 64] = u;
    }
  }
}

// ------------------------------------------------------------------------------------------
// Tiles.  Block = P <= 8 wavefronts working on one (head, 32 U rows); wave w takes the column
// parts w, w + P, ... (one pass of the loop below per part; a single pass whenever K <= 256).  Lane l of
// a wave owns the query rows r0 + 32 u + l % 32 and, in every 32-key chunk, the 16
// keys 16 (l / 32) + i of the chunk (see the key permutation above).
//
// Column of key j in row t: floor(j K / (t + 1)).  WIDE = false takes it in fp32 as
// trunc(j * (K / (t+1)) + 1 / (2 (t+1))) = trunc((j K + 1/2) / (t + 1)): j is exact, K / (t + 1)
// carries two roundings and the fused multiply-add a third, 3 * 2^-24 relative in all; the true
// quotient is at most K and lies at least 1 / (2 (t + 1)) away from every integer, so the
// truncation is exact while K (t + 1) < 2^24 / 6 (the launcher takes this form for K T <= 2^21).
// WIDE = true does the same in fp64 on the exact integer j K, where the half step exceeds the
// rounding error for any size the library accepts.  Keys j > t give a quotient >= K and keys outside the
// wave's columns one outside [c_lo, c_hi): both are clamped into a guard slot on either side of
// the row's bins, so no product needs a predicate.  Padding keys and rows past the end have
// all-zero features and add zeros.
// ------------------------------------------------------------------------------------------
// NCT > 0: the block also selects its rows' k^ columns (per-query grouping) and writes them as one bit per
// key of the row, which is all the attention needs; the scores then leave the chip only if A_hat is given.
// A wave takes 16 rows once the sums are known: a row's K <= 16 NCT scores go from the bins into four
// lanes, the search runs in registers, and each lane ORs the keys of its selected columns into the row's
// words.  B = 4, H = 12, T = 2048, K = 128: the pass over a score matrix in HBM that this replaces took
// 57 us (one row per wave), the whole forward 214 us, now 181.
// ------------------------------------------------------------------------------------------
template <int MS, bool WIDE, int NCT, int U, bool TOGETHER>  // MS = m / 16: contraction steps
__global__ __launch_bounds__(512, U == 1 ? 4 : 2) void rw_tiles_mfma_kernel(Shape s, const uint4* __restrict__ phiQ,
                                                            const uint4* __restrict__ phiK,
                                                            float* __restrict__ A_hat, int32_t parts,
                                                            int32_t part_cols, int32_t stride, int32_t cshift,
                                                            uint32_t* __restrict__ mbits, uint32_t* __restrict__ kb,
                                                            int32_t KWk, int32_t group_heads) {
  constexpr int kTileRows = 32 * U;  // query rows of the block
  extern __shared__ __align__(16) double lds[];  // [P][rows][stride] bins, [rows][P] row sums, [rows] inverses
  const int lane = threadIdx.x & 63, q = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int P = blockDim.x >> 6;
  double* bins = lds + static_cast<size_t>(wave) * kTileRows * stride;
  double* tot_s = lds + static_cast<size_t>(P) * kTileRows * stride;
  const uint32_t nch = (s.T + kChunk - 1) / kChunk;
  const uint32_t tiles = (s.T + kTileRows - 1) / kTileRows;
  // Heads in groups (heads_together), in a group the longest (last) row tiles first and heads fastest.  No groups: head-major, each
  // XCD on a run of blocks, in a head the longest tiles first.  Either way most of a head's blocks are on one XCD or two, whose
  // L2 serves all but the first read of its key features.
  uint32_t lb = blockIdx.x, first = 0, in_turn = 1;  // heads in turn
  if constexpr (TOGETHER) {
    const uint32_t per_group = static_cast<uint32_t>(group_heads) * tiles, grp = lb / per_group;
    first = grp * group_heads;
    in_turn = min(static_cast<uint32_t>(group_heads), static_cast<uint32_t>(s.N) - first);
    lb -= grp * per_group;
  } else {
    lb = xcd_contiguous(lb, gridDim.x);
  }
  const int64_t head = TOGETHER ? first + lb % in_turn : lb / tiles;
  const uint32_t tile = tiles - 1 - (TOGETHER ? lb / in_turn : lb % tiles);
  const int32_t r0 = static_cast<int32_t>(tile) * kTileRows;
  const int32_t b = static_cast<int32_t>(head / s.H);
  const int32_t len = s.seq_len ? min(max(s.seq_len[b], 0), s.T) : s.T;
  const int32_t r_last = min(min(r0 + kTileRows - 1, s.T - 1), len - 1);  // last active row of the tile
  const int32_t passes = (parts + P - 1) / P;
  // lane <-> (row, column) of a part when its bins leave: 2^cshift >= part_cols columns side by side
  const int32_t csub = lane & ((1 << cshift) - 1), rsub = lane >> cshift;

  bf16x8 qf[U][MS];
  float kinv[U], hinv[U];
  double winv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t tile32 = U * tile + u;
    const uint4* qp = phiQ + ((head * nch + min(tile32, nch - 1)) * MS) * 64 + lane;
#pragma unroll
    for (int st = 0; st < MS; ++st) {
      uint4 v = qp[st * 64];
      if (tile32 >= nch) v = uint4{0u, 0u, 0u, 0u};
      qf[u][st] = __builtin_bit_cast(bf16x8, v);
    }
    const int32_t t1 = r0 + 32 * u + q + 1;
    const float inv = 1.0f / static_cast<float>(t1);
    kinv[u] = static_cast<float>(s.K) * inv;
    hinv[u] = 0.5f * inv;
    winv[u] = 1.0 / static_cast<double>(t1);
  }
  const uint4* kp = phiK + (head * nch * MS) * 64 + lane;
  auto request = [&](bf16x8 (&kf)[MS], int32_t c) {
#pragma unroll
    for (int st = 0; st < MS; ++st)
      kf[st] = __builtin_bit_cast(bf16x8, kp[(static_cast<int64_t>(c) * MS + st) * 64]);
  };
  double rowtot[U] = {};  // row sums over the parts this wave has finished (rows 32 u + q)

  for (int32_t pass = 0; pass < passes; ++pass) {
    const int32_t part = pass * P + wave;
    const int32_t c_lo = min(part * part_cols, s.K), c_hi = min(s.K, c_lo + part_cols);
    const int32_t ncols = c_hi - c_lo;
    // index in `bins` of column 0 of the lane's rows: column c sits in slot c - (c_lo - 1), the
    // guards in slots 0 and ncols + 1
    int32_t base[U];
#pragma unroll
    for (int u = 0; u < U; ++u) base[u] = (32 * u + q) * stride - (c_lo - 1);
    // keys the wave's columns cover over the active rows: column starts grow with the row, so the
    // first key is row r0's start of c_lo and the last one precedes the last active row's start of c_hi
    int32_t cb = 0, ce = 0;
    if (r_last >= r0 && ncols > 0) {
      if (WIDE) {
        const int64_t j_begin = (static_cast<int64_t>(c_lo) * (r0 + 1) + s.K - 1) / s.K;
        const int64_t j_end = (static_cast<int64_t>(c_hi) * (r_last + 1) + s.K - 1) / s.K;
        cb = static_cast<int32_t>(j_begin / kChunk);
        ce = static_cast<int32_t>((j_end + kChunk - 1) / kChunk);
      } else {  // (everything below 2^22)
        cb = (c_lo * (r0 + 1) + s.K - 1) / s.K / kChunk;
        ce = ((c_hi * (r_last + 1) + s.K - 1) / s.K + kChunk - 1) / kChunk;
      }
    }
    bf16x8 kf[MS];
    if (cb < ce) request(kf, cb);
    for (int32_t x = lane; x < kTileRows * stride; x += 64) bins[x] = 0.0;
    const float lo_f = static_cast<float>(c_lo - 1), hi_f = static_cast<float>(c_hi);  // the guards
    // product i of chunk c in lane half h belongs to key 32 c + 16 h + i
    auto bin = [&](const floatx16 (&acc)[U], int32_t c, float jf, int i) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int32_t slot;
        if (WIDE) {
          const int64_t j = c * kChunk + 16 * h + i;
          const int32_t col = static_cast<int32_t>((static_cast<double>(j * s.K) + 0.5) * winv[u]);
          slot = min(max(col, c_lo - 1), c_hi);
        } else {
          // quotient clamped to the guards first: both are integers, so truncation commutes with the clamp
          slot = static_cast<int32_t>(__builtin_amdgcn_fmed3f(fmaf(jf + static_cast<float>(i), kinv[u], hinv[u]), lo_f, hi_f));
        }
        atomicAdd(&bins[base[u] + slot], static_cast<double>(acc[u][i]));
      }
    };
    __syncthreads();  // bins are clear (and, after the first pass, the previous part has left them)
    if (cb < ce) {
      // A SIMD holds two to four waves of this kernel: one's matrix products run under the other's binning.
      // Within the wave the next chunk's fragments are requested as soon as the products have
      // consumed the current ones, and arrive while the products are binned.
      for (int32_t c = cb; c < ce; ++c) {
        floatx16 acc[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[u][i] = 0.f;
#pragma unroll
        for (int st = 0; st < MS; ++st) {
#pragma unroll
          for (int u = 0; u < U; ++u) acc[u] = mfma32(kf[st], qf[u][st], acc[u]);
        }
        const float jf = static_cast<float>(c * kChunk + 16 * h);  // (exact, as is jf + i)
        __builtin_amdgcn_sched_barrier(0);
        if (c + 1 < ce) request(kf, c + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) bin(acc, c, jf, i);
      }
    }
    __syncthreads();  // every product of the part is in its bin
    // row sums of the part: lane (q, h) adds the columns c = h (mod 2) of its rows, the halves
    // meet by a lane swap
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double* row = bins + (32 * u + q) * stride + 1;
      double part_sum = 0.0;
      for (int32_t c = h; c < ncols; c += 2) part_sum += row[c];
      part_sum += __shfl_xor(part_sum, 32, kWave);
      rowtot[u] += part_sum;
    }
    if (passes > 1) {
      // more parts than the block has waves: the bins leave as they are, the rows are scaled at the end
      for (int32_t row = rsub; row < kTileRows && r0 + row < s.T; row += 64 >> cshift)
        if (csub < ncols)
          A_hat[(head * s.T + r0 + row) * s.K + c_lo + csub] = static_cast<float>(bins[row * stride + 1 + csub]);
    }
  }
  if (h == 0) {
#pragma unroll
    for (int u = 0; u < U; ++u) tot_s[(32 * u + q) * P + wave] = rowtot[u];
  }
  __syncthreads();
  double* inv_s = tot_s + kTileRows * P;  // [rows] 1 / row sum
  if (wave == 0 && lane < kTileRows) {
    double total = 0.0;
    for (int32_t w = 0; w < P; ++w) total += tot_s[lane * P + w];
    inv_s[lane] = (r0 + lane < len && total > 0.0) ? 1.0 / total : 0.0;
  }
  __syncthreads();
  if (passes == 1 && (NCT == 0 || A_hat)) {
    const int32_t c_lo = min(wave * part_cols, s.K), ncols = min(s.K, c_lo + part_cols) - c_lo;
    for (int32_t row = rsub; row < kTileRows && r0 + row < s.T; row += 64 >> cshift)
      if (csub < ncols)
        A_hat[(head * s.T + r0 + row) * s.K + c_lo + csub] =
            static_cast<float>(bins[row * stride + 1 + csub] * inv_s[row]);
  } else if (passes > 1) {
    // every lane scales the values it wrote itself (same wave, same part, same lane mapping)
    for (int32_t pass = 0; pass < passes; ++pass) {
      const int32_t c_lo = min((pass * P + wave) * part_cols, s.K), ncols = min(s.K, c_lo + part_cols) - c_lo;
      for (int32_t row = rsub; row < kTileRows && r0 + row < s.T; row += 64 >> cshift)
        if (csub < ncols) {
          float* out = A_hat + (head * s.T + r0 + row) * s.K + c_lo + csub;
          *out = static_cast<float>(static_cast<double>(*out) * inv_s[row]);
        }
    }
  }
  if constexpr (NCT > 0) {
    const int lr = lane & 15, lg = lane >> 4;
    const int32_t row = 16 * wave + lr, t = r0 + row;  // (the other waves have no rows)
    const bool active = wave < 2 * U && t < len;
    const int32_t Tw = t + 1, ncnd = active ? min(s.K, Tw) : 0;  // columns that hold a key
    const uint32_t nsel = static_cast<uint32_t>(min(s.k_hat, ncnd));
    const int32_t w0 = Tw / s.K, rm = Tw - w0 * s.K;
    const float invK = 1.0f / static_cast<float>(s.K);
    // first key of column c: ceil(c (t + 1) / K)
    auto start = [&](int32_t c) { return c * w0 + div_small(c * rm + s.K - 1, invK); };
    uint32_t key[NCT][4];
    bool sums = false;  // the row's scores sum to one
    if (wave < 2 * U) {
      const double inv = inv_s[row];
      sums = inv > 0x1p-100 && inv < 0x1p100;
      const uint32_t by_part = 65536u / static_cast<uint32_t>(part_cols) + 1u;  // c / part_cols, exact for c < 256
      const double* const row_bins = lds + row * stride + 1;
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        const int32_t c0 = 16 * ct + 4 * lg;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          int32_t at = ct / 2 * (kTileRows * stride) + 16 * (ct & 1) + 4 * lg + i;  // parts of 32 columns
          if (part_cols != 32 || 16 * ct + 16 > s.K) {
            const int32_t c = min(c0 + i, s.K - 1);
            const int32_t part = static_cast<int32_t>((static_cast<uint32_t>(c) * by_part) >> 16);
            at = part * kTileRows * stride + c - part * part_cols;
          }
          const double sum = row_bins[at];
          bool cand = active && c0 + i < s.K;
          if (w0 == 0) cand = cand && start(c0 + i + 1) > start(c0 + i);
          key[ct][i] = cand ? __float_as_uint(static_cast<float>(sum * inv)) | 0x80000000u : 0x40000000u;
        }
      }
    }
    __syncthreads();  // the bins are in registers: their place takes the rows' key bits
    if (wave >= 2 * U) return;
    uint32_t sel[NCT / 2];
    select_columns<NCT>(key, nsel, ncnd, NCT, s.k_hat, search_top(nsel, sums), lg, sel);
    if (mbits) {
      const int32_t kw = (s.K + 31) >> 5;
#pragma unroll
      for (int j = 0; j < NCT / 2; ++j) {
        const uint32_t word = rows_or_u(sel[j] << (4 * lg));
        if (lg == 0 && j < kw && t < s.T) mbits[(head * s.T + t) * kw + j] = word;
      }
    }
    // words of the 128-row tile the attention may look at; one word of padding per row keeps the rows' words in
    // different banks
    const int32_t nw = min(KWk, ((r0 | 127) >> 5) + 1), wstride = nw | 1;
    uint32_t* const words = reinterpret_cast<uint32_t*>(lds + static_cast<size_t>(wave) * (P / (2 * U)) * kTileRows * stride);
    for (int32_t x = lane; x < 16 * wstride; x += 64) words[x] = 0u;
    __builtin_amdgcn_wave_barrier();
    uint32_t* const wrow = words + lr * wstride;
    const bool whole = w0 + (rm > 0 ? 1 : 0) <= s.rep_cap;  // no column is wider than the cap: all its keys are emitted
    if (__ballot(active && !whole) == 0ull) {
      // A key's bit is the parity of the selection changes at or before it: one bit is flipped where a selected
      // column follows an unselected one or the reverse (columns without keys flip nothing: their flips meet in
      // one place), and the words are made of the flips on their way out.
      uint32_t carry = 0u;  // is column 16 ct - 1 selected (lane group 3 of the tile before)
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        const uint32_t nib = (sel[ct / 2] >> (16 * (ct & 1))) & 15u, top = nib >> 3;
        const uint32_t below = __shfl_up(top, 16, kWave);  // bit 3 of the lane group below
        const uint32_t prev = (nib << 1) | (lg == 0 ? carry : below);
        carry = __shfl(top, 48 + lr, kWave);
        const uint32_t flips = (nib ^ prev) & 15u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int32_t c = 16 * ct + 4 * lg + i, at = start(c);
          if (((flips >> i) & 1u) && c < s.K) atomicXor(&wrow[at >> 5], 1u << (at & 31));
        }
      }
      __builtin_amdgcn_wave_barrier();
      for (int32_t rr = 0; rr < 16 && r0 + 16 * wave + rr < s.T; ++rr) {
        const int32_t tr = r0 + 16 * wave + rr;
        uint32_t* const dst = kb + (head * s.T + tr) * KWk;
        uint32_t in = 0u;  // parity of all flips in earlier words
        for (int32_t x0 = 0; x0 < nw; x0 += 64) {
          const int32_t x = x0 + lane;
          uint32_t v = x < nw ? words[rr * wstride + x] : 0u;
#pragma unroll
          for (int d = 1; d < 32; d <<= 1) v ^= v << d;
          const uint64_t odd = __ballot((v >> 31) != 0u);
          const uint32_t before = in ^ (static_cast<uint32_t>(__popcll(odd & ((1ull << lane) - 1ull))) & 1u);
          v ^= 0u - before;
          // nothing past the row's own keys (the last column may be selected)
          const int32_t past = tr + 1 - 32 * x;
          v &= past >= 32 ? 0xffffffffu : (past <= 0 ? 0u : (1u << past) - 1u);
          if (x < nw) dst[x] = v;
          in ^= static_cast<uint32_t>(__popcll(odd)) & 1u;
        }
      }
    } else {
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if ((sel[ct / 2] >> (16 * (ct & 1) + i)) & 1u) {
            const int32_t c = 16 * ct + 4 * lg + i, s0 = start(c), w = start(c + 1) - s0, r = min(w, s.rep_cap);
            for (int32_t e = 0; e < r; ++e) {
              const int32_t j = s0 + (e * w) / r;
              atomicOr(&wrow[j >> 5], 1u << (j & 31));
            }
          }
      __builtin_amdgcn_wave_barrier();
      for (int32_t rr = 0; rr < 16 && r0 + 16 * wave + rr < s.T; ++rr) {
        uint32_t* const dst = kb + (head * s.T + r0 + 16 * wave + rr) * KWk;
        for (int32_t x = lane; x < nw; x += 64) dst[x] = words[rr * wstride + x];
      }
    }
  }
}

// 32-row tiles of a block: one (four waves per SIMD; the selection and the start and end of a block are chains of
// latencies: 189 -> 181 us for the forward of the kernel's comment), two where m = 256 leaves no registers for that
constexpr int row_tiles(int m) { return m == 256 ? 2 : 1; }

struct Plan {
  int32_t parts, part_cols, stride, waves, cshift;
  size_t lds;
};
Plan plan(const Shape& s, int32_t rows) {
  Plan p{};
  p.parts = (s.K + kPartCols - 1) / kPartCols;
  p.part_cols = (s.K + p.parts - 1) / p.parts;
  p.stride = (p.part_cols + 2) | 1;  // two guards; odd, so the 32 rows of a step fall into different banks
  p.waves = std::min(p.parts, 8);
  while ((1 << p.cshift) < p.part_cols) ++p.cshift;
  p.lds = (static_cast<size_t>(p.waves) * rows * p.stride + static_cast<size_t>(rows) * (p.waves + 1)) * sizeof(double);
  return p;
}
size_t side_bytes(const Shape& s) {
  const size_t t32 = (static_cast<size_t>(s.T) + kChunk - 1) / kChunk * kChunk;
  return (static_cast<size_t>(s.N) * t32 * s.m * sizeof(uint16_t) + 255) & ~size_t(255);
}

// Heads that are dealt out together, 0: head after head.  Together, what is left at a launch's end are short tiles, and all XCDs
// have the same work; head after head, the last head's longest tiles begin when the others are done, and with a few heads that
// are no multiple of eight an XCD has the longer half of one.  But an XCD's L2 (4 MB) then holds the key features of several
// heads.  Layer, us, head after head / together, K = m = 128, where nothing else is said:
//   all heads in one group: 12 heads of 2048 rows 73.8 / 70.7, of 4096 171 / 144, 24 of 1024 56.2 / 51.9, 32 of 1024 63.8 / 56.5;
//   not where a CU gets one block or none (<= 256), nor, of heads that share their XCDs with others (N % 8 == 4), those with few
//   tiles or some two blocks per CU: 12 heads of 1400 rows 54.1 / 55.1, 36 of 640 44.6 / 45.8, of 256 32.1 / 32.9;
//   not in launches that are hardly longer than one round of resident blocks and that hold several heads per XCD: m = 256, 24 heads of
//   1536 91.2 / 96, 36 of 1024 84.4 / 87.8, m = 64, 36 of 1024 61.6 / 64.2 (of 2048 and more rows the end counts: K = 64, 24 of 3072 158 / 150);
//   not with an odd number of heads, each on all XCDs, beyond sixteen and with more than 8 MB of features: 17 of 3000 139 / 151, of 2048 88 / 90
//   (few of them still gain by the even share: 9 of 4096, K = 100, 134 / 130; and so do blocks of two waves, K = 64, 17 of 2048 85 / 78);
//   more than 26 MB of features: groups whose features take 2 MB of an L2 (K = 128, 36 heads of 3072 238 / 236 and, all together, 239; B = 4,
//   T = 4096 467 / 450).  Up to there such groups only if they fill the chip one and a half times and the last one is no small rest:
//   48 of 2048 (32 and 16) 166.2 / 161.8, all together 166.3; but m = 256, 36 of 1024 (32 and 4) 94.6, K = 64, 36 of 2048 132, 116 together.
// Left as they are: 16 heads of 2800 107 / 109, m = 64, 12 of 1536 53.5 / 54.5.
int32_t heads_together(const Shape& s, int U, int32_t waves, uint32_t tiles) {
  const int64_t blocks = static_cast<int64_t>(s.N) * tiles, resident = 256 * std::max(1, (U == 1 ? 16 : 8) / waves);
  const int64_t head_bytes = static_cast<int64_t>(s.T) * s.m * 2;
  if (blocks <= 256) return 0;
  if (U == 1 && s.N % 8 == 4 && (s.T < 700 || (s.T < 1500 && blocks < 576))) return 0;
  if (s.N % 2 != 0 && s.N > 16 && s.K > 64 && s.N * head_bytes > int64_t(8) << 20) return 0;
  if (s.N >= 24 && s.T < 2048 && blocks > resident && 4 * blocks < 5 * resident) return 0;
  const int64_t fit = 8 * std::max<int64_t>(1, (int64_t(2) << 20) / head_bytes);
  if (s.N * head_bytes <= int64_t(26) << 20 && (2 * (s.N % fit) < fit || 2 * fit * tiles < 3 * resident)) return s.N;
  return static_cast<int32_t>(std::min<int64_t>(s.N, fit));
}

template <int MS, bool WIDE, int NCT, int U, bool TOGETHER>
hipError_t start_tiles(const Shape& s, const Plan& p, int32_t group_heads, const uint4* phiQ, const uint4* phiK, float* A_hat,
                       uint32_t* mbits, uint32_t* kb, hipStream_t st) {
  if (p.lds > (64u << 10)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&rw_tiles_mfma_kernel<MS, WIDE, NCT, U, TOGETHER>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(p.lds));
    if (e != hipSuccess) return e;
  }
  const uint32_t blocks = static_cast<uint32_t>(s.N) * ((s.T + 32 * U - 1) / (32 * U));
  hipLaunchKernelGGL((rw_tiles_mfma_kernel<MS, WIDE, NCT, U, TOGETHER>), dim3(blocks), dim3(64 * p.waves), p.lds, st, s, phiQ, phiK, A_hat,
                     p.parts, p.part_cols, p.stride, p.cshift, mbits, kb, (s.T + 31) / 32, group_heads);
  return hipGetLastError();
}

// (an instance for each order: the short launches, head after head, feel 0.3 us of the other one's divisions)
template <int MS, bool WIDE, int NCT, int U>
hipError_t launch_tiles(const Shape& s, const uint4* phiQ, const uint4* phiK, float* A_hat, uint32_t* mbits, uint32_t* kb,
                        hipStream_t st) {
  const Plan p = plan(s, 32 * U);
  const int32_t group_heads = heads_together(s, U, p.waves, (s.T + 32 * U - 1) / (32 * U));
  if (group_heads > 0) return start_tiles<MS, WIDE, NCT, U, true>(s, p, group_heads, phiQ, phiK, A_hat, mbits, kb, st);
  return start_tiles<MS, WIDE, NCT, U, false>(s, p, 0, phiQ, phiK, A_hat, mbits, kb, st);
}

template <int MC>
hipError_t launch(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* W, float* A_hat,
                  uint32_t* mbits, uint32_t* kb, void* ws, hipStream_t st) {
  uint4* phiQ = static_cast<uint4*>(ws);
  uint4* phiK = reinterpret_cast<uint4*>(static_cast<char*>(ws) + side_bytes(s));
  const double l2e = 1.4426950408889634;
  const float c_dot = static_cast<float>(l2e * std::sqrt(static_cast<double>(s.scale)));
  const float c_norm = static_cast<float>(l2e * 0.5 * static_cast<double>(s.scale));
  {
    StageScope scope(SEA_STAGE_FEATURES, st);
    const uint32_t nch = (s.T + kChunk - 1) / kChunk, tiles = (nch + 1) / 2;
    const int32_t iters = static_cast<int32_t>(std::min<int64_t>(8, std::max<int64_t>(1, static_cast<int64_t>(s.N) * tiles / 1024)));
    const uint32_t bph = (tiles + iters - 1) / iters;
    hipLaunchKernelGGL(rw_features_kernel<MC>, dim3(static_cast<uint32_t>(s.N) * bph, 2), dim3(256), 0, st, s, Q, K,
                       W, phiQ, phiK, c_dot, c_norm, iters);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  StageScope scope(SEA_STAGE_CONTRACT, st);
  const bool wide = static_cast<int64_t>(s.K) * s.T > (int64_t{1} << 21);
  constexpr int U = row_tiles(32 * MC);
  if (kb)  // K T <= 2^21 there
    return launch_tiles<2 * MC, false, 8, U>(s, phiQ, phiK, A_hat, mbits, kb, st);
  return wide ? launch_tiles<2 * MC, true, 0, 2>(s, phiQ, phiK, A_hat, nullptr, nullptr, st)
              : launch_tiles<2 * MC, false, 0, U>(s, phiQ, phiK, A_hat, nullptr, nullptr, st);
}

}  // namespace

bool rowwidth_mfma_supported(const Shape& s, sea_dtype dt) {
  return dt == SEA_BF16 && s.causal && (s.m == 64 || s.m == 128 || s.m == 256);
}

size_t rowwidth_mfma_workspace(const Shape& s) { return 2 * side_bytes(s); }

// The selection as key bits straight from the estimate: a wave for every 16 rows of a block, and room for those
// rows' key bits in the place of the bins.  Up to 128 columns: there a row's search is shorter than the way of its
// scores through memory.  Above, it is not: half of a block's waves stand by meanwhile, and a kernel of its own
// searches with all of them (whole forward, us, in the estimate / on its own: 12 heads, T = 1500, m = 128, K = 256, B = 2
// 114 / 92; 32 heads, m = K = 256, T = 2048, B = 1 229 / 209, B = 8 1718 / 1585, T = 260, B = 8 204 / 167; K = 128,
// T = 2048, 48 heads, m = 128 173 / 197, 24 heads, m = 256 134 / 144).  And only from one 64-row block per CU on:
// smaller launches leave the search the whole chip (12 heads of 500 rows, K = 128, 35 / 30; 48 heads 47 / 50).
bool rowwidth_select_supported(const Shape& s, sea_dtype dt) {
  if (!rowwidth_mfma_supported(s, dt) || s.grouping != 0 || s.K > 128 || s.T > 8192) return false;
  if (static_cast<int64_t>(s.N) * ((s.T + 63) / 64) < 256) return false;
  const int32_t U = row_tiles(s.m);
  const Plan p = plan(s, 32 * U);
  const size_t room = static_cast<size_t>(p.waves / (2 * U)) * 32 * U * p.stride * sizeof(double);
  return room >= static_cast<size_t>(16) * (((s.T + 31) / 32) | 1) * sizeof(uint32_t);
}

hipError_t launch_rowwidth_mfma(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* W,
                                float* A_hat, void* ws, hipStream_t st, uint32_t* mbits, uint32_t* kb) {
  if (kb && !rowwidth_select_supported(s, SEA_BF16)) return hipErrorNotSupported;
  switch (s.m) {
    case 64: return launch<2>(s, Q, K, W, A_hat, mbits, kb, ws, st);
    case 128: return launch<4>(s, Q, K, W, A_hat, mbits, kb, ws, st);
    default: return launch<8>(s, Q, K, W, A_hat, mbits, kb, ws, st);
  }
}

}  // namespace sea
