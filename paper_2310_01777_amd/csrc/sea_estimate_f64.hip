// Random-feature estimate of the compressed attention matrix, fp32 tensors with fp64
// arithmetic (Sec. 3 "Performer (FAVOR+)", Sec. 3.1 "Attention Matrix Estimation").
//
//   phi(x)[i] = exp(w_i.x - |x|^2/2), x = sqrt(scale) q;  state = phi(K)^T V_I (K x m bucket
//   sums, V_I the nearest-neighbour stretched identity);  A_hat = rownorm(phi(Q) state), a
//   causal row using the inclusive prefix of its own bucket instead of the full bucket sum.
//
// This is the reference-precision mode: every dot product and the exponential are fp64 so
// that the per-row top-k^ taken on A_hat agrees with an fp64 evaluation except where two
// scores differ by less than ~1e-7 relative.  The projections and the contraction run on the
// matrix cores (v_mfma_f64_16x16x4_f64: lane l supplies A[row l % 16][k l / 16] and
// B[k l / 16][col l % 16], and receives D[row 4 i + l / 16][col l % 16] in register i); the
// contraction index is free to permute as long as both operands agree, which lets every lane read
// its sixteen operand values as contiguous floats.
//
// Workspace layout (doubles): phiQ [N][T][m], phiK/prefix [N][T][m], stateT [N][m][K].
#include "sea_internal.h"
#include "sea_select.h"

namespace sea {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ doublex4 mfma_f64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// exp(x) in fp64: x = k ln 2 + r, |r| <= 0.35, Taylor series to r^13 (error < 1e-17 relative)
__device__ __forceinline__ double exp_f64(double x) {
  const double k = rint(x * 1.4426950408889634074);
  double r = fma(-k, 6.93147180369123816490e-01, x);
  r = fma(-k, 1.90821492927058770002e-10, r);
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, static_cast<int>(k));
}

// four consecutive elements of an fp32 tensor
__device__ __forceinline__ float4 load4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// phi for 16 rows per WPT waves, each of which takes its share of the features.  WPT = 4 in small launches (12
// heads of 1024 rows are then 6144 waves and not 1536: with less than two waves per SIMD the products of 16
// dependent steps and the exponentials ran one after the other; 23 -> 20 us at m = 128) and where a wave would
// hold more than 8 feature tiles (m = 256, 12 heads of 2048 rows 61 -> 52 us).  From 3072 row tiles on, queries and
// keys (m = 64: 2048), one wave per tile is the faster form, which loads its rows once (12 heads of 2048 rows
// 33 -> 31 us at m = 128, 23 -> 20 us at m = 64, 16 heads of 1024 rows 20 -> 17 us there) and leaves the features where the kernels that follow read them (per-row widths,
// m = 64, 24 heads of 2048 rows: tiles 278 -> 254 us).
// Queries are shifted by their row maximum (WPT = 4: it meets in LDS; any shift cancels in the normaliser);
// keys are not shifted and are zero beyond seq_len.
// D[row = token 4 i + lg][col = feature lr]; contraction slot (step s, lane group lg) stands for
// dimension 16 lg + s.
// NFT > 0: the exponent arguments of the wave's (at most NFT) feature tiles stay in registers between the
// projection and the exponential, and the unrolled tile loop lets the loads of W run ahead;
// NFT = 0: any m, the arguments take a round trip through the output buffer.
// COLS (whole columns of 1, 2, 4, 8 or 16 keys to a tile, 2^wl each): the column sums leave as well, and phi(K) leaves as
// its running sums inside the columns, which is what the rows kernel takes (bidirectional layers: not at all); a kernel of their
// own took 7 us of a layer of 12 heads of 1024 rows, most of it its launch.
template <int NFT, int WPT, bool COLS = false>
__global__ __launch_bounds__(256) void features_f64_kernel(Shape s, const float* __restrict__ Q,
                                                           const float* __restrict__ K, const float* __restrict__ W,
                                                           double* __restrict__ phiQ, double* __restrict__ phiK,
                                                           double* __restrict__ stateT, int32_t wl) {
  static_assert(!COLS || NFT > 0, "the features stay in registers");
  __shared__ double rowmax[4][16];
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int lr = lane & 15, lg = lane >> 4;
  const uint32_t tiles = (s.T + 15) / 16;
  const int64_t nw = static_cast<int64_t>(s.N) * tiles;  // row tiles of the queries, then of the keys
  const int64_t tile = WPT == 4 ? blockIdx.x : static_cast<int64_t>(blockIdx.x) * 4 + wid;
  if (WPT == 1 && tile >= 2 * nw) return;
  const int part = WPT == 4 ? wid : 0;  // this wave's share of the features
  const int which = tile >= nw;
  const int64_t wv = which ? tile - nw : tile;
  const int64_t head = wv / tiles;
  const int32_t r0 = static_cast<int32_t>(wv % tiles) * 16;
  const int32_t b = static_cast<int32_t>(head / s.H);
  const int32_t len = s.seq_len ? min(max(s.seq_len[b], 0), s.T) : s.T;
  const float* X = (which ? K : Q) + (head * s.T + min(r0 + lr, s.T - 1)) * kHeadDim + 16 * lg;
  const double rs = sqrt(static_cast<double>(s.scale));
  double xa[16];
  double nx = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = load4(X + 4 * q);
    xa[4 * q] = rs * v.x; xa[4 * q + 1] = rs * v.y; xa[4 * q + 2] = rs * v.z; xa[4 * q + 3] = rs * v.w;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) nx = fma(xa[e], xa[e], nx);
  nx += __shfl_xor(nx, 16, kWave);
  nx += __shfl_xor(nx, 32, kWave);  // |x|^2 of token r0 + lr, in every lane group
  if (r0 >= len) {  // nothing but padding (the block's tile, or this wave's)
    double* const to = (which ? phiK : phiQ) + (head * s.T + r0) * s.m;
    const int32_t n = min(16, s.T - r0) * s.m;
    for (int32_t x = WPT == 4 ? threadIdx.x : lane; x < n; x += WPT == 4 ? 256 : 64) to[x] = 0.0;
    if (COLS && which) {
      const int32_t cols = 16 >> wl;
      for (int32_t x = WPT == 4 ? threadIdx.x : lane; x < s.m * cols; x += WPT == 4 ? 256 : 64)
        stateT[(head * s.m + x / cols) * s.K + (r0 >> wl) + x % cols] = 0.0;
    }
    return;
  }
  // this lane's four result rows are tokens r0 + 4 i + lg
  double half_n[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) half_n[i] = 0.5 * __shfl(nx, 4 * i + lg, kWave);
  double* out = (which ? phiK : phiQ) + (head * s.T) * s.m;
  double amax[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  const int ntiles = s.m / 16;  // share p: tiles p, p + WPT, ...
  auto project = [&](int ft) {
    const float* w = W + static_cast<int64_t>(ft * 16 + lr) * kHeadDim + 16 * lg;
    float4 wv4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) wv4[q] = load4(w + 4 * q);
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc = mfma_f64(xa[4 * q], static_cast<double>(wv4[q].x), acc);
      acc = mfma_f64(xa[4 * q + 1], static_cast<double>(wv4[q].y), acc);
      acc = mfma_f64(xa[4 * q + 2], static_cast<double>(wv4[q].z), acc);
      acc = mfma_f64(xa[4 * q + 3], static_cast<double>(wv4[q].w), acc);
    }
    return acc;
  };
  double shift[4];
  auto row_shift = [&]() {
    if (which) {  // block-uniform
#pragma unroll
      for (int i = 0; i < 4; ++i) shift[i] = 0.0;
      return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double mx = amax[i];
#pragma unroll
      for (int mask = 1; mask < 16; mask <<= 1) mx = fmax(mx, __shfl_xor(mx, mask, kWave));
      shift[i] = mx;
      if (WPT == 4 && lr == 0) rowmax[wid][4 * i + lg] = mx;
    }
    if (WPT == 1) return;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * i + lg;
      shift[i] = fmax(fmax(rowmax[0][r], rowmax[1][r]), fmax(rowmax[2][r], rowmax[3][r]));
    }
  };
  if constexpr (NFT > 0) {
    double arg[NFT][4];
#pragma unroll
    for (int f = 0; f < NFT; ++f) {
      if (WPT * f + part < ntiles) {
        const doublex4 acc = project(WPT * f + part);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          arg[f][i] = acc[i] - half_n[i];
          amax[i] = fmax(amax[i], arg[f][i]);
        }
      }
    }
    row_shift();
#pragma unroll
    for (int f = 0; f < NFT; ++f) {
      if (WPT * f + part < ntiles) {
        const int32_t feature = (WPT * f + part) * 16 + lr;
        if (COLS && which) {
          double v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = r0 + 4 * i + lg < len ? exp_f64(arg[f][i] - shift[i]) : 0.0;
          // inclusive sums over the tokens 4 i + lg of a column: over lane groups, then over registers
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (wl >= 1) {
              const double below = __shfl_xor(v[i], 16, kWave);
              v[i] += (lg & 1) ? below : 0.0;
            }
            if (wl >= 2) {
              const double below = __shfl(v[i], lr + 16, kWave);
              v[i] += (lg & 2) ? below : 0.0;
            }
          }
          if (wl >= 3) {
            v[1] += __shfl(v[0], lr + 48, kWave);
            v[3] += __shfl(v[2], lr + 48, kWave);
          }
          if (wl == 4) {
            const double below = __shfl(v[1], lr + 48, kWave);
            v[2] += below;
            v[3] += below;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int32_t t = r0 + 4 * i + lg;
            if (((t + 1) & ((1 << wl) - 1)) == 0) stateT[(head * s.m + feature) * s.K + (t >> wl)] = v[i];
            if (s.causal) out[static_cast<int64_t>(t) * s.m + feature] = v[i];
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int32_t t = r0 + 4 * i + lg;
            if (t < s.T) out[static_cast<int64_t>(t) * s.m + feature] = t < len ? exp_f64(arg[f][i] - shift[i]) : 0.0;
          }
        }
      }
    }
  } else {
    for (int ft = part; ft < ntiles; ft += WPT) {
      const doublex4 acc = project(ft);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int32_t t = r0 + 4 * i + lg;
        const double a = acc[i] - half_n[i];
        amax[i] = fmax(amax[i], a);
        if (t < s.T) out[static_cast<int64_t>(t) * s.m + ft * 16 + lr] = a;  // exponent argument for now
      }
    }
    row_shift();
    // second pass over the lane's own values
    for (int ft = part; ft < ntiles; ft += WPT) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int32_t t = r0 + 4 * i + lg;
        if (t >= s.T) continue;
        double* o = out + static_cast<int64_t>(t) * s.m + ft * 16 + lr;
        *o = t < len ? exp_f64(*o - shift[i]) : 0.0;
      }
    }
  }
}

// One thread per (head, column c, feature i): walk the keys of the column, turning phiK into
// its inclusive within-column prefix in place, and write the column sum to stateT[i][c].
__global__ __launch_bounds__(256) void state_f64_kernel(Shape s, double* __restrict__ phiK,
                                                        double* __restrict__ stateT) {
  const int64_t gid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t total = static_cast<int64_t>(s.N) * s.K * s.m;
  if (gid >= total) return;
  const int32_t i = static_cast<int32_t>(gid % s.m);
  const int32_t c = static_cast<int32_t>((gid / s.m) % s.K);
  const int64_t head = gid / (static_cast<int64_t>(s.m) * s.K);
  const int32_t j0 = block_start(c, s.T, s.K), j1 = block_start(c + 1, s.T, s.K);
  double* col = phiK + (head * s.T) * s.m + i;
  double acc = 0.0;
  for (int32_t j = j0; j < j1; ++j) {
    acc += col[static_cast<int64_t>(j) * s.m];
    col[static_cast<int64_t>(j) * s.m] = acc;
  }
  stateT[(head * s.m + i) * s.K + c] = acc;
}

// A_hat rows.  Block = 8 waves on 32 rows: wave (rt, cq) takes row tile rt and the 16-column tiles
// cq, cq + 4, ... (interleaved, so that the columns a causal tile needs are shared out evenly); the row
// sums meet in LDS.  One wave per 16 rows and all columns gave 12 heads of 1024 rows 768 waves for 1024
// SIMDs (36 us); split, the same products are 3072 waves, and the two row tiles read the same state while
// it is in the cache (25 us).
// Tile (16 tokens x 16 columns) = phiQ x state over the m features, sixteen per four steps (slot (step e, lane
// group lg) = feature 4 lg + e, so that a lane's four feature values are 32 contiguous bytes); a causal row's own column is the diagonal of phiQ x prefix^T, each wave of a row
// tile taking a quarter of the features.  A wave's column tiles are taken in groups of NCT that stay in
// registers; with one group (K <= 64 NCT) a single pass normalises and stores, with more the groups are
// computed twice: once for the row sums, once for the normalised output.
__device__ __forceinline__ double2 load2(const double* base, uint32_t off) {
  return *reinterpret_cast<const double2*>(base + off);
}

// SELECT (one group): the rows' k^ columns (per-query grouping) leave as well, as one bit per column, and the scores only if A_hat
// is given.  They pass through LDS, and each wave chooses for four rows as the kernel of its own would: 5.8 us here for 7.1 there
// and a gap, 12 heads of 1024 rows, K = 128, layer 78.6 -> 77.0 us.  (Four rows side by side, to hide the scalar unit's latency, take
// as many steps as the slowest: 6.6 us.)
template <int NCT, bool SELECT = false>
__global__ __launch_bounds__(512, NCT <= 2 ? 4 : 2) void contract_f64_kernel(Shape s, const double* __restrict__ phiQ,
                                                           const double* __restrict__ pref,
                                                           const double* __restrict__ stateT,
                                                           float* __restrict__ A_hat, uint32_t* __restrict__ mbits) {
  __shared__ double red_s[2][4][16], diag_s[2][4][16];
  constexpr int kPlace = 64 * NCT + 4;  // floats per row of scores
  __shared__ float place[SELECT ? 32 * kPlace : 1];
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int rt = wid >> 2, cq = wid & 3;
  const int lr = lane & 15, lg = lane >> 4;
  const uint32_t tiles = (s.T + 31) / 32;
  // Causal rows need columns up to their own, so the blocks of a head's last rows take longest.  A launch of one to two
  // blocks per CU is resident at once and dealt to the 256 CUs in turn: those that get one block take the longest
  // ones, and the others one of the next with one of the shortest (head by head, both blocks of a CU had the same
  // rows of two heads: 12 heads of 1024 rows 24.9 -> 20.0 us).  Other launches: longest first.
  uint32_t rank = blockIdx.x;
  if (gridDim.x > 256u && gridDim.x <= 512u) {
    const uint32_t pairs = gridDim.x - 256u;
    rank = rank >= 256u ? gridDim.x - 1u - (rank - 256u) : (rank < pairs ? 256u - pairs + rank : rank - pairs);
  }
  const int64_t head = rank % static_cast<uint32_t>(s.N);
  const int32_t r0 = static_cast<int32_t>(tiles - 1u - rank / static_cast<uint32_t>(s.N)) * 32 + 16 * rt;  // (may lie past T: the wave then only joins the barriers)
  const int32_t b = static_cast<int32_t>(head / s.H);
  const int32_t len = s.seq_len ? min(max(s.seq_len[b], 0), s.T) : s.T;
  if (r0 - 16 * rt >= len) {  // nothing but padding (both row tiles)
    const int64_t row = head * s.T + r0 - 16 * rt, rows = min(32, s.T - (r0 - 16 * rt));
    if (!SELECT || A_hat)
      for (int64_t x = threadIdx.x; x < rows * s.K; x += 512) A_hat[row * s.K + x] = 0.f;
    const int32_t kw = (s.K + 31) / 32;
    if (SELECT)
      for (int64_t x = threadIdx.x; x < rows * kw; x += 512) mbits[row * kw + x] = 0u;
    return;
  }
  // uniform bases and 32-bit lane offsets (a head's m K state and the 16 rows' m values index with 32 bits)
  const int32_t rbase = min(r0, s.T - 1);
  const double* qb_ = phiQ + (head * s.T + rbase) * s.m;   // A operand: token lr
  const double* pb_ = pref + (head * s.T + rbase) * s.m;   // B operand: token lr as column
  const uint32_t roff = static_cast<uint32_t>(min(r0 + lr, s.T - 1) - rbase) * s.m + 4 * lg;
  const double* st = stateT + head * static_cast<int64_t>(s.m) * s.K;
  // columns this row tile needs: causal rows stop at the last row's own column
  const int32_t t_hi = min(r0 + 15, s.T - 1);
  const int32_t ncols = s.causal ? min(s.K, bucket_of(t_hi, s.T, s.K) + 1) : s.K;
  const int32_t ngroups = (ncols + 64 * NCT - 1) / (64 * NCT);

  // this lane's rows: tokens r0 + 4 i + lg
  double diag[4] = {0.0, 0.0, 0.0, 0.0}, rsum[4] = {0.0, 0.0, 0.0, 0.0}, inv[4];
  int32_t tcol[4];
  bool act[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int32_t t = r0 + 4 * i + lg;
    act[i] = t < len;
    tcol[i] = act[i] ? bucket_of(t, s.T, s.K) : -1;
  }
  if (s.causal) {
    // steps cq, cq + 4, ... in blocks of eight features (m is a multiple of 32)
    doublex4 dg = {0.0, 0.0, 0.0, 0.0};
    for (int32_t f0 = 16 * cq; f0 < s.m; f0 += 64) {
      const double2 q0 = load2(qb_ + f0, roff), q1 = load2(qb_ + f0 + 2, roff);
      const double2 p0 = load2(pb_ + f0, roff), p1 = load2(pb_ + f0 + 2, roff);
      dg = mfma_f64(q0.x, p0.x, dg);
      dg = mfma_f64(q0.y, p0.y, dg);
      dg = mfma_f64(q1.x, p1.x, dg);
      dg = mfma_f64(q1.y, p1.y, dg);
    }
    // the diagonal entry of token u sits in lane (lr = u, lg = u % 4), register u / 4
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (lr == 4 * i + lg) diag_s[rt][cq][lr] = dg[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = 4 * i + lg;
      diag[i] = (diag_s[rt][0][u] + diag_s[rt][1][u]) + (diag_s[rt][2][u] + diag_s[rt][3][u]);
    }
  }
  doublex4 acc[NCT];
  // Operands are requested a block of contraction steps ahead of the products that use them (two register
  // sets in turn).
  auto group = [&](int32_t g) {
    constexpr int FS = 4;  // contraction steps per block; m is a multiple of 32 = 8 steps
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) acc[ct] = doublex4{0.0, 0.0, 0.0, 0.0};
    int32_t c0[NCT];
    uint32_t soff[NCT];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      c0[ct] = 64 * (NCT * g + ct) + 16 * cq;
      soff[ct] = static_cast<uint32_t>(4 * lg * s.K + min(c0[ct] + lr, s.K - 1));
    }
    double aa[FS], ab[FS], ba[NCT][FS], bb[NCT][FS];
    auto ld = [&](int32_t f0, double (&qa)[FS], double (&bs)[NCT][FS]) {
      const double2 q0 = load2(qb_ + f0, roff), q1 = load2(qb_ + f0 + 2, roff);
      qa[0] = q0.x; qa[1] = q0.y; qa[2] = q1.x; qa[3] = q1.y;
#pragma unroll
      for (int e = 0; e < FS; ++e)
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
          if (c0[ct] < ncols) bs[ct][e] = (st + (f0 + e) * s.K)[soff[ct]];
    };
    auto mm = [&](const double (&qa)[FS], const double (&bs)[NCT][FS]) {
#pragma unroll
      for (int e = 0; e < FS; ++e)
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
          if (c0[ct] < ncols) acc[ct] = mfma_f64(qa[e], bs[ct][e], acc[ct]);
    };
    if (c0[0] < ncols) {
      ld(0, aa, ba);
      for (int32_t f0 = 0; f0 < s.m; f0 += 8 * FS) {
        ld(f0 + 4 * FS, ab, bb);
        mm(aa, ba);
        if (f0 + 8 * FS < s.m) ld(f0 + 8 * FS, aa, ba);
        mm(ab, bb);
      }
    }
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const int32_t c = c0[ct] + lr;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        double v = acc[ct][i];
        if (s.causal) {
          if (c == tcol[i]) v = diag[i];
          if (c > tcol[i]) v = 0.0;
        }
        if (!act[i] || c >= s.K || c0[ct] >= ncols) v = 0.0;
        acc[ct][i] = v;
      }
    }
  };
  auto add_sums = [&]() {
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int i = 0; i < 4; ++i) rsum[i] += acc[ct][i];
  };
  auto store = [&](int32_t g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int32_t t = r0 + 4 * i + lg;
      if (t >= s.T) continue;
      float* out = A_hat + (head * s.T + t) * s.K;
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        const int32_t c = 64 * (NCT * g + ct) + 16 * cq + lr;
        const float score = static_cast<float>(acc[ct][i] * inv[i]);
        if (SELECT) place[(16 * rt + 4 * i + lg) * kPlace + c] = score;
        if (c < s.K && (!SELECT || A_hat)) out[c] = score;
      }
    }
  };
  auto finish_sums = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double r = rsum[i];
#pragma unroll
      for (int mask = 1; mask < 16; mask <<= 1) r += __shfl_xor(r, mask, kWave);
      if (lr == 0) red_s[rt][cq][4 * i + lg] = r;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = 4 * i + lg;
      const double r = (red_s[rt][0][u] + red_s[rt][1][u]) + (red_s[rt][2][u] + red_s[rt][3][u]);
      inv[i] = r > 0.0 ? 1.0 / r : 0.0;
    }
  };
  if (SELECT || ngroups <= 1) {
    group(0);
    add_sums();
    finish_sums();
    store(0);
  } else {
    for (int32_t g = 0; g < ngroups; ++g) {
      group(g);
      add_sums();
    }
    finish_sums();
    for (int32_t g = 0; g < ngroups; ++g) {
      group(g);
      store(g);
    }
  }
  if constexpr (SELECT) {
    __syncthreads();  // the scores are there
    const int32_t kw = (s.K + 31) / 32;
    for (int rr = 0; rr < 4; ++rr) {
      const int32_t u = 4 * wid + rr, t = r0 - 16 * rt + u;
      if (t >= s.T) break;
      uint32_t* const mrow = mbits + (head * s.T + t) * kw;
      uint64_t take[NCT] = {};
      if (t < len) {
        const int32_t ncand = bucket_of(s.causal ? t : len - 1, s.T, s.K) + 1, n = min(s.k_hat, ncand);
        uint32_t key[NCT];
#pragma unroll
        for (int q = 0; q < NCT; ++q) {
          const float a = place[u * kPlace + 64 * q + lane];  // (columns past K: zeros)
          key[q] = 64 * q + lane < ncand ? ordered_key(a) : 0u;
        }
        const uint32_t tau = nth_largest(key, n);
        int above = 0;
#pragma unroll
        for (int q = 0; q < NCT; ++q) above += popc64(__ballot(key[q] > tau));
        int need = n - above;  // how many of the entries equal to tau are taken, lowest columns first
#pragma unroll
        for (int q = 0; q < NCT; ++q) {
          const uint64_t eq = __ballot(key[q] == tau);
          take[q] = __ballot(key[q] > tau || (key[q] == tau && lanes_below(eq, lane) < need));
          need -= min(need, popc64(eq));
        }
      }
#pragma unroll
      for (int q = 0; q < NCT; ++q) {
        if (lane == 0 && 2 * q < kw) mrow[2 * q] = static_cast<uint32_t>(take[q]);
        if (lane == 0 && 2 * q + 1 < kw) mrow[2 * q + 1] = static_cast<uint32_t>(take[q] >> 32);
      }
    }
    return;
  }
  // columns past the row tile's last one: zeros
  const int32_t all_groups = (s.K + 64 * NCT - 1) / (64 * NCT);  // groups past ncols hold zeros only
  for (int32_t g = max(ngroups, 1); g < all_groups; ++g) {
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) acc[ct] = doublex4{0.0, 0.0, 0.0, 0.0};
    store(g);
  }
}

template <int NFT, int WPT>
void start_features(const Shape& s, dim3 grid, const float* Q, const float* K, const float* W, double* phiQ, double* phiK,
                    double* stateT, int32_t wl, hipStream_t st) {
  if constexpr (NFT > 0) {
    if (stateT) {
      hipLaunchKernelGGL((features_f64_kernel<NFT, WPT, true>), grid, dim3(256), 0, st, s, Q, K, W, phiQ, phiK, stateT, wl);
      return;
    }
  }
  hipLaunchKernelGGL((features_f64_kernel<NFT, WPT>), grid, dim3(256), 0, st, s, Q, K, W, phiQ, phiK, nullptr, 0);
}
// (stateT: the column sums of columns of 2^wl keys, from features_in_columns layers)
void launch_features(const Shape& s, const float* Q, const float* K, const float* W, double* phiQ, double* phiK,
                     double* stateT, int32_t wl, hipStream_t st) {
  const int64_t tiles = 2 * static_cast<int64_t>(s.N) * ((s.T + 15) / 16);
  const dim3 split(static_cast<uint32_t>(tiles)), whole(static_cast<uint32_t>((tiles + 3) / 4));
  if (s.m <= 128 && tiles >= (s.m <= 64 ? 2048 : 3072)) start_features<8, 1>(s, whole, Q, K, W, phiQ, phiK, stateT, wl, st);
  else if (s.m <= 128) start_features<2, 4>(s, split, Q, K, W, phiQ, phiK, stateT, wl, st);
  else if (s.m <= 256) start_features<4, 4>(s, split, Q, K, W, phiQ, phiK, stateT, wl, st);
  else start_features<0, 4>(s, split, Q, K, W, phiQ, phiK, nullptr, 0, st);
}
// log2 of the keys per column where 16-key tiles hold whole columns and the features stay in registers, else -1
int32_t features_in_columns(const Shape& s) {
  if (s.T % 16 != 0 || s.T % s.K != 0 || s.m > 256) return -1;
  const int32_t w = s.T / s.K;
  return w <= 16 && (w & (w - 1)) == 0 ? __builtin_ctz(w) : -1;
}

}  // namespace

// phi(Q) (row-shifted) and phi(K) (zero past seq_len) in fp64, [N][T][m] each
hipError_t launch_features_f64(const Shape& s, const float* Q, const float* K, const float* W, double* phiQ,
                               double* phiK, hipStream_t st) {
  if (s.m % 16 != 0) return hipErrorNotSupported;
  launch_features(s, Q, K, W, phiQ, phiK, nullptr, 0, st);
  return hipGetLastError();
}

size_t estimate_f64_workspace(const Shape& s) {
  const size_t ntm = static_cast<size_t>(s.N) * s.T * s.m;
  const size_t nkm = static_cast<size_t>(s.N) * s.K * s.m;
  return (2 * ntm + nkm) * sizeof(double);
}

// One group of columns: the rows of a block are whole when its scores are.  us, contraction and selection apart / together:
//   K = 128, 12 heads of 4000 rows 78.3 / 72.2, 48 heads of 2048, bidirectional, 147.8 / 141.6; with few blocks the four rows that a
//   wave takes one after the other show (a kernel of its own has a wave per row), the layer, k^ = 32, 12 heads of 320 rows (120
//   blocks) 48.5 / 47.4, of 257 (108) 45.9 / 46.1, of 130 (60) 39.7 / 40.7, 4 heads of 257 (36) 39.0 / 40.0;
//   K <= 64, K % 4 == 0, have a selection kernel that takes sixteen rows per wave, which long launches gain more from than from a
//   launch less: K = 64, 48 heads of 2048 rows 100.2 / 104.3, K = 32, causal, 59.9 / 69.2, K = 64, 12 heads of 512 rows 22.3 / 15.6;
//   other K <= 64, one slot of columns: the layer, K = 50, 12 heads of 130 rows 32.1 / 31.6.
bool estimate_f64_selects(const Shape& s) {
  if (s.K > 128 || s.grouping != 0 || s.geometry != 0) return false;
  const int64_t blocks = static_cast<int64_t>(s.N) * ((s.T + 31) / 32);
  if (s.K > 64) return blocks >= 112;
  return s.K % 4 != 0 || blocks <= 1024;
}

hipError_t launch_estimate_f64(const Shape& s, const float* Q, const float* K, const float* W,
                               float* A_hat, void* ws, hipStream_t st, uint32_t* mbits) {
  const size_t ntm = static_cast<size_t>(s.N) * s.T * s.m;
  double* phiQ = static_cast<double*>(ws);
  double* phiK = phiQ + ntm;
  double* stateT = phiK + ntm;
  const int32_t wl = features_in_columns(s);
  {
    StageScope scope(SEA_STAGE_FEATURES, st);
    launch_features(s, Q, K, W, phiQ, phiK, wl >= 0 ? stateT : nullptr, wl, st);
  }
  if (wl < 0) {
    StageScope scope(SEA_STAGE_STATE, st);
    const int64_t total = static_cast<int64_t>(s.N) * s.K * s.m;
    hipLaunchKernelGGL(state_f64_kernel, dim3(static_cast<uint32_t>((total + 255) / 256)), dim3(256),
                       0, st, s, phiK, stateT);
  }
  {
    StageScope scope(SEA_STAGE_CONTRACT, st);
    const dim3 grid(static_cast<uint32_t>(s.N) * ((s.T + 31) / 32));
#define SEA_LAUNCH_CONTRACT(...) hipLaunchKernelGGL((contract_f64_kernel<__VA_ARGS__>), grid, dim3(512), 0, st, s, phiQ, phiK, stateT, A_hat, mbits)
    if (mbits && s.K <= 64) SEA_LAUNCH_CONTRACT(1, true);
    else if (mbits) SEA_LAUNCH_CONTRACT(2, true);
    else if (s.K <= 64) SEA_LAUNCH_CONTRACT(1);
    else if (s.K <= 128) SEA_LAUNCH_CONTRACT(2);
    else SEA_LAUNCH_CONTRACT(4);
#undef SEA_LAUNCH_CONTRACT
  }
  return hipGetLastError();
}

}  // namespace sea
