// Tiled attention for column-selected masks of ANY column widths (Sec. 3.1.1 rho, sigma, A* V with
// the mask of Sec. 3.1 "Linear Sparse Attention Mask Generation", App. A.5.3): K need not divide T
// and a selected column may emit any number of keys.  bf16 tensors; the power-of-two shapes have a
// kernel of their own (sea_tile_attn.hip), whose register groups share one mask bit, and so have layers
// whose rows select few keys (sea_column_gather.hip).
//
// The keys a head can use form one compact list, ascending in position: all T keys when whole
// columns are emitted, else r keys of each of the K columns.  A block of 4 waves takes 128 query
// rows (other splits below) and walks it in 64-key steps staged through LDS, as the power-of-two kernel does.  With
// columns of any width a lane's score registers belong to columns that change from step to step, so
// bit tests per register would cost more than the softmax.  The mask goes through the matrix
// product instead: the contraction is extended by NX slots, one per column of the 32-key sub-chunk.
// On the key side slot x holds the lowest bf16 value, -(1 - 2^-8) 2^128, for the keys of the sub-chunk's
// x-th column (one-hot, staged beside the keys, the same for every row and head); on
// the query side it holds 2 where the row did NOT select that column and 0 where it did.  One more
// 32x32x16 product then takes every finite unselected score below -(1 - 2^-6) 2^128 and adds exact zeros to
// the others.  Building the query side takes nine vector instructions per sub-chunk from the row's mask
// window.
//
// What a row does not select cannot reach it: a score that is not finite passes the mask as NaN, and a value
// that is not finite gives NaN against a weight of zero, so a row whose accumulators and sum are finite met
// neither.  The others (and rows whose scores all lie at the mask's level) are computed again from their own
// keys at the end of the block.
//
// The softmax weights go into the second product as the sum of three bf16 values (sea_tile.h), i.e. as the
// fp32 numbers they are: products of weights and values are exact, as in the per-row kernel.
//
// Bound: issue (about 200 vector instructions and 17 matrix products per 32-key sub-chunk and wave).  The keys and
// values of a step go straight to LDS, which leaves registers for four waves per SIMD (three before).  On the layer
// B = 8, H = 32, T = 2000 (padded by 0-25 %), K = 256, k^ = 64 the kernel takes 0.26 ms (0.29 ms with three waves per
// SIMD and rows that pass through registers); the per-row gather kernel takes 2.71 ms and its key lists another
// 0.57 ms to write.  Small launches take as long as their longest list: there three or six sets of waves share it.
#include "sea_columns.h"
#include "sea_gather.h"
#include "sea_internal.h"
#include "sea_tile.h"

#include <type_traits>

namespace sea {
namespace {

// Staged rows are 128 bytes, their 16-byte pieces exchanged by row as in the power-of-two kernel.
constexpr int kRow = kHeadDim;

struct ColumnArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const uint16_t* V;
  const uint32_t* mbits;  // [N][T][KW] selected-column bits
  uint16_t* O;
  const int32_t* seq_len;
  int32_t N, H, T, KW;
  ColumnList g;
  // column of list entry u = floor(u A / D); 32 entries further: q32 more, remainder r32 more
  int32_t A, D, q32, r32;
  int32_t qh, rh, qs, rs;  // and half a step, a step further
  int32_t causal, group_heads;
  float c;           // scale * log2(e)
};

// NX = contraction slots for the mask: 8 (at least 5 keys per column: a 32-key sub-chunk touches at
// most 8 columns), 16 (3 or 4 keys) or 32 (1 or 2 keys).
// RW waves side by side take 32 rows each; NS sets of them share the rows, each with every NS-th SC sub-chunks of
// the list (see the launch).
// ODD: K or V starts between two 4-byte words, so a step's pieces wait in registers (three waves per SIMD).
template <int NX, int RW, int NS, int SC, bool ODD = false>
__global__ __launch_bounds__(64 * RW * NS, NS == 1 && !ODD ? 4 : 3) void column_attn_kernel(ColumnArgs a) {
  constexpr int kRows = 32 * RW, kThreads = 64 * RW * NS, kWaves = RW * NS;
  constexpr int kStep = 32 * SC * NS;  // keys per step
  static_assert(8 * kStep == 2 * kThreads, "two K and V pieces per thread and step");
  __shared__ __attribute__((aligned(16))) uint16_t KVs[2][2][kStep * kRow];  // [place][K, V]
  __shared__ __attribute__((aligned(16))) uint16_t Xs[2][kStep * NX];        // the keys' slots of the mask product
  extern __shared__ uint32_t Ms[];  // the block's rows' mask words, KW per row
  const int tid = threadIdx.x, lane = tid & 63;
  const int wall = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wid = NS > 1 ? wall % RW : wall, set = NS > 1 ? wall / RW : 0;
  const int ql = lane & 31, g = lane >> 5;
  // launch order as in the power-of-two kernel: heads in groups, in a group the longest tiles first
  const uint32_t wgs = (a.T + kRows - 1) / kRows;
  const uint32_t per_group = static_cast<uint32_t>(a.group_heads) * wgs;
  const uint32_t place_b = dealt_in_turn(blockIdx.x, gridDim.x, NS == 1 ? 4 : 1, a.causal);
  const uint32_t grp = place_b / per_group, rem_b = place_b - grp * per_group;
  const uint32_t nh = min(static_cast<uint32_t>(a.group_heads), static_cast<uint32_t>(a.N) - grp * a.group_heads);
  const int64_t head = static_cast<int64_t>(grp) * a.group_heads + rem_b % nh;
  const int32_t wg_tile = static_cast<int32_t>(wgs - 1 - rem_b / nh);
  const int32_t row0 = wg_tile * kRows, q0 = row0 + 32 * wid, t = q0 + ql;
  const int32_t b = static_cast<int32_t>(head / a.H);
  const int32_t len = a.seq_len ? min(max(a.seq_len[b], 0), a.T) : a.T;
  if (row0 >= len && padding_returns(gridDim.x, NS == 1 ? 4 : 1, a.causal)) {  // nothing but padding: no keys are walked for it
    zero_rows<kThreads>(a.O + (head * a.T + row0) * kHeadDim, min(kRows, a.T - row0));
    return;
  }
  const bool row_active = t < len;
  const int32_t wg_hi = min(row0 + kRows - 1, a.T - 1), t_hi = min(q0 + 31, a.T - 1);
  const int32_t u_end_wg = list_count(a.g, a.causal ? min(wg_hi, len - 1) : len - 1);
  const int32_t u_end = q0 < len ? list_count(a.g, a.causal ? min(t_hi, len - 1) : len - 1) : 0;
  // entries below u_free are admissible for every active row of the wave
  const int32_t u_free = min(u_end, list_count(a.g, a.causal ? min(q0, len - 1) : len - 1));
  const int32_t my_ucount = list_count(a.g, row_active ? (a.causal ? min(t, len - 1) : len - 1) : -1);
  const int32_t nsteps = (u_end_wg + kStep - 1) / kStep;

  // staging: slot tid & 7 of the K and V rows (tid >> 3) and (tid >> 3) + 8 kWaves of a step: its wave's
  // first rows lie in the step's sub-chunk wall / 4, its second ones in sub-chunk (wall + kWaves) / 4.  The rows go
  // straight to LDS.  Rows past the list or past the sequence re-read its last row; their scores are masked.
  const int srow = tid >> 3, spart = tid & 7;
  const uint32_t kpart = 16 * (spart ^ ((srow >> 1) & 7)), vpart = 16 * (spart ^ (((srow >> 1) & 1) << 2));
  uint32_t x0[NX == 32 ? 2 : 1], x1[NX == 32 ? 2 : 1];  // this thread's words of the two rows' one-hot slots
  const uint32_t row_bytes = kHeadDim * 2, head_bytes = static_cast<uint32_t>(a.T) * row_bytes;
  const uint16_t* Kh = a.K + head * static_cast<int64_t>(a.T) * kHeadDim;
  const uint16_t* Vh = a.V + head * static_cast<int64_t>(a.T) * kHeadDim;
  const u32x4 Kres = buffer_words(Kh, head_bytes), Vres = buffer_words(Vh, head_bytes);
  // column and remainder of this thread's next row, and of the next sub-chunk's first entry
  int32_t ucur = srow, ccol = (srow * a.A) / a.D, crem = srow * a.A - ccol * a.D;
  int32_t scol = 0, srem = 0;
  auto advance_by = [&](int32_t& col, int32_t& rem, int32_t q, int32_t r) {
    col += q;
    rem += r;
    const bool carry = rem >= a.D;
    col += carry ? 1 : 0;
    rem -= carry ? a.D : 0;
  };
  auto advance = [&](int32_t& col, int32_t& rem) { advance_by(col, rem, a.q32, a.r32); };
  // half a step and a whole one further (NS == 1: two sub-chunks per step)
  auto advance_half = [&](int32_t& col, int32_t& rem) { advance_by(col, rem, a.qh, a.rh); };
  // (several sets) first columns of the sub-chunks this wave's two rows lie in
  int32_t tcol0 = 0, trem0 = 0, tcol1 = 0, trem1 = 0;
  if (NS > 1) {
    for (int e = 0; e < (wall >> 2); ++e) advance(tcol0, trem0);
    for (int e = 0; e < ((wall + kWaves) >> 2); ++e) advance(tcol1, trem1);
    for (int e = 0; e < SC * set; ++e) advance(scol, srem);
  }
  auto onehot = [&](int32_t lc, uint32_t* x) {
    const uint32_t v = (lc & 1) ? 0xff7f0000u : 0x0000ff7fu;  // the lowest value
#pragma unroll
    for (int e = 0; e < (NX == 32 ? 2 : 1); ++e) x[e] = (lc >> 1) == spart + 8 * e ? v : 0u;
  };
  auto row_off = [&]() -> uint32_t {
    const int32_t pos = a.g.r == 0 ? ucur : entry_pos(a.g, ccol, crem);
    return static_cast<uint32_t>(max(min(pos, len - 1), 0)) * row_bytes;
  };
  int32_t cs0 = 0, cs1 = 0, cs2 = 0;  // first columns of the fetched step's sub-chunks and of the one after
  u32x4 odd[4];
  auto park = [&](int place) __attribute__((always_inline)) {
    if constexpr (ODD) {
      uint16_t* const at = &KVs[place][0][wall * 8 * kRow];
      park16(at, odd[0]);
      park16(at + 8 * kWaves * kRow, odd[1]);
      park16(at + kStep * kRow, odd[2]);
      park16(at + (kStep + 8 * kWaves) * kRow, odd[3]);
    }
  };
  auto fetch = [&](int place) __attribute__((always_inline)) {
    cs0 = scol;
    if (NS == 1) {
      advance(scol, srem);
      cs1 = scol;
      advance(scol, srem);
      cs2 = scol;
    } else {
      int32_t ncol = scol, nrem = srem;
      advance(ncol, nrem);
      cs1 = ncol;
      if (SC == 2) advance(ncol, nrem);
      cs2 = ncol;
      advance_by(scol, srem, a.qs, a.rs);
    }
    const uint32_t oa = row_off();
    onehot(ccol - (NS == 1 ? cs0 : tcol0), x0);
    ucur += kStep / 2;
    advance_half(ccol, crem);
    const uint32_t ob = row_off();
    onehot(ccol - (NS == 1 ? cs1 : tcol1), x1);
    ucur += kStep / 2;
    advance_half(ccol, crem);
    if (NS > 1) advance_by(tcol0, trem0, a.qs, a.rs);
    if (NS > 1) advance_by(tcol1, trem1, a.qs, a.rs);
    if constexpr (ODD) {
      odd[0] = load16_odd(Kres, oa + kpart);
      odd[1] = load16_odd(Kres, ob + kpart);
      odd[2] = load16_odd(Vres, oa + vpart);
      odd[3] = load16_odd(Vres, ob + vpart);
    } else {
      uint16_t* const at = &KVs[place][0][wall * 8 * kRow];
      buffer_load_lds16(Kres, at, oa + kpart, at + 8 * kWaves * kRow, ob + kpart);
      buffer_load_lds16(Vres, at + kStep * kRow, oa + vpart, at + (kStep + 8 * kWaves) * kRow, ob + vpart);
    }
    if (NX >= 16 || spart < NX / 2) {
#pragma unroll
      for (int e = 0; e < (NX == 32 ? 2 : 1); ++e) {
        *reinterpret_cast<uint32_t*>(&Xs[place][srow * NX + 2 * (spart + 8 * e)]) = x0[e];
        *reinterpret_cast<uint32_t*>(&Xs[place][(srow + 8 * kWaves) * NX + 2 * (spart + 8 * e)]) = x1[e];
      }
    }
  };
  // the first step's rows and the mask words are requested ahead of the query rows
  if (nsteps > 0) fetch(0);
  {
    const int32_t nwords = min(kRows, a.T - row0) * a.KW;  // (words past the last row repeat the last one)
    const u32x4 Mres = buffer_words(a.mbits + (head * a.T + row0) * a.KW, static_cast<uint32_t>(nwords) * 4u);
    for (int32_t x = 0; x < kRows * a.KW; x += kThreads)
      buffer_load_lds4(Mres, &Ms[x + 64 * wall], static_cast<uint32_t>(min(x + tid, nwords - 1)) * 4u);
  }
  const uint32_t* mrow = &Ms[(32 * wid + ql) * a.KW];
  const uint32_t row_closed = row_active ? 0u : 0xffffffffu;
  const uint16_t* Qr = a.Q + (head * a.T + min(t, a.T - 1)) * kHeadDim + 8 * g;
  bf16x8 bq[4];
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) bq[kc] = *reinterpret_cast<const bf16x8*>(Qr + 16 * kc);
  // (through an empty asm: plain register values inside the loop, not results of pending loads)
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) asm volatile("" : "+v"(bq[kc]));

  // this lane's pieces of a K row: slots 2 kc + g of row ql
  int kat[4];
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) kat[kc] = ql * kRow + 8 * ((2 * kc + g) ^ ((ql >> 1) & 7));

  floatx16 oacc[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) { oacc[0][i] = 0.f; oacc[1][i] = 0.f; }
  // Streaming softmax in log2 units, y = s c - m_ref.  A masked score is about -2^128 c (or -inf), far
  // below m_thr's start value, so it never becomes a reference; afterwards m_thr is how far a row's
  // maximum may exceed its reference before that is moved.
  float m_ref = 0.f, m_thr = -fminf(a.c * 0x1p126f, 3.0e38f), l_run = 0.f;
  const uint32_t gmask = (NX == 8 && g != 0) ? 0u : 0x40004000u;  // NX = 8: the upper half's slots are unused

  const MinusOnes minus = minus_ones();

  if (nsteps > 0) park(0);
  lds_loads_done();
  __syncthreads();
  // one step, its place in the double buffer known to the compiler
  auto walk = [&](int32_t step, auto stage_c) __attribute__((always_inline)) {
    constexpr int stage = decltype(stage_c)::value;
    const int32_t c0[3] = {cs0, cs1, cs2};  // (uniform) columns at the start of this step's sub-chunks
    if (step + 1 < nsteps) fetch(stage ^ 1);
#pragma unroll
    for (int sc = 0; sc < SC; ++sc) {
      const int32_t u0 = step * kStep + 32 * (SC * set + sc);
      if (u0 >= u_end) break;  // wave-uniform: beyond what this wave's rows can see
      const int32_t wi = c0[sc] >> 5;
      // the row's unselected columns from the sub-chunk's first one on (past the last column: of entries past the list)
      const uint32_t win = ~__builtin_amdgcn_alignbit(mrow[min(wi + 1, a.KW - 1)], mrow[min(wi, a.KW - 1)], c0[sc] & 31) | row_closed;
      const int32_t ncol = min(c0[sc + 1] - c0[sc] + 1, NX);
      const uint32_t cmask = 0xffffffffu >> (32 - ncol);
      if (__ballot((win & cmask) != cmask) == 0ull) continue;  // no row of the wave uses it
      const uint16_t* Kr = &KVs[stage][0][32 * (SC * set + sc) * kRow];
      floatx16 sv;
#pragma unroll
      for (int i = 0; i < 16; ++i) sv[i] = 0.f;
#pragma unroll
      for (int kc = 0; kc < 4; ++kc)
        sv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(Kr + kat[kc]), bq[kc],
                                                     sv, 0, 0, 0);
      // mask product: slots 8 g .. 8 g + 7 of this lane half (and 16 more for NX = 32)
#pragma unroll
      for (int e = 0; e < (NX == 32 ? 2 : 1); ++e) {
        const uint32_t un = NX == 8 ? (win & 0xffu) : ((win >> (16 * e + 8 * g)) & 0xffu);
        const uint32_t xx = un | (un << 15);  // bits 2 j and 2 j + 1 sit at 2 j and 2 j + 16
        const u32x4 bx = {(xx << 14) & gmask, (xx << 12) & gmask, (xx << 10) & gmask, (xx << 8) & gmask};
        const uint16_t* Ke = &Xs[stage][(32 * (SC * set + sc) + ql) * NX + (NX == 8 ? 0 : 16 * e + 8 * g)];
        sv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(Ke),
                                                     __builtin_bit_cast(bf16x8, bx), sv, 0, 0, 0);
      }
      float y[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) y[i] = fmaf(sv[i], a.c, -m_ref);
      if (u0 + 32 > u_free) {  // straddles the causal diagonal or the end of the sequence
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int32_t slot = 8 * (i >> 2) + 4 * g + (i & 3);  // reg i <-> entry u0 + slot
          y[i] = u0 + slot < my_ucount ? y[i] : -INFINITY;
        }
      }
      // V^T fragments through the LDS transpose read, requested ahead of the softmax
      bf16x8 av[2][2];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const uint16_t* Vr = &KVs[stage][1][(32 * (SC * set + sc) + 4 * g + ((ql & 15) >> 2)) * kRow +
                                        32 * (mt ^ ((ql >> 3) & 1)) + (ql & 16) + 4 * (ql & 3)];
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) {
          const bf16x4 lo = lds_transpose4(Vr + (16 * c2) * kRow);
          const bf16x4 hi = lds_transpose4(Vr + (16 * c2 + 8) * kRow);
          av[mt][c2] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
      }
      float ymax = max_of(y);
      if (__ballot(ymax > m_thr) != 0ull) {
        ymax = half_max(ymax);
        const bool refresh = ymax > m_thr;
        const float delta = refresh ? ymax : 0.f;
        const float corr = (refresh && m_thr > 0.f) ? __builtin_amdgcn_exp2f(-delta) : 1.f;
        l_run *= corr;
#pragma unroll
        for (int i = 0; i < 16; ++i) { oacc[0][i] *= corr; oacc[1][i] *= corr; }
        m_ref += delta;
        m_thr = refresh ? kRefSlack : m_thr;
#pragma unroll
        for (int i = 0; i < 16; ++i) y[i] -= delta;
      }
      // O^T += V^T P^T, V^T fragments in the key order of the P registers
      l_run += add_weighted_rows(y, av, minus, oacc);
    }
    if (step + 1 < nsteps) park(stage ^ 1);
    lds_loads_done();
    __syncthreads();
  };
  for (int32_t step = 0; step < nsteps; step += 2) {
    walk(step, std::integral_constant<int, 0>{});
    if (step + 1 < nsteps) walk(step + 1, std::integral_constant<int, 1>{});
  }
  if constexpr (NS > 1) {
    // merge of the sets' partial results in the place of the last step's keys and values (the loop ended
    // with a barrier)
    constexpr int kPart = 64 * RW * kPartFloats;
    static_assert((NS - 1) * kPart * 4 <= static_cast<int>(sizeof(KVs)), "every set's result has a place");
    auto place = [&](int e) { return reinterpret_cast<float*>(&KVs[0][0][0]) + (e - 1) * kPart + 64 * wid + lane; };
    float m_own = m_thr > 0.f ? m_ref : -INFINITY;
    if (set > 0) store_part<64 * RW>(place(set), oacc, l_run, m_own);
    __syncthreads();
    if (set > 0) return;
    for (int e = 1; e < NS; ++e) merge_part<64 * RW>(place(e), oacc, l_run, m_own);
  }
  l_run = half_sum(l_run);
  uint32_t rows_again = rows_not_finite(l_run, oacc) & static_cast<uint32_t>(__ballot(row_active));
  if (!row_active) {  // zero times what it met need not be zero
#pragma unroll
    for (int i = 0; i < 16; ++i) { oacc[0][i] = 0.f; oacc[1][i] = 0.f; }
  }
  uint32_t selected = 0u;
  if (!(l_run > 0.f)) {  // no weight at all: rows without keys, or scores at the mask's level
    for (int32_t wi = 0; wi < a.KW; ++wi) selected |= mrow[wi];
  }
  rows_again |= static_cast<uint32_t>(__ballot(row_active && selected != 0u));  // (both halves hold the row's words)
  if (rows_again != 0u) {
    // (the column list takes the place of the mask words of the wave's rows, which no other wave reads now)
    uint16_t* const place = reinterpret_cast<uint16_t*>(&Ms[32 * wid * a.KW]);
    for (uint32_t rows = rows_again; rows != 0u; rows &= rows - 1u) {
      const int64_t tr = q0 + __ffs(static_cast<int>(rows)) - 1, row = head * a.T + tr;
      const ColumnKeys keys(a.g, a.mbits + row * a.KW, a.KW, a.causal ? min(static_cast<int32_t>(tr), len - 1) : len - 1, place);
      gather_row_bf16(keys, a.c, a.Q + row * kHeadDim, Kh, Vh, a.O + row * kHeadDim);
    }
  }
  const float inv = (row_active && l_run > 0.f) ? 1.f / l_run : 0.f;
  // (behind the partial results of other waves, where there are such)
  constexpr int kPartBytes = (NS - 1) * 64 * RW * kPartFloats * 4;
  static_assert(kPartBytes + RW * 32 * kRow * 2 <= static_cast<int>(sizeof(KVs)), "rows on their way out fit the keys' and values' place");
  store_rows(&KVs[0][0][0] + kPartBytes / 2 + wid * 32 * kRow, oacc, inv, 0u, [&](int r) -> uint16_t* {
    return q0 + r < a.T && ((rows_again >> r) & 1u) == 0u ? a.O + (head * a.T + q0 + r) * kHeadDim : nullptr;
  });
}

template <int NX, int RW, int NS, int SC, bool ODD = false>
void launch_column(const Shape& s, ColumnArgs a, hipStream_t st) {
  if constexpr (!ODD) {
    if (starts_odd(a.K) || starts_odd(a.V)) return launch_column<NX, RW, NS, SC, true>(s, a, st);
  }
  constexpr int kRows = 32 * RW, kThreads = 64 * RW * NS, kStep = 32 * SC * NS;  // (mask words arrive kThreads at a time)
  a.qh = kStep / 2 * a.A / a.D; a.rh = kStep / 2 * a.A % a.D;
  a.qs = kStep * a.A / a.D; a.rs = kStep * a.A % a.D;
  hipLaunchKernelGGL((column_attn_kernel<NX, RW, NS, SC, ODD>), dim3(static_cast<uint32_t>(s.N) * ((s.T + kRows - 1) / kRows)),
                     dim3(64 * RW * NS), static_cast<size_t>((kRows * a.KW + kThreads - 1) / kThreads * kThreads) * sizeof(uint32_t), st, a);
}

}  // namespace

// Any fixed-bucket selection; the scale must leave -2^128 scale far below every real score.
bool column_attn_supported(const Shape& s, sea_dtype dt) {
  return dt == SEA_BF16 && column_list_supported(s) && s.scale > 1e-20f;
}

hipError_t launch_column_attn(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                              const uint32_t* mbits, uint16_t* O, hipStream_t st) {
  if (!column_attn_supported(s, SEA_BF16)) return hipErrorNotSupported;
  if (column_gather_pays(s, SEA_BF16)) return launch_column_gather(s, SEA_BF16, Q, K, V, mbits, O, st);
  StageScope scope(SEA_STAGE_SPARSE, st);
  ColumnArgs a{};
  a.Q = Q; a.K = K; a.V = V; a.mbits = mbits; a.O = O; a.seq_len = s.seq_len;
  a.N = s.N; a.H = s.H; a.T = s.T; a.KW = (s.K + 31) / 32;
  a.g = column_list(s);
  a.A = a.g.r == 0 ? s.K : 1; a.D = a.g.r == 0 ? s.T : a.g.r;
  a.q32 = 32 * a.A / a.D; a.r32 = 32 * a.A % a.D;
  a.causal = s.causal; a.c = s.scale * kLog2e;
  a.group_heads = group_heads_for(s, a.g.U);
  // How the waves of a block are split: three sets of four waves where the launch leaves room (128-row blocks:
  // one per CU; causal, two, since half of them are short) or its longest lists dominate it, and six sets of
  // two on 64 rows where those still leave room.  Whole forward, K = 128, k^ = 48, H = 12, causal, us with one /
  // three / six sets: T = 501, B = 1 (48 blocks) 35 / 33 / 29, B = 4 (192) 38 / 36 / 38; T = 1001, B = 1 (96)
  // 51 / 44 / 37, B = 4 (384) 59 / 55 / 62; T = 2041, B = 1 (192) 83 / 66 / 55, B = 2 (384) 86 / 70 / 80, B = 4
  // (768) 106 / 118 / 140; whole columns of T = 8001 (756) 355 / 303 / 299, T = 16001 (1512) 1095 / 859 / -;
  // bidirectional, T = 2041, B = 1 81 / 64 / 75, B = 2 104 / 104 / 103.
  const int64_t blocks = static_cast<int64_t>(s.N) * ((s.T + 127) / 128);
  const bool six = blocks <= (s.causal && a.g.U >= 2000 ? 256 : 128);
  const bool three = blocks <= 256 || (s.causal && (blocks <= 512 || (blocks <= 2048 && a.g.U >= 8000)));
  const int32_t per = a.g.r == 0 ? a.g.cg.w0 : a.g.r;  // least keys per column
#define SEA_COLUMN(NX_)                                     \
  if (six) launch_column<NX_, 2, 6, 1>(s, a, st);           \
  else if (three) launch_column<NX_, 4, 3, 2>(s, a, st);    \
  else launch_column<NX_, 4, 1, 2>(s, a, st)
  if (per >= 5) { SEA_COLUMN(8); }
  else if (per >= 3) { SEA_COLUMN(16); }
  else { SEA_COLUMN(32); }
#undef SEA_COLUMN
  return hipGetLastError();
}

}  // namespace sea
