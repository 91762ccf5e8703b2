#pragma once
#include "sea_rowlanes.h"

namespace sea {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

// Per-row top-k^ on 16 rows of a wave, in registers.  A row lives in the four lanes l % 16 + 16 q; key[ct][i]
// is the order-preserving key of its column 16 ct + 4 lg + i (bit patterns of negated scores in [0, 1];
// 0x40000000 for columns that are no candidates), nsel its quota, ncnd its number of candidates; columns
// from 16 nct on hold no candidate of the wave's rows.  nib[ct]: bit i set iff that column is selected.
template <int NCT>
__device__ __forceinline__ void select_columns(const uint32_t (&key)[NCT][4], uint32_t nsel, int32_t ncnd, int32_t nct_wave,
                                               int32_t k_hat, int lg, uint32_t (&nib)[NCT]) {
  uint32_t tau = 0x80000000u, cge = static_cast<uint32_t>(ncnd);
  bool dropped = false;  // the row's threshold lies just above the one key too many that it had found
  bool counted = false;  // (uniform) some row's selection may hold equals of one key
  // The compare-and-count loop runs over the tiles that hold candidates of this wave's rows only
  // (causal: the leading ones), in even steps so that a handful of loop bodies covers all cases.
  // Bits 29..16 are searched on the keys' high halves, two keys per register: both halves of
  // hp - trial (16-bit wrap-around differences; candidates and trial lie in [0x8000, 0xc000),
  // non-candidates are 0x4000) have bit 15 set exactly for keys below the trial; a byte permute
  // spreads each sign over a byte, four differences at a time, and the matrix product adds the bytes
  // up.  The trial's
  // low half is zero in that phase, so the counts are those of the full keys.  Bits 15..0 then
  // compare whole keys.
#define SEA_SEARCH_STEP(COUNT_BODY_, REDUCE_)                                                    \
    /* done when every row's count of keys >= tau is its quota or one more */                    \
    if (__ballot(cge > nsel + 1u && nsel != 0u) == 0ull) break;                                  \
    const bool pend = (cge != nsel) && (nsel != 0u);                                             \
    const uint32_t trial = tau | (1u << bit);                                                    \
    uint32_t cnt = 0;                                                                            \
    COUNT_BODY_                                                                                  \
    REDUCE_                                                                                      \
    const bool take = pend && cnt >= nsel;                                                       \
    tau = take ? trial : tau;                                                                    \
    cge = take ? cnt : cge;
#define SEA_SEARCH(NT_)                                                                          \
  {                                                                                              \
    ushort2v hp[2 * (NT_)];                                                                      \
    _Pragma("unroll") for (int ct = 0; ct < (NT_); ++ct) {                                        \
      hp[2 * ct] = __builtin_bit_cast(ushort2v, __builtin_amdgcn_perm(key[ct][1], key[ct][0], 0x07060302u)); \
      hp[2 * ct + 1] = __builtin_bit_cast(ushort2v, __builtin_amdgcn_perm(key[ct][3], key[ct][2], 0x07060302u)); \
    }                                                                                            \
    /* Count of the ROW's keys at or above a trial whose low half is zero.  A byte permute turns  \
       the signs of four differences into four bytes 0x00 / 0xff (selectors 8..11 take the sign \
       of bytes 1, 3, 5, 7), i.e. 0 / -1 as 8-bit integers; sixteen of them are one operand of  \
       the 8-bit matrix product, whose column is the query row (lane % 16) and whose           \
       contraction runs over the lane's sixteen keys and the row's four lanes: against an      \
       all -1 operand every result row is the number of the row's keys BELOW the trial, summed \
       over the four lanes, so the counting and the cross-lane sum leave the vector pipe. */    \
    auto count_high = [&](uint32_t trial_) {                                                     \
      const uint32_t th = trial_ >> 16;                                                          \
      const ushort2v th2 = __builtin_bit_cast(ushort2v, th | (th << 16));                        \
      const intx4 neg1 = {-1, -1, -1, -1};                                                       \
      intx4 below = {0, 0, 0, 0};                                                                \
      _Pragma("unroll") for (int q4 = 0; q4 < ((NT_) + 3) / 4; ++q4) {                            \
        intx4 fl = {0, 0, 0, 0};                                                                 \
        _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                           \
          if (4 * q4 + j < (NT_)) {                                                              \
            const int pr = 2 * (4 * q4 + j);                                                     \
            const uint32_t d0 = __builtin_bit_cast(uint32_t, static_cast<ushort2v>(hp[pr] - th2)); \
            const uint32_t d1 = __builtin_bit_cast(uint32_t, static_cast<ushort2v>(hp[pr + 1] - th2)); \
            fl[j] = static_cast<int>(__builtin_amdgcn_perm(d1, d0, 0x0b0a0908u));                \
          }                                                                                      \
        }                                                                                        \
        below = __builtin_amdgcn_mfma_i32_16x16x64_i8(neg1, fl, below, 0, 0, 0);                 \
      }                                                                                          \
      return 16u * static_cast<uint32_t>(NT_) - static_cast<uint32_t>(below[0]);                 \
    };                                                                                           \
    /* Bits 29..27 at once: a row whose quota of scores lies at or above 2^-15 (rows sum to 1    \
       over at most 256 columns, so nearly every row) would take all three bits, because the     \
       count only grows as the trial falls; one count then stands for three steps.  A wave with  \
       a row that fails the test searches from bit 29 as before. */                              \
    int bit_top = 29;                                                                            \
    {                                                                                            \
      const bool pend = (cge != nsel) && (nsel != 0u);                                           \
      const uint32_t trial = 0xb8000000u;                                                        \
      const uint32_t cnt = count_high(trial);                                                    \
      if (__ballot(pend && cnt < nsel) == 0ull) {                                                \
        tau = pend ? trial : tau;                                                                \
        cge = pend ? cnt : cge;                                                                  \
        bit_top = 26;                                                                            \
      }                                                                                          \
    }                                                                                            \
    _Pragma("unroll 1") for (int bit = bit_top; bit >= 16; --bit) {                               \
      SEA_SEARCH_STEP(cnt = count_high(trial);, )                                                \
    }                                                                                            \
  }                                                                                              \
  _Pragma("unroll 1") for (int bit = 15; bit >= 0; --bit) {                                       \
    SEA_SEARCH_STEP(                                                                             \
      _Pragma("unroll") for (int ct = 0; ct < (NT_); ++ct)                                        \
        _Pragma("unroll") for (int i = 0; i < 4; ++i) cnt += (key[ct][i] >= trial) ? 1u : 0u;,   \
      cnt = rows_sum_u(cnt);)                                                                    \
  }                                                                                              \
  /* A row with one key too many drops its smallest at or above tau (differences that wrap belong \
     to keys below tau).  The slowest of 16 rows would take three more steps of the search for   \
     it, some of them on whole keys.  Layers, us without / with: c4 at T = 32768 758 / 727, c3   \
     400 / 389, c5 74.0 / 70.7, one short sentence 17.4 / 16.1. */                               \
  dropped = cge == nsel + 1u && nsel != 0u;                                                      \
  if (__ballot(dropped) != 0ull) {                                                               \
    uint32_t least = 0xffffffffu;                                                                \
    _Pragma("unroll") for (int ct = 0; ct < (NT_); ++ct)                                          \
      _Pragma("unroll") for (int i = 0; i < 4; ++i) least = min(least, key[ct][i] - tau);         \
    least = rows_min_u(least);                                                                   \
    tau = dropped ? tau + least + 1u : tau;                                                      \
    cge = dropped ? nsel : cge;                                                                  \
  }
  if (k_hat == 1) {
    // one column per row: the threshold is the row maximum itself (several columns holding it
    // are told apart by the tie rule below)
    uint32_t mx = 0u;
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = max(mx, key[ct][i]);
    // (taken for the one key it is; the count of the selection below finds its equals)
    tau = rows_max_u(mx);
    cge = nsel;
    counted = true;
  } else if (NCT >= 16 && nct_wave > 12) {
    SEA_SEARCH(NCT >= 16 ? 16 : NCT)
  } else if (NCT >= 16 && nct_wave > 8) {
    SEA_SEARCH(NCT >= 16 ? 12 : NCT)
  } else if (NCT >= 8 && nct_wave > 6) {
    SEA_SEARCH(NCT >= 8 ? 8 : NCT)
  } else if (NCT >= 8 && nct_wave > 4) {
    SEA_SEARCH(NCT >= 8 ? 6 : NCT)
  } else if (nct_wave > 2) {
    SEA_SEARCH(4)
  } else {
    SEA_SEARCH(2)
  }
#undef SEA_SEARCH
#undef SEA_SEARCH_STEP
  // selection: keys >= tau; when more keys than the quota tie at tau (exact duplicates at the
  // boundary), the lowest columns among them win.  nib[ct]: bit i set iff column 16 ct + 4 lg + i
  // of this lane's row is selected.
  bool tied = __ballot(cge != nsel && nsel != 0u) != 0ull;
  if (!tied) {
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      uint32_t bits = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) bits |= (nsel != 0u && key[ct][i] >= tau) ? (1u << i) : 0u;
      nib[ct] = bits;
    }
    if (counted || __ballot(dropped) != 0ull) {  // where the key that went had equals, they went with it
      uint32_t cnt = 0;
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) cnt += __popc(nib[ct]);
      tied = __ballot(rows_sum_u(cnt) != nsel) != 0ull;
    }
  }
  if (tied) {
    tau = dropped ? tau - 1u : tau;
    uint32_t cgt = 0;
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int i = 0; i < 4; ++i) cgt += (key[ct][i] > tau) ? 1u : 0u;
    cgt = rows_sum_u(cgt);
    int32_t need_eq = static_cast<int32_t>(nsel) - static_cast<int32_t>(cgt);  // ties still to take, in column order
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      uint32_t eqm = 0, gtm = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        eqm |= (key[ct][i] == tau && nsel != 0u) ? (1u << i) : 0u;
        gtm |= (key[ct][i] > tau && nsel != 0u) ? (1u << i) : 0u;
      }
      // columns ascend with (ct, lg, i): ties of lower lane rows of this tile come first
      uint32_t below;
      const uint32_t total = rows_sum_prefix_u(static_cast<uint32_t>(__popc(eqm)), lg, &below);
      uint32_t bits = gtm;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int32_t rank = static_cast<int32_t>(below) + __popc(eqm & ((1u << i) - 1u));
        if (((eqm >> i) & 1u) && rank < need_eq) bits |= 1u << i;
      }
      nib[ct] = bits;
      need_eq -= min(need_eq, static_cast<int32_t>(total));
    }
  }
}

}  // namespace sea
