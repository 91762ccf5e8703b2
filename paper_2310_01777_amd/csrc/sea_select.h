#pragma once
#include "sea_rowlanes.h"
#include "sea_search.h"

namespace sea {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

// Marks of keys at or above a floor, one comparison and one addition each: the comparison's bit is carried into twice the
// marks so far.  A comparison's mask is read two instructions later at the earliest, the distance that gfx950 wants between
// a vector instruction that writes scalars and one that reads them.
// bits i and 16 + i: a[i] and b[i]
__device__ __forceinline__ uint32_t mark_at_least(const uint32_t (&a)[4], const uint32_t (&b)[4], uint32_t floor) {
  uint32_t w = 0;
  uint64_t m0, m1, m2;
  asm(
      "v_cmp_ge_u32 %1, %11, %12\n\tv_cmp_ge_u32 %2, %10, %12\n\t"
      "v_cmp_ge_u32 %3, %9, %12\n\tv_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
      "v_cmp_ge_u32 %1, %8, %12\n\tv_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
      "v_cmp_ge_u32 %2, %7, %12\n\tv_addc_co_u32 %0, vcc, %0, %0, %3\n\t"
      "v_cmp_ge_u32 %3, %6, %12\n\tv_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
      "v_lshlrev_b32 %0, 12, %0\n\tv_cmp_ge_u32 %1, %5, %12\n\t"
      "v_addc_co_u32 %0, vcc, %0, %0, %2\n\tv_cmp_ge_u32 %2, %4, %12\n\t"
      "v_addc_co_u32 %0, vcc, %0, %0, %3\n\tv_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
      "v_addc_co_u32 %0, vcc, %0, %0, %2"
      : "+&v"(w), "=&s"(m0), "=&s"(m1), "=&s"(m2)
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(floor)
      : "vcc");
  return w;
}
// w with sixteen bits more at its low end, bit i for the bits of v[i]
typedef float floatx16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ uint32_t mark_at_least(floatx16 v, uint32_t floor, uint32_t w) {
  uint64_t m0, m1, m2;
  asm(
      "v_cmp_ge_u32 %1, %19, %20\n\tv_cmp_ge_u32 %2, %18, %20\n\t"
      "v_cmp_ge_u32 %3, %17, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
      "v_cmp_ge_u32 %1, %16, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
      "v_cmp_ge_u32 %2, %15, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %3\n\t"
      "v_cmp_ge_u32 %3, %14, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
      "v_cmp_ge_u32 %1, %13, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
      "v_cmp_ge_u32 %2, %12, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %3\n\t"
      "v_cmp_ge_u32 %3, %11, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
      "v_cmp_ge_u32 %1, %10, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
      "v_cmp_ge_u32 %2, %9, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %3\n\t"
      "v_cmp_ge_u32 %3, %8, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
      "v_cmp_ge_u32 %1, %7, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
      "v_cmp_ge_u32 %2, %6, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %3\n\t"
      "v_cmp_ge_u32 %3, %5, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
      "v_cmp_ge_u32 %1, %4, %20\n\tv_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
      "v_addc_co_u32 %0, vcc, %0, %0, %3\n\tv_addc_co_u32 %0, vcc, %0, %0, %1"
      : "+&v"(w), "=&s"(m0), "=&s"(m1), "=&s"(m2)
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]),
        "v"(v[8]), "v"(v[9]), "v"(v[10]), "v"(v[11]), "v"(v[12]), "v"(v[13]), "v"(v[14]), "v"(v[15]), "v"(floor)
      : "vcc");
  return w;
}

// Where the search of a row starts from above: fewer than nsel keys have a high half at or above this.  Scores that sum to
// one (`sums`) hold fewer than nsel of 1.02 / nsel; anything else below infinity lies under 0xc000.
__device__ __forceinline__ float search_top(uint32_t nsel, bool sums) {
  const uint32_t bound = __float_as_uint(1.02f * __builtin_amdgcn_rcpf(static_cast<float>(max(nsel, 1u))));
  return static_cast<float>(sums ? (0x8000u | (bound >> 16)) + 1u : 0xc000u);
}

// Per-row top-k^ on 16 rows of a wave, in registers.  A row lives in the four lanes l % 16 + 16 q; key[ct][i]
// is the order-preserving key of its column 16 ct + 4 lg + i (bit patterns of negated scores in [0, 1];
// from 0x40000000 below 0x80000000 for columns that are no candidates), nsel its quota, ncnd its number of candidates; columns
// from 16 nct on hold no candidate of the wave's rows; top: see search_top.  sel[j]: bit 16 h + i set iff column
// 16 (2 j + h) + 4 lg + i is selected.
template <int NCT>
__device__ __forceinline__ void select_columns(const uint32_t (&key)[NCT][4], uint32_t nsel, int32_t ncnd, int32_t nct_wave,
                                               int32_t k_hat, float top, int lg, uint32_t (&sel)[NCT / 2]) {
  uint32_t tau = 0x80000000u, cge = static_cast<uint32_t>(ncnd);
  bool dropped = false;  // the row's threshold lies just above the one key too many that it had found
  bool lacking = false;  // the row's threshold is the largest key below one that leaves it a key short
  bool counted = false;  // (uniform) some row's selection may hold equals of one key
  // The compare-and-count loop runs over the tiles that hold candidates of this wave's rows only
  // (causal: the leading ones), in even steps so that a handful of loop bodies covers all cases.
  // The keys' high halves are searched first, two keys per register: both halves of hp - trial (16-bit
  // wrap-around differences; candidates and trial lie in [0x8000, 0xc000), non-candidates in [0x4000, 0x8000)) have bit 15 set
  // exactly for keys below the trial; a byte permute spreads each sign over a byte, four differences at a time, and
  // the matrix product adds the bytes up.  The trial's low half is zero in that phase, so the counts are those of the
  // full keys.
  // Trials between two counts (RowSearch); done when a row has its quota, one key more or one fewer.
#define SEA_SEARCH(NT_)                                                                          \
  {                                                                                              \
    ushort2v hp[2 * (NT_)];                                                                      \
    _Pragma("unroll") for (int ct = 0; ct < (NT_); ++ct) {                                        \
      hp[2 * ct] = __builtin_bit_cast(ushort2v, __builtin_amdgcn_perm(key[ct][1], key[ct][0], 0x07060302u)); \
      hp[2 * ct + 1] = __builtin_bit_cast(ushort2v, __builtin_amdgcn_perm(key[ct][3], key[ct][2], 0x07060302u)); \
    }                                                                                            \
    /* Number of the ROW's keys below a trial whose low half is zero.  A byte permute turns      \
       the signs of four differences into four bytes 0x00 / 0xff (selectors 8..11 take the sign \
       of bytes 1, 3, 5, 7), i.e. 0 / -1 as 8-bit integers; sixteen of them are one operand of  \
       the 8-bit matrix product, whose column is the query row (lane % 16) and whose           \
       contraction runs over the lane's sixteen keys and the row's four lanes: against an      \
       all -1 operand every result row is the number of the row's keys BELOW the trial, summed \
       over the four lanes, so the counting and the cross-lane sum leave the vector pipe. */    \
    auto count_below = [&](uint32_t th) {                                                        \
      const ushort2v th2 = __builtin_bit_cast(ushort2v, __builtin_amdgcn_perm(th, th, 0x01000100u)); \
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
      return below[0];                                                                           \
    };                                                                                           \
    /* (rows without a quota start with nothing to search; whole numbers below 2^16 throughout) */ \
    const float over = static_cast<float>(16 * (NT_)) - static_cast<float>(nsel);                \
    RowSearch row = {nsel != 0u ? 32768.f : top - 1.f, top, static_cast<float>(ncnd) - static_cast<float>(nsel), \
                     static_cast<float>(nsel) + 0.25f};                                          \
    _Pragma("unroll 1") for (int32_t step = 0; __ballot(row.pending()) != 0ull; ++step) {        \
      const float trial = row.trial(step, __builtin_amdgcn_rcpf(row.a + row.b));                 \
      row.counted(trial, over - static_cast<float>(count_below(static_cast<uint32_t>(trial))));  \
    }                                                                                            \
    lacking = row.a > 1.f && row.b == 1.f && nsel != 0u;                                         \
    cge = lacking ? nsel : nsel + static_cast<uint32_t>(row.a);                                  \
    tau = static_cast<uint32_t>(lacking ? row.hi : row.lo) << 16;                                \
  }                                                                                              \
  /* rows with several keys of one high half around their quota: bits 15..0 on whole keys */     \
  _Pragma("unroll 1") for (int bit = 15; bit >= 0; --bit) {                                       \
    if (__ballot(cge > nsel + 1u && nsel != 0u) == 0ull) break;                                  \
    const bool pend = (cge != nsel) && (nsel != 0u);                                             \
    const uint32_t trial = tau | (1u << bit);                                                    \
    uint32_t cnt = 0;                                                                            \
    _Pragma("unroll") for (int ct = 0; ct < (NT_); ++ct)                                          \
      _Pragma("unroll") for (int i = 0; i < 4; ++i) cnt += (key[ct][i] >= trial) ? 1u : 0u;      \
    cnt = rows_sum_u(cnt);                                                                       \
    const bool take = pend && cnt >= nsel;                                                       \
    tau = take ? trial : tau;                                                                    \
    cge = take ? cnt : cge;                                                                      \
  }                                                                                              \
  /* A row with one key too many drops its smallest at or above tau, a row with one too few takes its largest below tau    \
     (differences that wrap belong to keys on the other side, and those of non-candidates are larger than any key's).      \
     The slowest of 16 rows would take three more steps of the search for it, some of them on whole keys.  Layers, us       \
     without / with the dropping: c4 at T = 32768 758 / 727, c3 400 / 389, c5 74.0 / 70.7, one short sentence 17.4 / 16.1. */ \
  dropped = cge == nsel + 1u && nsel != 0u;                                                      \
  if (__ballot(dropped || lacking) != 0ull) {                                                    \
    const uint32_t flip = lacking ? ~0u : 0u, from = lacking ? tau : 0u - tau;                   \
    uint32_t least = 0xffffffffu;                                                                \
    _Pragma("unroll") for (int ct = 0; ct < (NT_); ++ct)                                          \
      _Pragma("unroll") for (int i = 0; i < 4; ++i) least = min(least, (key[ct][i] ^ flip) + from); \
    least = rows_min_u(least);                                                                   \
    tau = dropped ? tau + least + 1u : lacking ? tau - 1u - least : tau;                         \
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
  // Selection: keys >= tau; when more keys than the quota tie at tau (exact duplicates at the
  // boundary), the lowest columns among them win.
  if (nsel == 0u) tau = 0xffffffffu;
  bool tied = __ballot(cge != nsel && nsel != 0u) != 0ull;
  if (!tied) {
#pragma unroll
    for (int j = 0; j < NCT / 2; ++j) sel[j] = mark_at_least(key[2 * j], key[2 * j + 1], tau);
    if (counted || __ballot(dropped || lacking) != 0ull) {  // equals of the key that went went with it, of one that came came with it
      uint32_t cnt = 0;
#pragma unroll
      for (int j = 0; j < NCT / 2; ++j) cnt += __popc(sel[j]);
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
    for (int j = 0; j < NCT / 2; ++j) sel[j] = 0u;
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      asm volatile("" : "+v"(tau), "+v"(need_eq));  // (one tile after the other: side by side they double the kernel's registers)
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
      sel[ct / 2] |= bits << (16 * (ct & 1));
      need_eq -= min(need_eq, static_cast<int32_t>(total));
    }
  }
}

__device__ __forceinline__ uint32_t ordered_key(float a) {
  a += 0.0f;  // -0 -> +0
  uint32_t u = __float_as_uint(a);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ int popc64(uint64_t x) { return __popcll(x); }
__device__ __forceinline__ int lanes_below(uint64_t mask, int lane) {
  return __popcll(mask & ((1ull << lane) - 1ull));
}

// One row per wave, column 64 q + lane in slot q: the largest tau with #{key >= tau} >= n, i.e. the n-th largest key
// (topk_mask_kernel has the same steps in place).
template <int SLOTS>
__device__ __forceinline__ uint32_t nth_largest(const uint32_t (&key)[SLOTS], int n) {
  uint32_t tau = 0;
  int bit = 31;
  {
    // Scores below 2 of which the quota lies at or above 2^-15, as nearly every row of an estimate: bits 31..27 are
    // those of 2^-15.  One count instead of five steps; the scalar unit counts, and the four SIMDs of a CU share it
    // (with the quotients above from the host, lists of B = 4, H = 12, T = 2048, K = 128: 84 -> 72 us).
    int c_ge = 0, c_two = 0;
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) {
      c_ge += popc64(__ballot(key[q] >= 0xb8000000u));
      c_two += popc64(__ballot(key[q] >= 0xc0000000u));
    }
    if (c_two == 0 && c_ge >= n) {
      tau = 0xb8000000u;
      bit = c_ge == n ? -1 : 26;
    }
  }
#pragma unroll 1
  for (; bit >= 0; --bit) {
    const uint32_t trial = tau | (1u << bit);
    int c_ge = 0;
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) c_ge += popc64(__ballot(key[q] >= trial));
    if (c_ge >= n) tau = trial;
    if (c_ge == n) break;  // the keys >= tau are exactly the n to take (one row per wave: uniform)
  }
  return tau;
}

}  // namespace sea
