// The search for a row's selection threshold: which key to count at next, from the counts so far.  Nothing but arithmetic, so
// that the steps it takes can be counted on any machine.
//
// A row keeps `lo` with a keys more than its quota at or above it and `hi` with b keys fewer (b + 1/4 while hi is only known
// from above, by search_top).  Keys are the high halves 0x8000 .. 0xc000 of the negated scores' bit patterns, a logarithmic
// scale, on which a row's scores are spread evenly enough for the next trial to come from a and b: 0.15 to 0.85 of the way,
// and no further than the reach, since most of the way down to zero holds no scores.  Scores that are not spread so (most of
// a row far below its largest, or zero) would be walked down to in steps of a few octaves, so the reach, eight octaves at
// first, doubles with every step, and from the ninth step on the range is halved: 8 + 14 steps at most.
//
// Steps for the slowest of 16 rows (simulated on one to three heads), bit by bit, as far as the quota or one key more / so: c4 9.2 / 5.1, c3
// (k^ = 64) 10.1 / 5.6, c2 6.4 / 3.3; queries and keys of twice c3's size 8.9 / 6.5, of three times 8.5 / 8.1; a tenth of the
// columns sixty octaves above the rest 8.6 / 8.0, most scores zero 11.5 / 12.8, all but twenty 15 / 19.  (With a reach of
// eight octaves throughout and no halving: 4.9, 5.6, 3.0, 10.8, 27, 25, 36, 68.  The layer of c3 at three times the size: 481 us
// bit by bit, 595 with that reach, 462 so; at its own size 396 / 377 / 377.)
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>

namespace sea {

struct RowSearch {
  float lo, hi, a, b;

  // done with the quota, one key more or one fewer, or between neighbours
  __host__ __device__ __forceinline__ bool pending() const { return a > 1.f && b != 1.f && hi - lo > 1.f; }

  // the key of step 0, 1, ..; per_key = 1 / (a + b), whose last bits do not matter
  __host__ __device__ __forceinline__ float trial(int32_t step, float per_key) const {
    // (whole numbers, which the wave's scalar unit keeps: numbers of one sign have the order of their bit patterns)
    const float range = hi - lo;
    const int32_t reach = (137 + step) << 23;              // 1024 2^step
    const int32_t weight_bits = step < 8 ? 0x3f333333 : 0;  // 0.7
    int32_t way_bits;
    float way, weight;
    memcpy(&way_bits, &range, sizeof(way_bits));
    way_bits = way_bits < reach ? way_bits : reach;
    memcpy(&way, &way_bits, sizeof(way));
    memcpy(&weight, &weight_bits, sizeof(weight));
    const float part = fmaf(fmaf(b, per_key, -0.5f), weight, 0.5f);
    return truncf(fmaxf(fmaf(-part, way, hi), lo + 1.f));
  }

  // d: keys at or above the trial less the quota
  __host__ __device__ __forceinline__ void counted(float trial, float d) {
    const bool enough = d >= 0.f;
    lo = enough ? trial : lo;
    hi = enough ? hi : trial;
    a = enough ? d : a;
    b = enough ? b : -d;
  }
};

}  // namespace sea
