// How the electron launch divides its work, in units of sub-chunks, among its
// workgroups: plain functions of counts.
#pragma once

#include <stdint.h>

namespace hd {

// Fewest units of a range when there are `all`: one while that makes no more
// than kFewRanges, then as many as make that number, up to one for each wave
// of the workgroup (waves beyond have no sub-chunk, and a workgroup sets up and
// flushes in the time of one).  More workgroups wait for each other's counts
// and deposits at the flush.  Per step in us with one, two, four and eight
// units each (FP32): 16,284 electrons 21.1, 21.2, 21.6, 21.9; 51,100: 23.5,
// 22.4, 22.5, 23.1; 99,996: 27.3, 25.0, 24.3, 24.4; 179,100: 30.2, 30.1, 27.5,
// 27.3; 262,044: 30.3, 30.1, 28.6, 27.7.  FP64 prefers four to eight up to the
// last (99,996: 28.4, 26.0, 24.9, 26.4).
constexpr uint32_t kFewRanges = 128;
__host__ __device__ __forceinline__ uint32_t least_length(uint32_t all, uint32_t waves) {
  const uint32_t l = (all + kFewRanges - 1u) / kFewRanges;
  return l < waves ? l : waves;
}

// Length of the ranges of `all` units that makes at most G of them.
__host__ __device__ __forceinline__ uint32_t range_length(uint32_t all, uint32_t G, uint32_t waves) {
  const uint32_t share = (all + G - 1u) / G, least = least_length(all, waves);
  return share > least ? share : least;
}

// The ranges of one discharge of `subs` sub-chunks whose fluid update counts as
// `fluid` more: their number n and length.  The last one updates the fluid; while
// there are workgroups enough it does only that (sub-chunks after the update
// of four species kept a workgroup for 5 us after the others: 250,000 electrons,
// 22.3 us per launch instead of 17.8).
struct Ranges {
  uint32_t n, per;
};
__host__ __device__ __forceinline__ Ranges ranges_of_one(uint32_t subs, uint32_t fluid, uint32_t G,
                                                         uint32_t waves) {
  const uint32_t all = subs + fluid, least = least_length(all, waves);
  const uint32_t few = (subs + least - 1u) / least + 1u;
  if (few <= G) return {few, least};
  const uint32_t per = range_length(all, G, waves);
  return {(all + per - 1u) / per, per};
}

// Workgroups of the launch for D discharges when G fit on the device at once:
// each takes one range, and those that find none end at once.  A few
// discharges can always be divided into G ranges, none much longer than an
// equal share; many need more ranges than G, which start as workgroups end.
__host__ __device__ __forceinline__ uint32_t launch_groups(uint32_t D, uint32_t G) {
  return D == 1u || 8u * D <= G ? G : G + D;
}

// How many ranges of length per make up u units: ceil(u / per), with inv =
// 1 / per.  Up to 2^24 units the product is off by less than one.
__host__ __device__ __forceinline__ uint32_t ranges_in(uint32_t u, uint32_t per, float inv) {
  const uint32_t x = u + per - 1u;
  const uint32_t q = (uint32_t)((float)x * inv);
  const int32_t r = (int32_t)(x - q * per);
  return r < 0 ? q - 1u : (r >= (int32_t)per ? q + 1u : q);
}

// What a range costs beside its units: a workgroup sets up and flushes for
// each.  24 discharges of 396 units on 64 workgroups took 117, 130 and 127 us
// per step in two, three and five rounds of 92, 68 and 34 units; 300 of 68
// units on 512 took 102 us in two rounds of 24 and 107 in one of 68.
constexpr float kRangeUnits = 16.0f;

// Length of the ranges of several discharges of `all` units, `longest` units
// in the largest, `active` discharges that have any: the length that fills G
// workgroups once if that makes no more than G ranges, else the best of some.
// `most` ranges are allowed, at least one per discharge.  length(g) is the length for g ranges in all,
// number(per) how many ranges there are of length per (each discharge's last
// one may be shorter).
//
// k rounds of G ranges cost k times the length or, at most, an equal share and
// one range more, and k set-ups.  The length for k rounds is the smallest of
// those that n, n - active / 2 and n - active ranges would have for which n
// ranges are enough, n = k G or `most`; one range per discharge always is.  k
// starts where every discharge can have a range and grows while an equal
// share and the set-ups cost less than the best so far.
template <class Length, class Number>
__host__ __device__ __forceinline__ uint32_t batch_length(uint32_t all, uint32_t longest,
                                                          uint32_t active, uint32_t G,
                                                          uint32_t most, Length length,
                                                          Number number) {
  if (active <= G) {
    const uint32_t l = length(G);
    if (number(l) <= G) return l;
  }
  const float share = (float)all / (float)G;
  float best = 3e38f;
  uint32_t best_per = longest;
  uint32_t k = (active + G - 1u) / G;
  for (bool more = true; more && share + (float)k * kRangeUnits < best;
       k += k < 4u ? 1u : k / 2u) {
    more = k * G < most;
    const uint32_t n = more ? k * G : most;
    uint32_t per = longest;
    for (uint32_t c = k == 1u ? 1u : 0u; c < 3u; ++c) {
      const uint32_t cut = c * active / 2u;
      if (n <= cut) break;
      const uint32_t l = length(n - cut);
      if (l >= longest) break;
      if (number(l) <= n) {
        // no longer than the largest discharge's ranges need to be
        const uint32_t parts = (longest + l - 1u) / l, even = (longest + parts - 1u) / parts;
        per = even < l && number(even) <= n ? even : l;
        break;
      }
    }
    const float rounds = (float)k * (float)per, spread = share + (float)per;
    const float cost = (rounds < spread ? rounds : spread) + (float)k * kRangeUnits;
    if (cost < best) {
      best = cost;
      best_per = per;
    }
  }
  return best_per;
}

}  // namespace hd
