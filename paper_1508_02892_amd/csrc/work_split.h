// How the electron launch divides its work, in units of sub-chunks, among its
// workgroups: plain functions of counts.
#pragma once

#include <stdint.h>

namespace hd {

// Length of the ranges of `all` units on G workgroups: one each while there
// are workgroups enough, else at least one per wave (a workgroup sets up and
// flushes in the time of one sub-chunk and works on as many as it has waves
// at once).  Launches of 64 sub-chunks (16,384 electrons) take 13.0 us with
// one each and 16.2 with eight; of 1,192 on 512 workgroups (305,043 electrons,
// 1,471 cells) 19.3 with three each and 16.8 with eight.
__host__ __device__ __forceinline__ uint32_t range_length(uint32_t all, uint32_t G, uint32_t waves) {
  const uint32_t share = (all + G - 1u) / G;
  return all <= G ? 1u : (share > waves ? share : waves);
}

// What a range costs beside its units: a workgroup sets up and flushes for
// each.  24 discharges of 396 units on 64 workgroups took 117, 130 and 127 us
// per step in two, three and five rounds of 92, 68 and 34 units; 300 of 68
// units on 512 took 102 us in two rounds of 24 and 107 in one of 68.
constexpr float kRangeUnits = 16.0f;

// Length of the ranges of several discharges of `all` units, `longest` units
// in the largest, `active` discharges that have any, when ranges of the length
// that fills G workgroups once are more than G.  length(g) is the length for g
// ranges in all, number(per) how many ranges there are of length per (each
// discharge's last one may be shorter).
//
// k rounds of ranges, each workgroup taking every G-th, cost k times the
// length or, at most, an equal share and one range more, and k set-ups.  The
// length for k rounds is the smallest of those that k G, k G - active / 2 and
// k G - active ranges would have for which k G ranges are enough; one range
// per discharge always is.  k starts where every discharge can have a range
// and grows, to most_rounds at most, while an equal share and the set-ups cost
// less than the best so far.
template <class Length, class Number>
__host__ __device__ __forceinline__ uint32_t batch_length(uint32_t all, uint32_t longest,
                                                          uint32_t active, uint32_t G,
                                                          uint32_t most_rounds, Length length,
                                                          Number number) {
  const float share = (float)all / (float)G;
  float best = 3e38f;
  uint32_t best_per = longest;
  for (uint32_t k = (active + G - 1u) / G;
       k <= most_rounds && share + (float)k * kRangeUnits < best; k += k < 4u ? 1u : k / 2u) {
    const uint32_t slots = k * G;
    uint32_t per = longest;
    for (uint32_t c = k == 1u ? 1u : 0u; c < 3u; ++c) {
      const uint32_t cut = c * active / 2u;
      if (slots <= cut) break;
      const uint32_t l = length(slots - cut);
      if (l >= longest) break;
      if (number(l) <= slots) {
        per = l;
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
