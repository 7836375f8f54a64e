// When groups of an r = 64 batch run faster alone in a wavefront than two and
// two.  Free of HIP headers: the tests compile it with a host compiler.
#pragma once

#include <stdint.h>

namespace xg {

// What a trip of the batch loop costs in words of the kind, and the share of the
// second group on a SIMD that the first one there waits for; fitted to tables of
// 100 to 2000 groups of one to four requests, equal, nearly equal, uniform and
// log-uniform, of 2^6 to 2^17 words, each timed in pairs and alone.
struct PairCost {
  float trip, second;
};
constexpr PairCost pair_cost(bool wide, bool normals) {
  return !wide ? (normals ? PairCost{1300.0f, 0.55f} : PairCost{1900.0f, 0.3f})
               : (normals ? PairCost{575.0f, 0.8f} : PairCost{1250.0f, 0.15f});
}

// Whether groups of different lengths are faster alone.  The halves of a
// wavefront part where either's request ends, which costs a trip a request;
// alone, groups take from each other: where more run than SIMDs, a share of
// the words of the groups that come second there (second: their mean, or 0), and
// a little of the memory's time before (first: words of the largest group).
// Plan and batch in us, pairs and alone: 1000 single uint32 requests of 2^6 to 2^12
// words 29.3 and 27.9, of 60000 to 65536 words 111 and 114; 2000 such streams'
// normals 191 and 249, FP64 normals 316 and 528, of 2^6 to 2^12 words 51.2 and 49.5.
constexpr bool lone_groups_pay(bool wide, bool normals, uint32_t requests, float first, float second) {
  const PairCost cost = pair_cost(wide, normals);
  return (float)requests * cost.trip > second * cost.second + first * (1.0f / 32.0f);
}

}  // namespace xg
