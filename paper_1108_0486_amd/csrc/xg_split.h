// Rows cut into parts (plain launches with few streams): the distances whose
// jump polynomials are built into the library, and the rule that picks a
// launch's parts.  Free of HIP headers: the program that writes the
// polynomials at build time includes it too.
//
// A launch of few streams leaves most of the chip idle, since a stream's
// recurrence runs on one wavefront.  Such a launch cuts each stream's row of n
// values into `parts` parts of 2^exp values (the last one takes the rest),
// finds each part's start state by jump-ahead, and runs every part on a
// wavefront of its own; the values are the same.  The start states wait in
// the output, in the words that their parts overwrite afterwards, so the call
// needs no memory of its own.
#pragma once

#include <stdint.h>

namespace xg {

constexpr uint32_t kSplitMinExp = 11, kSplitMaxExp = 20;
constexpr uint32_t kSplitMaxParts = 256;
// Every part has at least this many values, so its start state (at most three
// steps' worth of words) fits in its own full steps, ahead of any ragged tail.
constexpr uint32_t kSplitMinPart = 256;

// Polynomials z^D mod P are kept for D = k 2^e, k < kSplitMaxParts, e in
// kSplitMinExp .. kSplitMaxExp; with k = o 2^t (o odd) D is o 2^(e + t), so
// only odd multiples are stored, by exponent: 128 up to kSplitMaxExp, then
// half as many for each further one.
constexpr uint32_t kSplitOdds = kSplitMaxParts / 2;
constexpr uint32_t kSplitTopExp = kSplitMaxExp + 7;
constexpr uint32_t split_odds(uint32_t e) { return e <= kSplitMaxExp ? kSplitOdds : kSplitOdds >> (e - kSplitMaxExp); }
constexpr uint32_t split_base(uint32_t e) {
  return e <= kSplitMaxExp ? (e - kSplitMinExp) * kSplitOdds
                           : (kSplitMaxExp - kSplitMinExp + 1) * kSplitOdds + kSplitOdds - (kSplitOdds >> (e - kSplitMaxExp - 1));
}
constexpr uint32_t kSplitEntries = split_base(kSplitTopExp) + split_odds(kSplitTopExp);
// The entry of D = k 2^e, 1 <= k < kSplitMaxParts.
constexpr uint32_t split_entry(uint32_t e, uint32_t k) {
  return (k & 1u) ? split_base(e) + (k >> 1) : split_entry(e + 1, k >> 1);
}

struct Split {
  uint32_t parts = 0;  // 0: the launch is not split
  uint32_t exp = 0;
};

// What a launch's member and kind cost: picoseconds a wavefront takes per value of
// a row, nanoseconds of a round of jumps (a workgroup per compute unit), and
// the bytes of all wavefronts' values with one n (values of a wavefront: one
// per stream, two streams for the r = 64 members).
struct SplitCost {
  uint32_t value_ps, round_ns, value_bytes;
};
constexpr uint64_t kSplitLaunchNs = 3000;  // a plain launch without its values
constexpr uint64_t kSplitBaseNs = 5000;    // the two launches without jumps and values
// What either form writes at best.  (At 5000, long launches on half of the SIMDs
// stayed whole: 512 x 2^20 uint32 486 us and 390 cut in two, FP32 568 and 397;
// 1024 x 2^20 of the 32-bit r = 64 member 1032 and 817, bulk-fill 1085 and 671.
// A saving of a tenth by these costs is not always one: 300 x 40001 normals 40
// us whole and 42.)
constexpr uint64_t kSplitBytesPerNs = 5800;
// Measured (a wavefront alone on its SIMD; 1 to 1024 workgroups).  By member
// (XG_FAMILY_*), then words and normals.
constexpr SplitCost kSplitCost[3][2] = {
    {{470, 3200, 4}, {900, 3200, 4}},
    {{1000, 4500, 8}, {1900, 6000, 8}},
    {{1320, 14000, 16}, {4000, 14000, 16}},
};

// The parts of a launch of `waves` wavefronts (one per stream, or one per two
// streams for the r = 64 members) with n values per stream on `cus` compute
// units: those of the least time by the costs above, with at most one
// wavefront per SIMD; none where that saves less than a fifth, or where more
// than half of the SIMDs have a wavefront as it is.  Nor are rows cut that are too
// long for the stored distances: 256 parts of 2^20 values (and the 255 more
// that a last part may have), or 2^20 for each SIMD where several wavefronts
// share them.  One value more and such a row runs whole, as every row
// did before: one stream x (2^28 + 255) uint32 takes 0.49 ms, one value more 122 ms.
inline Split plan_split(uint64_t waves, uint64_t n, uint64_t cus, const SplitCost &c) {
  Split s;
  const uint64_t slots = 4 * cus;
  if (waves == 0 || n < 2 * kSplitMinPart || 2 * waves > slots || n >> 40) return s;
  const uint64_t write_ns = n * waves * c.value_bytes / kSplitBytesPerNs, whole_ns = n * c.value_ps / 1000;
  uint64_t best = (kSplitLaunchNs + (whole_ns > write_ns ? whole_ns : write_ns)) * 4 / 5;
  for (uint32_t e = kSplitMinExp; e <= kSplitMaxExp; ++e) {
    const uint64_t parts = ((n - kSplitMinPart) >> e) + 1;
    if (parts < 2) break;
    if (parts > kSplitMaxParts || parts * waves > slots) continue;
    const uint64_t last = n - ((parts - 1) << e), longest = last > (1ull << e) ? last : 1ull << e;
    const uint64_t part_ns = longest * c.value_ps / 1000;
    const uint64_t ns = kSplitBaseNs + (parts * waves + cus - 1) / cus * c.round_ns +
                        (part_ns > write_ns ? part_ns : write_ns);
    if (ns < best) {
      best = ns;
      s.parts = (uint32_t)parts;
      s.exp = e;
    }
  }
  return s;
}

}  // namespace xg
