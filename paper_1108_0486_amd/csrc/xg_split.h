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

// The parts of a launch of `waves` wavefronts (one per stream, or one per two
// streams for the r = 64 members) with n values per stream: the shortest
// parts that give no more than `slots` wavefronts in all.
inline Split plan_split(uint64_t waves, uint64_t n, uint64_t slots, uint64_t min_n) {
  Split s;
  if (waves == 0 || n < min_n || 2 * waves > slots) return s;
  uint64_t want = slots / waves;
  if (want > kSplitMaxParts) want = kSplitMaxParts;
  for (uint32_t e = kSplitMinExp; e <= kSplitMaxExp; ++e) {
    const uint64_t parts = ((n - kSplitMinPart) >> e) + 1;
    if (parts <= want) {
      if (parts > 1) {
        s.parts = (uint32_t)parts;
        s.exp = e;
      }
      return s;
    }
  }
  return s;
}

}  // namespace xg
