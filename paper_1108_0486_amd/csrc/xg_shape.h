// Host rules that pick a plain launch's kernel by its sizes.  Free of HIP
// headers: the tests compile them with a host compiler.
#pragma once

#include <stdint.h>

#include "xg.h"

namespace xg {

// Request kinds of the plain launch (the three output types of xg.h plus the
// fused normal-moments reduction).
enum Kind : uint32_t { kU32 = XG_U32, kF32 = XG_F32, kNormal = XG_NORMAL, kMoments = 3, kU64 = XG_U64, kF64 = XG_F64 };

// Whether a stream-major launch (out: its address) takes cached stores instead
// of non-temporal ones.  Cached stores leave dirty lines that a launch writes
// back at its end, which costs a launch of a few MB more than they save; above
// that (times in us, non-temporal and cached):
//  - rows that start inside a 128-byte line: non-temporal stores write both
//    ends of each wavefront's 256 bytes as partial lines (4096 x 65537 uint32:
//    366 and 199; 1024 x 100003: 137 and 80).  Words with a wavefront on every SIMD
//    gain from 20 MB on, 64-bit ones from 30 MB (4096 x 1000 FP32, 16 MB: 5.3 and
//    6.0; 2300 x 2500 uint32, 22 MB: 7.5 and 7.0), with fewer wavefronts from 32 MB.
//    Normals, with more to do for each value, gain from 64 MB, those of the r = 64
//    members from 40 and 80 (2048 x 5001: 12.2 and 13.3; 2000 x 10001: 22.6 and 20.6);
//  - words on whole lines in launches with two wavefronts per SIMD of Section
//    2's member (2048 x 2^15 uint32, 256 MB: 55 and 40; 4096 x 2^18: 805 and 760; one
//    per SIMD, 1024 x 2^20: 705 and 730), one of the 32-bit r = 64 member (2048 x
//    2^19 uint32: 798 and 739), save its longest FP32 rows, whose stores the map
//    spaces (2048 x 2^19: 752 and 771; 2048 x 2^15: 52 and 49), and five for eight
//    SIMDs of the 64-bit one (2000 x 2^17 uint64: 427 and 397; 1024 x 2^17: 181 and
//    185).  Below 64 MB, or 80 where few wavefronts run, non-temporal ones
//    are faster (2048 x 2^11 uint64, 32 MB: 6.9 and 8.3; 2048 x 2^13 uint32,
//    64 MB, of r = 64: 13.7 and 14.6; of Section 2's member: 13.4 and 12.2), and where
//    many more streams wait than run (20000 x 2^13 uint32: 115.5 and 122.3), but for
//    what the last-level cache takes whole (20000 x 2^11: 31.1 and 27.5).
inline bool cached_stores(uint32_t family, Kind kind, uint64_t count, uint64_t n, uintptr_t out, int num_cus) {
  if (kind == kMoments) return false;
  const bool paper = family == XG_FAMILY_R128_W32, wide = family == XG_FAMILY_R64_W64;
  const uint64_t cus = num_cus > 0 ? (uint64_t)num_cus : 1;
  const uint64_t every_simd = (paper ? 4 : 8) * cus;  // streams that give every SIMD a wavefront
  const uint64_t row = n * (wide ? 8 : 4), mb = (count * row) >> 20;
  const bool lines = (row | out) % 128 == 0;
  if (kind == kNormal) return !lines && mb >= (paper ? 64u : wide ? 80u : 40u);
  if (!lines) return mb >= (count < every_simd ? 32u : wide ? 30u : 20u);
  if (count < (paper ? 8 : wide ? 5 : 8) * cus) return false;
  if (count == every_simd && kind == kF32 && mb >= 512) return false;
  if (count >= 64 * cus) return mb >= 128 && mb < 192;
  return mb >= (count < (wide ? 1 : 2) * every_simd ? 80u : 64u);
}

}  // namespace xg
