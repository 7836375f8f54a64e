// The host rules of plain launches (xg_shape.h, xg_split.h) on 256 compute
// units, on cases from standard input, one answer a line:
//   stores FAMILY KIND COUNT N OUT   1 where the launch takes cached stores
//   split FAMILY KIND COUNT N        PARTS EXP of its rows (0 0: whole)
#include <cstdio>
#include <cstring>

#include "xg_shape.h"
#include "xg_split.h"

int main() {
  char what[16];
  unsigned long long family, kind, count, n, out;
  while (std::scanf("%15s %llu %llu %llu %llu", what, &family, &kind, &count, &n) == 5) {
    if (std::strcmp(what, "stores") == 0) {
      if (std::scanf("%llu", &out) != 1) return 1;
      std::printf("%d\n", xg::cached_stores((uint32_t)family, (xg::Kind)kind, count, n, (uintptr_t)out, 256));
    } else if (std::strcmp(what, "split") == 0) {
      const uint64_t waves = family == XG_FAMILY_R128_W32 ? count : (count + 1) / 2;
      const xg::Split s = xg::plan_split(waves, n, 256, xg::kSplitCost[family][kind == xg::kNormal]);
      std::printf("%u %u\n", s.parts, s.exp);
    } else {
      return 1;
    }
  }
  return 0;
}
