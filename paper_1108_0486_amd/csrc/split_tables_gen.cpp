// Writes the jump polynomials of xg_split.h as the initialisers of one array
// per member (run by build.py; the library's own jump code computes them).
//
//   split_tables_gen OUTPUT
#include <cstdio>
#include <vector>

#include "xg_host.h"
#include "xg_split.h"

int main(int argc, char **argv) {
  if (argc != 2) return 2;
  FILE *f = std::fopen(argv[1], "w");
  if (!f) return 1;
  for (uint32_t family = 0; family < 3; ++family) {
    const uint32_t words = (uint32_t)xg::member_degree(family) / 64;
    std::vector<uint64_t> all((size_t)xg::kSplitEntries * words), level;
    for (uint32_t e = xg::kSplitMinExp; e <= xg::kSplitTopExp; ++e) {
      const uint32_t count = 2 * xg::split_odds(e) - 1;  // k = 1 .. the largest odd multiple
      level.resize((size_t)count * words);
      if (!xg::jump_table(family, 1ull << e, count, level.data())) return 1;
      for (uint32_t k = 1; k <= count; k += 2)
        for (uint32_t w = 0; w < words; ++w)
          all[(size_t)xg::split_entry(e, k) * words + w] = level[(size_t)(k - 1) * words + w];
    }
    std::fprintf(f, "#ifdef XG_SPLIT_FAMILY_%u\n", family);
    for (size_t i = 0; i < all.size(); ++i) std::fprintf(f, "0x%llxull,%s", (unsigned long long)all[i], i % 4 == 3 ? "\n" : "");
    std::fprintf(f, "#endif\n");
  }
  return std::fclose(f) == 0 ? 0 : 1;
}
