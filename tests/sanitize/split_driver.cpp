// Split launches' host rules (xg_split.h): every plan covers its row with
// parts that can hold a start state, every distance has an entry of its own,
// and the entries written at build time are the library's jump polynomials.
#include <cstdio>
#include <cstring>
#include <vector>

#include "xg_host.h"
#include "xg_split.h"

static const uint64_t table0[] = {
#define XG_SPLIT_FAMILY_0
#include "xg_split_tables.inc"
#undef XG_SPLIT_FAMILY_0
};
static const uint64_t table1[] = {
#define XG_SPLIT_FAMILY_1
#include "xg_split_tables.inc"
#undef XG_SPLIT_FAMILY_1
};
static const uint64_t table2[] = {
#define XG_SPLIT_FAMILY_2
#include "xg_split_tables.inc"
#undef XG_SPLIT_FAMILY_2
};

#define CHECK(c) \
  do { if (!(c)) { std::printf("FAIL %s line %d\n", #c, __LINE__); return 1; } } while (0)

int main() {
  using namespace xg;
  std::vector<uint64_t> sizes;
  for (int e = 0; e < 40; ++e)
    for (int d = -2; d <= 258; d += (d < 2 || d > 253) ? 1 : 251)
      if ((int64_t)(1ull << e) + d > 0) sizes.push_back((1ull << e) + d);
  for (uint64_t k = 1; k < 300; ++k) sizes.push_back(k * 4096 + 255), sizes.push_back(k * 4096 + 256);
  uint64_t split = 0;
  for (uint64_t waves : {1, 2, 3, 5, 24, 100, 255, 256, 257, 511, 512, 513, 1024, 100000})
    for (uint64_t n : sizes)
      for (int kind = 0; kind < 6; ++kind) {
        const Split s = plan_split(waves, n, 256, kSplitCost[kind / 2][kind % 2]);
        if (!s.parts) continue;
        ++split;
        CHECK(s.parts > 1 && s.parts <= kSplitMaxParts && s.parts * waves <= 1024);
        CHECK(s.exp >= kSplitMinExp && s.exp <= kSplitMaxExp);
        const uint64_t done = (uint64_t)(s.parts - 1) << s.exp;
        CHECK(n > done && n - done >= kSplitMinPart && n - done < (1ull << s.exp) + kSplitMinPart);
      }
  CHECK(split > 1000);
  CHECK(plan_split(0, 1 << 20, 256, kSplitCost[0][0]).parts == 0);

  std::vector<int> seen(kSplitEntries, 0);
  for (uint32_t e = kSplitMinExp; e <= kSplitMaxExp; ++e)
    for (uint32_t k = 1; k < kSplitMaxParts; ++k) {
      CHECK(split_entry(e, k) < kSplitEntries);
      if (k & 1) ++seen[split_entry(e, k)];
      else CHECK(e == kSplitMaxExp || split_entry(e, k) == split_entry(e + 1, k / 2));
    }
  for (uint32_t e = kSplitMaxExp + 1; e <= kSplitTopExp; ++e)
    for (uint32_t k = 1; k < 2 * split_odds(e); k += 2) ++seen[split_entry(e, k)];
  for (int v : seen) CHECK(v == 1);

  const uint64_t *tables[3] = {table0, table1, table2};
  const size_t sizes_of[3] = {sizeof table0, sizeof table1, sizeof table2};
  for (uint32_t f = 0; f < 3; ++f) {
    const size_t words = (size_t)member_degree(f) / 64;
    CHECK(sizes_of[f] == kSplitEntries * words * 8);
    std::vector<uint64_t> g(words);
    for (uint32_t e : {11u, 12u, 16u, 20u})
      for (uint32_t k : {1u, 2u, 3u, 40u, 97u, 128u, 254u, 255u}) {
        CHECK(jump_polynomial_uncached(f, (uint64_t)k << e, g.data()));
        CHECK(!std::memcmp(g.data(), tables[f] + split_entry(e, k) * words, words * 8));
      }
  }
  std::printf("OK\n");
  return 0;
}
