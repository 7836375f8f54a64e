// The jump polynomials of split launches (xg_split.h), one constant array per
// member in the library's device code; build.py writes their initialisers.
#include <hip/hip_runtime.h>

#include <mutex>

#include "xg.h"
#include "xg_internal.h"
#include "xg_split.h"

namespace {

// Not const: host code that takes the address of a constant device variable
// gets a host copy of it, which hipGetSymbolAddress does not know.
__device__ uint64_t r128_w32[xg::kSplitEntries * 64] = {
#define XG_SPLIT_FAMILY_0
#include "xg_split_tables.inc"
#undef XG_SPLIT_FAMILY_0
};
__device__ uint64_t r64_w32[xg::kSplitEntries * 32] = {
#define XG_SPLIT_FAMILY_1
#include "xg_split_tables.inc"
#undef XG_SPLIT_FAMILY_1
};
__device__ uint64_t r64_w64[xg::kSplitEntries * 64] = {
#define XG_SPLIT_FAMILY_2
#include "xg_split_tables.inc"
#undef XG_SPLIT_FAMILY_2
};

constexpr int kMaxDevices = 64;
std::once_flag g_once[kMaxDevices];
const uint64_t *g_table[kMaxDevices][3];

}  // namespace

namespace xg {

const uint64_t *split_table(uint32_t family, int dev) {
  if (dev < 0 || dev >= kMaxDevices || family >= 3) return nullptr;
  std::call_once(g_once[dev], [dev] {
    auto find = [](const auto &symbol) -> const uint64_t * {
      void *p = nullptr;
      return hipGetSymbolAddress(&p, symbol) == hipSuccess ? static_cast<const uint64_t *>(p) : nullptr;
    };
    g_table[dev][XG_FAMILY_R128_W32] = find(r128_w32);
    g_table[dev][XG_FAMILY_R64_W32] = find(r64_w32);
    g_table[dev][XG_FAMILY_R64_W64] = find(r64_w64);
  });
  return g_table[dev][family];
}

}  // namespace xg
