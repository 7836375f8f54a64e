// The rules of xg_shape.h on cases from standard input, one answer a line:
//   stores FAMILY KIND COUNT N OUT   1 where the launch takes cached stores
#include <cstdio>
#include <cstring>

#include "xg_shape.h"

int main() {
  char what[16];
  while (std::scanf("%15s", what) == 1) {
    unsigned long long family, kind, count, n, out;
    if (std::strcmp(what, "stores") != 0 || std::scanf("%llu %llu %llu %llu %llu", &family, &kind, &count, &n, &out) != 5)
      return 1;
    std::printf("%d\n", xg::cached_stores((uint32_t)family, (xg::Kind)kind, count, n, (uintptr_t)out, 256));
  }
  return 0;
}
