// lone_groups_pay (xg_pairs.h) on cases from standard input, one answer a line:
//   WIDE NORMALS REQUESTS FIRST SECOND
#include <cstdio>

#include "xg_pairs.h"

int main() {
  int wide, normals;
  unsigned requests;
  float first, second;
  while (std::scanf("%d %d %u %f %f", &wide, &normals, &requests, &first, &second) == 5)
    std::printf("%d\n", xg::lone_groups_pay(wide, normals, requests, first, second));
  return 0;
}
