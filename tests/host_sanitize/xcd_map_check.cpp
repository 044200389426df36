// Reads grid sizes n from standard input and prints, for each, the slots of blocks 0..n-1 on a line.
#define __host__
#define __device__
#define __forceinline__ inline
#include <cstdio>

#include "xcd_map.h"

int main() {
  unsigned n;
  while (std::scanf("%u", &n) == 1) {
    for (unsigned b = 0; b < n; ++b) std::printf("%u ", vecchia::xcd_slot(b, n));
    std::printf("\n");
  }
  return 0;
}
