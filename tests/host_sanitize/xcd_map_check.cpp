// Reads lines "n even" from standard input and prints, for each, the slots of blocks 0..n-1 on a line.
#define __host__
#define __device__
#define __forceinline__ inline
#include <cstdio>

#include "xcd_map.h"

int main() {
  unsigned n, even;
  while (std::scanf("%u %u", &n, &even) == 2) {
    for (unsigned b = 0; b < n; ++b) std::printf("%u ", vecchia::xcd_slot(b, n, even != 0));
    std::printf("\n");
  }
  return 0;
}
