// Reads lines "q x" or "c x" and prints the node-table quantile -Phi^{-1}(x) or CDF Phi(x).
#include <cstdio>

#define __host__
#define __device__
#define __forceinline__ inline
#include "device_nodes_f64.h"

int main() {
  char w;
  double x;
  while (std::scanf(" %c %lf", &w, &x) == 2)
    std::printf("%.17g\n", w == 'q' ? vecchia::ninv_nodes(vecchia::kNormNodeTable, x)
                                    : vecchia::phi_nodes(vecchia::kNormNodeTable, x));
  return 0;
}
