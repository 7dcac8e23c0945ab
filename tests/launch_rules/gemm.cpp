// Prints gemm_wgrad_tiles_wanted for lines "tile_shape M N K lda ldb dtype" on standard input.
#include <cstdio>

#include "kernels.h"

int main() {
  int shape, m, n, k, lda, ldb, dtype;
  while (std::scanf("%d %d %d %d %d %d %d", &shape, &m, &n, &k, &lda, &ldb, &dtype) == 7)
    std::printf("%d\n", (int)cdp::gemm_wgrad_tiles_wanted(shape, m, n, k, lda, ldb, dtype));
  return 0;
}
