// Prints conv_wgrad_small_wanted for launches of one problem given as lines "dtype M N K ranges misaligned" on standard input.
#include <cstdio>
#include <cstring>

#include "kernels.h"

int main() {
  int dtype, m, n, k, ranges, misaligned;
  while (std::scanf("%d %d %d %d %d %d", &dtype, &m, &n, &k, &ranges, &misaligned) == 6) {
    static cdp::GemmBatch b;
    std::memset(&b, 0, sizeof(b));
    b.n = 1;
    b.p[0].M = m; b.p[0].N = n; b.p[0].K = k; b.p[0].splits = ranges;
    b.p[0].A = reinterpret_cast<const void*>((uintptr_t)(256 + 8 * misaligned));
    std::printf("%d\n", (int)cdp::conv_wgrad_small_wanted(b, dtype));
  }
  return 0;
}
