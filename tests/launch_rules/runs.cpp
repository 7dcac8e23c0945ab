// Prints conv_wgrad_xcd_run for launches of one problem given as lines "M N K ranges" on standard input.
#include <cstdio>
#include <cstring>

#include "kernels.h"

int main() {
  int m, n, k, ranges;
  while (std::scanf("%d %d %d %d", &m, &n, &k, &ranges) == 4) {
    static cdp::GemmBatch b;
    std::memset(&b, 0, sizeof(b));
    b.n = 1;
    b.p[0].M = m; b.p[0].N = n; b.p[0].K = k; b.p[0].splits = ranges;
    const int rows = m >= 128 ? 128 : 64;
    b.total_tiles = ((m + rows - 1) / rows) * ((n + 127) / 128) * ranges;
    std::printf("%d\n", cdp::conv_wgrad_xcd_run(b));
  }
  return 0;
}
