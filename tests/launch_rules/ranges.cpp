// Prints conv_wgrad_splits_alone for problems given as lines "dtype M N K room" on standard input.
#include <cstdio>
#include <cstring>

#include "kernels.h"

int main() {
  int dtype, m, n, k, room;
  while (std::scanf("%d %d %d %d %d", &dtype, &m, &n, &k, &room) == 5) {
    cdp::GemmProb p;
    std::memset(&p, 0, sizeof(p));
    p.M = m; p.N = n; p.K = k;
    std::printf("%d\n", cdp::conv_wgrad_splits_alone(p, dtype, room));
  }
  return 0;
}
