// Prints attention_fused for lines "backward dtype samples tokens width-of-all-heads heads" on standard input.
#include <cstdio>

#include "kernels.h"

int main() {
  int backward, dtype, b, t, d, heads;
  while (std::scanf("%d %d %d %d %d %d", &backward, &dtype, &b, &t, &d, &heads) == 6)
    std::printf("%d\n", (int)cdp::attention_fused(backward != 0, b, t, d, heads, dtype));
  return 0;
}
