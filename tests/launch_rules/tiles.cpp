// Prints conv_dl_tile for launches of one bf16 problem given as lines "M N K shared" on standard input.
#include <cstdio>
#include <cstring>

#include "kernels.h"

int main() {
  int m, n, k, shared;
  while (std::scanf("%d %d %d %d", &m, &n, &k, &shared) == 4) {
    cdp::GemmProb p;
    std::memset(&p, 0, sizeof(p));
    p.M = m; p.N = n; p.K = k;
    p.a_mode = p.b_mode = cdp::OP_PLAIN_K;
    p.lda = p.ldb = k; p.ldo = n;
    p.epi = cdp::EPI_FWD;
    std::printf("%d\n", cdp::conv_dl_tile(&p, 1, cdp::DT_BF16, shared != 0));
  }
  return 0;
}
