// Prints conv_launch_tile for launches of one bf16 problem given as lines "M N K shared beside" on standard input.  beside: what the
// epilogue reads or does: 0 nothing, 1 residual, 2 mask, 3 addend, 4 accumulates, 5 GELU, 6 the GELU's derivative.
#include <cstdio>
#include <cstring>

#include "kernels.h"

int main() {
  int m, n, k, shared, beside;
  static char tensor[16];
  void* const other = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(tensor) + 15) & ~(uintptr_t)15);
  while (std::scanf("%d %d %d %d %d", &m, &n, &k, &shared, &beside) == 5) {
    cdp::GemmProb p;
    std::memset(&p, 0, sizeof(p));
    p.M = m; p.N = n; p.K = k;
    p.a_mode = p.b_mode = cdp::OP_PLAIN_K;
    p.lda = p.ldb = k; p.ldo = n;
    p.epi = beside == 0 || beside == 1 || beside == 5 ? cdp::EPI_FWD : cdp::EPI_DGRAD;
    if (beside == 1 || beside == 2 || beside == 6) p.aux1 = other;
    if (beside == 3) p.aux0 = other;
    if (beside == 4) p.flags = cdp::GF_ACCUM;
    if (beside == 5) p.aux2 = other;
    if (beside >= 5) p.flags = cdp::GF_GELU;
    std::printf("%d\n", cdp::conv_launch_tile(&p, 1, cdp::DT_BF16, shared != 0));
  }
  return 0;
}
