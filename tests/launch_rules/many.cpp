// launch_conv_dl for several bf16 products in one launch, as a function for ctypes.
#include <cstring>

#include "kernels.h"

extern "C" int many(int n, const int* mnk, void* const* a_b_out, int tile, void* stream) {
  static cdp::GemmBatch b;
  std::memset(&b, 0, sizeof(b));
  if (n > cdp::GEMM_MAX_PROBS) return -1;
  b.n = n;
  for (int i = 0; i < n; ++i) {
    cdp::GemmProb& p = b.p[i];
    p.M = mnk[3 * i]; p.N = mnk[3 * i + 1]; p.K = mnk[3 * i + 2];
    p.A = a_b_out[3 * i]; p.B = a_b_out[3 * i + 1]; p.out = a_b_out[3 * i + 2];
    p.a_mode = p.b_mode = cdp::OP_PLAIN_K;
    p.lda = p.ldb = p.K; p.ldo = p.N;
    p.epi = cdp::EPI_FWD;
  }
  return (int)cdp::launch_conv_dl(b, cdp::DT_BF16, tile, static_cast<hipStream_t>(stream));
}
