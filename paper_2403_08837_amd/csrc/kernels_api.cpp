// C ABI of the kernel-level entry points (include/cdp_kernels.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstring>

#include "../../include/cdp.h"
#include "../../include/cdp_kernels.h"
#include "kernels.h"

using namespace cdp;

// Both operands run along the output (a weight gradient): the weight-gradient tiles of the Linear launch read them as they lie and
// transpose on the way out of LDS, where the generic kernel scatters 2- or 4-byte elements into LDS.  Against the generic kernel's
// best tile over outputs of 64 x 64 to 4096 x 4096, 8 to 4096 rows: fp32 64 x 64 x 8 13 -> 7 us, bf16 4096 x 4096 x 64 52 -> 16 us,
// 4096^3 1124 -> 271 us.  Not so in fp32 for large results on the generic kernel's 128 x 128 tile, where what counts is how the result
// leaves: if rows of an operand are not whole 16-byte chunks (us, generic / these: 4001 x 3003 x 16 29 / 40, x 64 55 / 50, x 2000 830 / 945), and for
// up to one slab of 16 if rows of the result are not whole 128-byte lines (4672 x 2320 x 16 24 / 28, x 17 35 / 28, 4096 x 4096 x 8 40 / 30).  At
// 512 tiles of 64 x 128 these are 1.5 times as fast, at 1025 they are not.
bool cdp::gemm_wgrad_tiles_wanted(int tile_shape, int M, int N, int K, int lda, int ldb, int dtype) {
  if (dtype != DT_F32 || tile_shape != TILE_128x128) return true;
  if ((int64_t)((M + 63) / 64) * ((N + 127) / 128) < 768) return true;
  const bool whole = M % 4 == 0 && N % 4 == 0 && lda % 4 == 0 && ldb % 4 == 0;
  return whole && (K > 16 || N % 32 == 0);
}

static_assert((int64_t)CDP_CONV_SHARE_BYTES == CONV_SPLIT_WS_BYTES + CONV_SPLIT_SLOTS * 4, "partial tiles, then counters");

extern "C" {

int cdp_k_gemm(int dtype, int tile_shape, int a_kmajor, int b_kmajor, const void* A, const void* B, float* C, int M, int N,
               int K, int lda, int ldb, void* stream) {
  // tile shapes: 0 .. 2 generic kernel, 3, 4 tick launch with 64 / 128 columns, 5 fastest, 6 tick launch as the engine makes it, 7 .. 9 generic
  // kernel in every layout
  constexpr int FASTEST = TILE_COUNT + 2, AS_ENGINE = TILE_COUNT + 3, GENERIC = TILE_COUNT + 4;
  if (!A || !B || !C || M <= 0 || N <= 0 || K <= 0 || tile_shape < 0 || tile_shape >= GENERIC + TILE_COUNT) return CDP_EINVAL;
  if (tile_shape >= TILE_COUNT && tile_shape < GENERIC && !(a_kmajor && b_kmajor)) return CDP_EINVAL;
  if (dtype != DT_F32 && dtype != DT_BF16) return CDP_EINVAL;
  GemmBatch b;
  memset(&b, 0, sizeof(b));
  b.n = 1;
  GemmProb& p = b.p[0];
  p.A = A; p.B = B; p.out = C;
  p.M = M; p.N = N; p.K = K; p.lda = lda; p.ldb = ldb; p.ldo = N;
  p.a_mode = a_kmajor ? OP_PLAIN_K : OP_PLAIN_R;
  p.b_mode = b_kmajor ? OP_PLAIN_K : OP_PLAIN_R;
  p.epi = EPI_FWD;
  p.flags = GF_OUT_F32;
  p.splits = 1;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipError_t e;
  if (tile_shape >= GENERIC) {
    e = launch_gemm_batch(b, dtype, tile_shape - GENERIC, st);
  } else if (!a_kmajor && !b_kmajor && gemm_wgrad_tiles_wanted(tile_shape, M, N, K, lda, ldb, dtype)) {
    p.epi = EPI_WGRAD;
    p.flags = 0;
    e = launch_linear_tick(b, dtype, false, false, st);
  } else if (tile_shape == FASTEST && gemm_stream_wanted(A, B, M, N, K, lda, ldb, dtype)) {
    e = launch_gemm_stream(A, B, C, M, N, K, lda, ldb, dtype, st);
  } else if (tile_shape >= TILE_COUNT) {
    e = launch_linear_tick(b, dtype, tile_shape == TILE_COUNT + 1, tile_shape == FASTEST || tile_shape == AS_ENGINE, st);
  } else {
    e = launch_gemm_batch(b, dtype, tile_shape, st);
  }
  return e == hipSuccess ? CDP_OK : CDP_EHIP;
}

int cdp_k_conv(int dtype, int which, const void* in0, const void* in1, void* out, int B, int H, int W, int Cin, int Cout,
               int ks, int stride, int pad, void* workspace, size_t workspace_bytes, void* stream) {
  if (!in0 || !in1 || !out || B <= 0 || H <= 0 || W <= 0 || Cin <= 0 || Cout <= 0 || ks <= 0 || stride <= 0 || pad < 0)
    return CDP_EINVAL;
  if (dtype != DT_F32 && dtype != DT_BF16) return CDP_EINVAL;
  if (H + 2 * pad < ks || W + 2 * pad < ks) return CDP_EINVAL;
  const int Ho = (H + 2 * pad - ks) / stride + 1, Wo = (W + 2 * pad - ks) / stride + 1;
  GemmBatch b;
  memset(&b, 0, sizeof(b));
  b.n = 1;
  GemmProb& p = b.p[0];
  p.splits = 1;
  p.A = in0; p.B = in1; p.out = out;
  ConvGeom& g = p.g;
  g.KH = ks; g.KW = ks; g.stride = stride; g.pad = pad;
  const bool force256 = which >= 3 && which <= 6;  // the direct-to-LDS tile regardless of the launch heuristic
  const int forced_tile = which >= 5 ? DL_256x128 : DL_256x256;
  const bool shared = which == 7 || which == 8, accumulate = which == 9, gelu = which == 10 || which == 11;
  if (force256) which -= which >= 5 ? 5 : 3;
  if (shared) which -= 7;
  if (accumulate) which = 2;
  if (gelu) which -= 10;
  if (which == 0) {
    p.M = B * Ho * Wo; p.N = Cout; p.K = ks * ks * Cin;
    p.a_mode = OP_CONV_FWD; p.b_mode = OP_PLAIN_K; p.ldb = p.K; p.ldo = Cout;
    g.H = H; g.W = W; g.C = Cin; g.OH = Ho; g.OW = Wo;
    p.epi = EPI_FWD;
  } else if (which == 1) {
    p.M = B * H * W; p.N = Cin; p.K = ks * ks * Cout;
    p.a_mode = OP_CONV_DGRAD; p.b_mode = OP_PLAIN_K; p.ldb = p.K; p.ldo = Cin;
    g.H = Ho; g.W = Wo; g.C = Cout; g.OH = H; g.OW = W;
    p.epi = EPI_DGRAD;
  } else if (which == 2) {
    p.M = Cout; p.N = ks * ks * Cin; p.K = B * Ho * Wo;
    p.a_mode = OP_PLAIN_R; p.lda = Cout; p.b_mode = OP_CONV_WGRAD; p.ldo = p.N;
    g.H = H; g.W = W; g.C = Cin; g.OH = Ho; g.OW = Wo;
    p.epi = EPI_WGRAD;
  } else {
    return CDP_EINVAL;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (shared && (!conv_fast_eligible(p, dtype) || !workspace || workspace_bytes < (size_t)CDP_CONV_SHARE_BYTES)) return CDP_EINVAL;
  if (gelu) {
    if (dtype != DT_BF16 || p.N <= 64 || !conv_fast_eligible(p, dtype) || !workspace || workspace_bytes / 2 < (size_t)p.M * p.N) return CDP_EINVAL;
    if (which == 0) p.aux2 = workspace;
    else p.aux1 = workspace;
    p.flags |= GF_GELU;
    if (!conv_gelu_valid(b, dtype)) return CDP_EINVAL;
  }
  // the fast implicit-GEMM paths where the shape allows, as in the engine; what is different for a call on its own: no workspace to share
  // reductions in (which = 7, 8 have one), ranges of the weight gradient for a launch of its own, and a fold that overwrites
  if (which == 2) {
    const size_t range_bytes = (size_t)p.M * p.N * 4;
    const int room = (int)std::min<size_t>(INT_MAX, workspace ? workspace_bytes / range_bytes : 0);
    if (conv_fast_eligible(p, dtype) && room >= 1) {
      const int splits = conv_wgrad_splits_alone(p, dtype, room);
      // two phases: partial sums per reduction range, then the fold
      WReduceBatch rb;
      memset(&rb, 0, sizeof(rb));
      rb.n = 1;
      rb.p[0].part = static_cast<const float*>(workspace);
      rb.p[0].G = static_cast<float*>(out);
      rb.p[0].Cout = p.M; rb.p[0].Ncol = p.N; rb.p[0].splits = splits;
      rb.p[0].overwrite = !accumulate;
      p.out = workspace;
      p.splits = splits;
      if (launch_conv_wgrad(b, dtype, p.M >= 128, st) != hipSuccess) return CDP_EHIP;
      return launch_wgrad_reduce(rb, dtype, st) == hipSuccess ? CDP_OK : CDP_EHIP;
    }
    if (accumulate) return CDP_EINVAL;
  } else if (force256) {
    if (!conv_gemm256_eligible(p, dtype)) return CDP_EINVAL;
    return launch_conv_dl(b, dtype, forced_tile, st) == hipSuccess ? CDP_OK : CDP_EHIP;
  } else if (conv_fast_eligible(p, dtype)) {
    if (shared) {
      b.thin_ws = static_cast<float*>(workspace);
      b.thin_cnt = reinterpret_cast<unsigned int*>(static_cast<char*>(workspace) + CONV_SPLIT_WS_BYTES);
    }
    if (conv_gemm256_wanted(&p, 1, dtype)) return launch_conv_dl(b, dtype, DL_256x256, st) == hipSuccess ? CDP_OK : CDP_EHIP;
    int bm, bn;
    conv_gemm_tile(&p, 1, &bm, &bn);
    return launch_conv_gemm(b, dtype, bm, bn, st) == hipSuccess ? CDP_OK : CDP_EHIP;
  }
  const int shape = p.M <= 64 ? (p.N >= 128 ? TILE_64x128 : TILE_64x64) : (p.N <= 64 ? TILE_64x64 : TILE_128x128);
  return launch_gemm_batch(b, dtype, shape, st) == hipSuccess ? CDP_OK : CDP_EHIP;
}

int cdp_k_layernorm(int dtype, int backward, const void* x, const void* dy, const void* add, const float* gamma,
                    const float* beta, void* out, float* dgamma, float* dbeta, void* workspace, size_t workspace_bytes,
                    int rows, int C, void* stream) {
  if (!x || !gamma || !out || rows <= 0 || C <= 0 || C > 1024 || (dtype != DT_F32 && dtype != DT_BF16)) return CDP_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (!backward) {
    if (!beta) return CDP_EINVAL;
    return launch_layernorm_fwd(x, gamma, beta, out, rows, C, dtype, st) == hipSuccess ? CDP_OK : CDP_EHIP;
  }
  if (!dy || !dgamma || !dbeta || !workspace || (int64_t)workspace_bytes < layernorm_bwd_workspace_bytes(rows, C)) return CDP_EINVAL;
  return launch_layernorm_bwd(x, dy, add, gamma, out, dgamma, dbeta, static_cast<float*>(workspace), rows, C, dtype, st) == hipSuccess
             ? CDP_OK : CDP_EHIP;
}

int cdp_k_gelu(int dtype, int backward, const void* x, const void* dy, void* out, int64_t n, void* stream) {
  if (!x || !out || n <= 0 || (backward && !dy) || (dtype != DT_F32 && dtype != DT_BF16)) return CDP_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const hipError_t e = backward ? launch_gelu_bwd(x, dy, out, n, dtype, st) : launch_gelu_fwd(x, out, n, dtype, st);
  return e == hipSuccess ? CDP_OK : CDP_EHIP;
}

int cdp_k_attention(int dtype, int backward, const void* qkv, void* P, const void* dout, void* out, void* workspace,
                    size_t workspace_bytes, int B, int T, int D, int heads, void* stream) {
  if (!qkv || !P || !out || !workspace || B <= 0 || T <= 0 || T > 1024 || D <= 0 || heads <= 0 || D % heads ||
      (dtype != DT_F32 && dtype != DT_BF16))
    return CDP_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t tt = (int64_t)B * heads * T * T;
  if (!backward) {
    if ((int64_t)workspace_bytes < 4 * tt) return CDP_EINVAL;
    return launch_attention_fwd(qkv, P, out, static_cast<float*>(workspace), B, T, D, heads, dtype, st) == hipSuccess ? CDP_OK : CDP_EHIP;
  }
  const int64_t dp_bytes = (4 * tt + 255) / 256 * 256;
  if (!dout || (int64_t)workspace_bytes < dp_bytes + tt * (dtype == DT_BF16 ? 2 : 4)) return CDP_EINVAL;
  return launch_attention_bwd(qkv, P, dout, out, static_cast<float*>(workspace), static_cast<char*>(workspace) + dp_bytes, B, T, D,
                              heads, dtype, st) == hipSuccess ? CDP_OK : CDP_EHIP;
}

}  // extern "C"
