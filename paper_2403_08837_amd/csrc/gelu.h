// Exact GELU and its derivative on values of type T (fp32 arithmetic): the elementwise kernels and the epilogues of the
// convolution kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cdp {

// Phi(v) and phi(v).  fp32 results take the library's erf and exp.  Where the result is rounded to bf16 the two-branch erf
// (lanes of a wavefront take both) makes the kernels arithmetic-bound; there Phi of |v| comes from one exponential that
// the density needs anyway: Phi(-u) = exp(-u^2 / 2) * t * R(t), t = 1 / (1 + 0.3 u), R the polynomial of degree 7 that
// fits erfcx(u / sqrt 2) / (2 t) on 0 <= u <= 14 with the least relative error (1.8e-7, by least squares on Chebyshev
// points).  Error of x Phi(x) and its derivative against 64 bits before the rounding, 2-norms for v ~ N(0, 1.2): 3.7e-8
// and 5.8e-8 (erf and exp: 3.7e-8 and 4.1e-8), after it 1.7e-3 for either.
template <typename T> __device__ __forceinline__ void gauss(float v, float& Phi, float& phi);
template <> __device__ __forceinline__ void gauss<float>(float v, float& Phi, float& phi) {
  Phi = 0.5f * (1.f + erff(v * 0.70710678118654752f));
  phi = 0.3989422804014327f * expf(-0.5f * v * v);
}
template <> __device__ __forceinline__ void gauss<uint16_t>(float v, float& Phi, float& phi) {
  const float u = fabsf(v), t = __builtin_amdgcn_rcpf(fmaf(0.3f, u, 1.f));
  const float e = __builtin_amdgcn_exp2f(-0.72134752044448170f * (v * v));
  float r = 0.03622337058186531f;
  r = fmaf(r, t, -0.1593545526266098f);
  r = fmaf(r, t, 0.20981964468955994f);
  r = fmaf(r, t, -0.05664501339197159f);
  r = fmaf(r, t, 0.13000500202178955f);
  r = fmaf(r, t, 0.09951350837945938f);
  r = fmaf(r, t, 0.12081217765808105f);
  r = fmaf(r, t, 0.11962586641311646f);
  const float q = e * (t * r);
  Phi = v > 0.f ? 1.f - q : q;
  phi = 0.3989422804014327f * e;
}
template <typename T> __device__ __forceinline__ float gelu_f(float v) {
  float Phi, phi;
  gauss<T>(v, Phi, phi);
  return v * Phi;
}
template <typename T> __device__ __forceinline__ float gelu_df(float v) {
  float Phi, phi;
  gauss<T>(v, Phi, phi);
  return Phi + v * phi;
}

}  // namespace cdp
