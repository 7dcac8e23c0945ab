// Element types of the contractions (bf16 as raw 16-bit words, fp32) and the small device helpers
// every kernel file uses: conversions, per-type constants, 16-byte chunks, problem lookup, MFMA call.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.h"

namespace cdp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 v8bf16_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float v16f_t;

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
// round to nearest even, in hardware (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t f32_to_bf16(float f) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f)); }

template <typename T> struct Elem;
template <> struct Elem<uint16_t> {
  static constexpr int VEC = 8;      // elements per 16-byte chunk
  static constexpr int MFMA_K = 16;  // reduction elements per MFMA
  static constexpr int KPL = 8;      // reduction elements per lane per MFMA
  __device__ static __forceinline__ float to_f32(uint16_t v) { return bf16_to_f32(v); }
  __device__ static __forceinline__ uint16_t from_f32(float f) { return f32_to_bf16(f); }
};
template <> struct Elem<float> {
  static constexpr int VEC = 4, MFMA_K = 2, KPL = 1;
  __device__ static __forceinline__ float to_f32(float v) { return v; }
  __device__ static __forceinline__ float from_f32(float f) { return f; }
};

template <typename T> __device__ __forceinline__ float ld_f32(const T* p, int64_t i) { return Elem<T>::to_f32(p[i]); }
template <typename T> __device__ __forceinline__ void st_f32(T* p, int64_t i, float v) { p[i] = Elem<T>::from_f32(v); }

template <typename T> union Chunk16 {
  uint4 v;
  uint2 h[2];
  T e[16 / sizeof(T)];
};

// Problem of a launch of n problems that owns tile number `tile` (problems are listed by ascending tile_begin): compares on
// scalars that one or two wide reads bring in, no loop whose every step waits for a read.  A launch of one problem reads none of them
// (linear_tick_body does: it has the whole table read ahead, in one round with what it needs anyway).
template <int MAX> __device__ __forceinline__ int tile_starts_find(const TileStarts<MAX>& t, int n, int tile) {
  auto past = [&](int at) { return (int)((unsigned)(at - 1 - tile) >> 31); };  // tile >= at, without a trip through the vector unit
  int pi = 0;
  if (n > 1) {
#pragma unroll
    for (int q = 1; q < 8; ++q) pi += past(t.at[q]);
    if (n > 8) {
#pragma unroll
      for (int q = 8; q < MAX; ++q) pi += past(t.at[q]);
    }
  }
  return pi;
}
// A descriptor of the argument block in registers, all of it in one round of scalar reads (the asm takes every part at once, so none
// is put off).  Read field by field where they are used, a descriptor is a read of 300 ns at every place
// the compiler moves one to: a small tile of linear_tick_kernel waits for six of them, of the nine microseconds it takes.
template <typename S> __device__ __forceinline__ S read_args(const S& src) {
  typedef uint32_t w16 __attribute__((ext_vector_type(16), aligned(4)));
  typedef uint32_t w4 __attribute__((ext_vector_type(4), aligned(4)));
  typedef uint32_t w2 __attribute__((ext_vector_type(2), aligned(4)));
  constexpr int N = sizeof(S) / 4;
  static_assert(sizeof(S) % 4 == 0 && (N == 38 || N == 24 || N == 20), "sizes this is written for");
  const uint32_t* const p = reinterpret_cast<const uint32_t*>(&src);
  struct alignas(alignof(S)) Words { uint32_t w[N]; } words;
  w16 a = *reinterpret_cast<const w16*>(p);
  if constexpr (N == 38) {
    w16 b = *reinterpret_cast<const w16*>(p + 16);
    w4 c = *reinterpret_cast<const w4*>(p + 32);
    w2 d = *reinterpret_cast<const w2*>(p + 36);
    asm volatile("" : "+s"(a), "+s"(b), "+s"(c), "+s"(d));
#pragma unroll
    for (int i = 0; i < 16; ++i) words.w[16 + i] = b[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) words.w[32 + i] = c[i];
    words.w[36] = d[0];
    words.w[37] = d[1];
  } else if constexpr (N == 24) {
    w4 b = *reinterpret_cast<const w4*>(p + 16), c = *reinterpret_cast<const w4*>(p + 20);
    asm volatile("" : "+s"(a), "+s"(b), "+s"(c));
#pragma unroll
    for (int i = 0; i < 4; ++i) { words.w[16 + i] = b[i]; words.w[20 + i] = c[i]; }
  } else {
    w4 b = *reinterpret_cast<const w4*>(p + 16);
    asm volatile("" : "+s"(a), "+s"(b));
#pragma unroll
    for (int i = 0; i < 4; ++i) words.w[16 + i] = b[i];
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) words.w[i] = a[i];
  return __builtin_bit_cast(S, words);
}
__device__ __forceinline__ int find_problem(const GemmBatch& batch, int tile) { return tile_starts_find(batch.starts, batch.n, tile); }

// blockIdx -> logical tile so that runs of G consecutive logical tiles (neighbours in a problem's tile grid, which
// read the same operand rows) execute on one XCD and find each other's rows in its L2: consecutive workgroup ids
// are dealt round-robin to the 8 XCDs, so inside every block of 8 * G ids the k-th id that lands on XCD x takes
// logical tile x * G + k.  The ids past the last whole block keep their number.
__device__ __forceinline__ int xcd_block_cyclic(int bid, int total, int G) {
  const int block = 8 * G, whole = total - total % block;
  if (bid >= whole) return bid;
  const int s = bid / block, r = bid - s * block;
  return s * block + (r & 7) * G + (r >> 3);
}

__device__ __forceinline__ v16f_t mfma_bf16(uint4 a, uint4 b, v16f_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf16_t, a), __builtin_bit_cast(v8bf16_t, b), c, 0, 0, 0);
}

// f(0), f(1), .. f(N - 1) with the index as a constant: code that has to be straight-line, whatever the unroller thinks of it.
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

}  // namespace cdp
