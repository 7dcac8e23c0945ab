// C[M][N] (fp32) = A B^T for one problem of few rows, both operands k-contiguous in whole 16-byte chunks: a Linear layer on a
// small batch on its own.
//
// It streams B once (33 MB for 4096 x 4096 in bf16, 6.5 us at the rate of a large copy) and is otherwise a chain of
// memory latencies, so what counts is how many CUs take part and how many bytes each has in flight.  The tiles of the
// tick launch are 64 (or 32) columns wide, which suits the sixteen problems of a tick and leaves one problem on 64 CUs.
// Here a workgroup owns 16 columns of up to 64 rows, and its eight wavefronts share the reduction: wavefront w takes the
// 128-byte pieces w, w + 8, ... of every row, two pieces ahead.  A load covers 8 rows x 128 bytes and the fragments are read
// back out of a staging block of the wavefront's own in LDS (no barrier); loaded in fragment layout, 16 rows x 64 bytes,
// the address path of the CU bounds the kernel at 14 bytes per cycle (64 rows, 4096 x 4096: 20.3 us).  The partial tiles
// meet in LDS and are added in wavefront order.
// 64 rows, 4096 x 4096, bf16: 26.9 us on the tick launch's tiles, 11.9 us so; 32 rows 15.6 -> 7.6; fp32 97 -> 28 us.
#include <algorithm>

#include "elem.h"
#include "kernels.h"

namespace cdp {

namespace {

typedef float v4f_t __attribute__((ext_vector_type(4)));

struct StreamArgs {
  const void* A;
  const void* B;
  float* C;
  int M, N, K, lda, ldb;
};

constexpr int GS_WAVES = 8;

// 64 bytes of k of 16 x 16 outputs: a lane holds one 16-byte chunk of row lane % 16 of either operand.
template <typename T> __device__ __forceinline__ v4f_t stream_mfma(uint4 a, uint4 b, v4f_t c) {
  if constexpr (sizeof(T) == 2) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf16_t, a), __builtin_bit_cast(v8bf16_t, b), c, 0, 0, 0);
  } else {  // four steps of four k, in an order that both operands share
    const float4 x = __builtin_bit_cast(float4, a), y = __builtin_bit_cast(float4, b);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.x, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, y.y, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, y.z, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, y.w, c, 0, 0, 0);
  }
}

// MT: blocks of 16 rows.  FAR: rows so long that byte offsets inside a workgroup's rows may not fit 32 bits (gemm_stream_far).
template <typename T, int MT, bool FAR>
__global__ __launch_bounds__(64 * GS_WAVES, 2) void gemm_stream_kernel(const StreamArgs g) {
  constexpr int VEC = Elem<T>::VEC, PIECE = 8 * VEC;   // elements of a 128-byte piece
  constexpr int NL = 2 * MT + 2;                       // loads per piece: 8 rows x 128 bytes each, A's then B's
  constexpr int PITCH = PIECE + VEC;                   // rows of a staged piece: 144 bytes
  constexpr int STAGE = 8 * NL * PITCH * (int)sizeof(T), PART = MT * 16 * 17 * 4;
  static_assert(PART <= STAGE, "the partial tile takes the place of the staged piece");
  __shared__ __attribute__((aligned(16))) unsigned char smem[GS_WAVES * STAGE];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l15 = lane & 15, q = lane >> 4;
  const int col0 = blockIdx.x * 16, row0 = blockIdx.y * (16 * MT);
  T* const st = reinterpret_cast<T*>(smem + wave * STAGE);
  const int lr = lane >> 3, lk = (lane & 7) * VEC;
  // Buffer loads, all of them unconditional: the wait for a piece counts the loads behind it, and with requests under a condition
  // the compiler waits as if the last had not been made, one piece ahead instead of two.  Pieces past the last read nothing (a
  // buffer of no bytes), nor do chunks past the end of a row; rows and columns past the end repeat the last one: they only
  // reach outputs that are not stored.  A wave with a single piece asks for no other.  us, under conditions / so:
  //   bf16 64 x 4096 x 4096 12.1 / 11.9, 64 x 512 x 512 3.7 / 3.1, 33 x 8192 x 512 5.6 / 5.0, 100 x 1000 x 3000 8.8 / 8.1
  //   fp32 64 x 4096 x 4096 30.5 / 27.9, 30 x 500 x 2004 9.3 / 8.2, 8 x 64 x 64 3.5 / 2.9
  // Far rows are read at 64-bit addresses, just as unconditionally: chunks past the end of a row read its last one and become zeros on
  // their way into LDS.
  constexpr int ES = (int)sizeof(T);
  const char* const pa = static_cast<const char*>(g.A) + (int64_t)row0 * g.lda * ES;
  const char* const pb = static_cast<const char*>(g.B) + (int64_t)col0 * g.ldb * ES;
  unsigned off[NL];
  const char* far[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int r = j < 2 * MT ? min(8 * j + lr, g.M - 1 - row0) : min(8 * (j - 2 * MT) + lr, g.N - 1 - col0), ld = j < 2 * MT ? g.lda : g.ldb;
    if constexpr (FAR) far[j] = (j < 2 * MT ? pa : pb) + (int64_t)r * ld * ES;
    else off[j] = (unsigned)(r * ld + lk) * ES;
  }
  const int step = GS_WAVES * PIECE, first = wave * PIECE;
  const int pieces = first < g.K ? (g.K - first + step - 1) / step : 0;
  auto load = [&](uint4 (&r)[NL], int i) {
    if constexpr (FAR) {
      const unsigned k = min((unsigned)first + (unsigned)i * step + lk, (unsigned)(g.K - VEC));
#pragma unroll
      for (int j = 0; j < NL; ++j) r[j] = *reinterpret_cast<const uint4*>(far[j] + (uint64_t)k * ES);
      return;
    }
    const int k = first + i * step;
    const unsigned records = i < pieces ? 0xfffffff0u : 0u;
    const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(pa), (short)0, records, 0x00020000);
    const auto rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(pb), (short)0, records, 0x00020000);
#pragma unroll
    for (int j = 0; j < NL; ++j) r[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(j < 2 * MT ? ra : rb, k + lk < g.K ? off[j] + (unsigned)k * ES : 0xfffffff0u, 0, 0));
  };
  v4f_t acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i] = v4f_t{0.f, 0.f, 0.f, 0.f};
  // The staged piece is the wavefront's own, whose LDS instructions execute in order: no barrier.
  auto product = [&](const uint4 (&r)[NL], int i) {
    // (by bits: of `past ? zeros : r[j]` the compiler made a branch that left 12 of the 16 registers of the last four chunks as they were)
    const unsigned in = FAR && (unsigned)first + (unsigned)i * step + lk >= (unsigned)g.K ? 0u : ~0u;
#pragma unroll
    for (int j = 0; j < NL; ++j)
      *reinterpret_cast<uint4*>(st + (8 * j + lr) * PITCH + lk) = FAR ? make_uint4(r[j].x & in, r[j].y & in, r[j].z & in, r[j].w & in) : r[j];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const T* f = st + l15 * PITCH + (4 * h + q) * VEC;
      const uint4 b = *reinterpret_cast<const uint4*>(f + 16 * MT * PITCH);
#pragma unroll
      for (int i = 0; i < MT; ++i) acc[i] = stream_mfma<T>(*reinterpret_cast<const uint4*>(f + 16 * i * PITCH), b, acc[i]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  uint4 r0[NL], r1[NL], r2[NL];
  if (pieces == 1) {
    load(r0, 0);
    product(r0, 0);
  } else if (pieces > 1) {
    load(r0, 0);
    load(r1, 1);
    for (int i = 0;;) {  // two pieces ahead
      load(r2, i + 2);
      product(r0, i);
      if (++i == pieces) break;
      load(r0, i + 2);
      product(r1, i);
      if (++i == pieces) break;
      load(r1, i + 2);
      product(r2, i);
      if (++i == pieces) break;
    }
  }
  float (*part)[17] = reinterpret_cast<float (*)[17]>(smem + wave * STAGE);
  // acc[i][v]: row 16 i + 4 q + v, column l15
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[16 * i + 4 * q + v][l15] = acc[i][v];
  __syncthreads();
  for (int e = threadIdx.x; e < MT * 256; e += 64 * GS_WAVES) {
    const int r = e >> 4, c = e & 15;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < GS_WAVES; ++w) s += reinterpret_cast<const float*>(smem + w * STAGE)[r * 17 + c];
    if (row0 + r < g.M && col0 + c < g.N) g.C[(int64_t)(row0 + r) * g.N + col0 + c] = s;
  }
}

template <typename T, bool FAR>
void launch_stream(const StreamArgs& g, hipStream_t stream) {
  const dim3 cols((g.N + 15) / 16, 1), block(64 * GS_WAVES);
  if (g.M <= 16) hipLaunchKernelGGL((gemm_stream_kernel<T, 1, FAR>), cols, block, 0, stream, g);
  else if (g.M <= 32) hipLaunchKernelGGL((gemm_stream_kernel<T, 2, FAR>), cols, block, 0, stream, g);
  else hipLaunchKernelGGL((gemm_stream_kernel<T, 4, FAR>), dim3(cols.x, (g.M + 63) / 64), block, 0, stream, g);
}

// 32-bit byte offsets reach 64 rows of so many elements and the reduction behind them.
bool gemm_stream_far(const StreamArgs& g) { return std::max({g.lda, g.ldb, g.K}) > (1 << 22); }

}  // namespace

// Up to two workgroups per CU: past that the wider tiles of the tick launch fill the chip too and read A less often (us, tick
// launch / here: 64 rows bf16 8192 x 512 8.6 / 5.8, 16384 x 4096 30 / 42; 128 rows 4096 x 4096 27.5 / 22.5, 8192 x 512 9.0 / 10.4;
// fp32 64 rows 4096 x 4096 97 / 32, 16384 x 4096 102 / 115).  Measured for 4 to 128 rows.
bool gemm_stream_wanted(const void* A, const void* B, int M, int N, int K, int lda, int ldb, int dtype) {
  const int vec = dtype == DT_BF16 ? 8 : 4;
  if (K % vec || lda % vec || ldb % vec || ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) & 15)) return false;
  return M <= 128 && (int64_t)((N + 15) / 16) * (M <= 64 ? 1 : 2) <= 512;
}

hipError_t launch_gemm_stream(const void* A, const void* B, float* C, int M, int N, int K, int lda, int ldb, int dtype, hipStream_t stream) {
  const StreamArgs g{A, B, C, M, N, K, lda, ldb};
  const bool far = gemm_stream_far(g);
  if (dtype == DT_BF16) far ? launch_stream<uint16_t, true>(g, stream) : launch_stream<uint16_t, false>(g, stream);
  else far ? launch_stream<float, true>(g, stream) : launch_stream<float, false>(g, stream);
  return hipGetLastError();
}

}  // namespace cdp
