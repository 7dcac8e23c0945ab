// What the forward / data-gradient kernels of conv_kernels.hip and conv256_kernels.hip share: the taps of a tile row and
// the epilogue.
#pragma once
#include "elem.h"
#include "gelu.h"
#include "kernels.h"

namespace cdp {

// Address base (elements) and valid taps (bit kh * KW + kw) of output position r of the gathered operand.  The valid taps are
// the columns that are inside for every row that is, so rows and columns are looked at apart: tap by tap, with a division
// each, the nine taps of a 3x3 data gradient took 2 us per tile.
__device__ __forceinline__ void conv_row(const ConvGeom& g, int mode, int r, int& base, unsigned& mask) {
  const int b = r / (g.OH * g.OW);
  const int rem = r - b * (g.OH * g.OW);
  const int oh = rem / g.OW, ow = rem - oh * g.OW;
  mask = 0;
  if (mode == OP_CONV_FWD) {
    const int ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
    base = ((b * g.H + ih0) * g.W + iw0) * g.C;
    const int kw_lo = max(0, -iw0), kw_hi = min(g.KW, g.W - iw0);
    const unsigned cols = kw_hi > kw_lo ? ((1u << kw_hi) - 1u) & ~((1u << kw_lo) - 1u) : 0u;
    for (int kh = max(0, -ih0); kh < min(g.KH, g.H - ih0); ++kh) mask |= cols << (kh * g.KW);
  } else {  // OP_CONV_DGRAD: (oh, ow) is an input position, the gathered tensor is dy
    const int qh = (oh + g.pad) / g.stride, eh = (oh + g.pad) - qh * g.stride;
    const int qw = (ow + g.pad) / g.stride, ew = (ow + g.pad) - qw * g.stride;
    base = ((b * g.H + qh) * g.W + qw) * g.C;
    unsigned cols = 0;  // taps on the stride lattice whose source lies inside dy
    for (int kw = 0; kw < g.KW; ++kw) {
      const int uw = kw / g.stride;
      if (kw - uw * g.stride == ew && (unsigned)(qw - uw) < (unsigned)g.W) cols |= 1u << kw;
    }
    for (int kh = 0; kh < g.KH; ++kh) {
      const int uh = kh / g.stride;
      if (kh - uh * g.stride == eh && (unsigned)(qh - uh) < (unsigned)g.H) mask |= cols << (kh * g.KW);
    }
  }
}

// What a contraction's result goes through: forward act(acc + bias + residual), data gradient mask(acc + addend (+ old)).  GF_GELU (bf16):
// the forward also stores GELU of the stored result in aux2, the data gradient is that of the GELU's input, aux1.  Both round where the
// kernels of their own round, so the bits are theirs.
//
// Epilogues of a wave tile of MI x NI blocks of 32 x 32.  The blocks are contracted TRANSPOSED (the weight rows are the row
// operand): a lane holds one tile row (its lane % 32) and, per group of four accumulator registers, four neighbouring
// columns of it.
//
// Out of the registers (bf16): one exchange between the lane halves makes eight columns, a 16-byte piece, of them.  No LDS traffic
// and no barrier, but an instruction touches 32 rows, which the address path of the CU takes at less than half the rate of
// whole rows.  Stores count with the loads here, and a load on some path between two stores makes the compiler wait for every
// store before the next one (sixteen round trips one after the other: 10 of the 30 us of a 256 x 256 x 768 tile).  So everything is chosen per
// tile, outside the loops: NSUM tensors are added (forward: the residual; data gradient: addend, old result), MASK: aux1 is a mask or the
// GELU's input.  Operands of the row block after this one are requested before this one's results leave.  Loads and stores
// are buffer instructions: what lies outside the matrix is outside the buffer, no branch, and every tile stores the same number of
// times (conv_gemm_run_kernel counts them).
template <int MI, int NI, bool FWD, int NSUM, bool MASK, bool GELU>
__device__ __forceinline__ void conv_epilogue_as(const GemmProb& P, v16f_t (&acc)[MI][NI], int row0, int col0, int lane) {
  using E = Elem<uint16_t>;
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  constexpr int VEC = 8, NS = 2 * NI, NT = NSUM + (MASK ? 1 : 0), AHEAD = MI * NI > 4 ? 1 : 2;
  const int l31 = lane & 31, hi = lane >> 5;
  const bool fwd = P.epi == EPI_FWD, relu = FWD && fwd && (P.flags & GF_RELU);  // FWD also takes data gradients that read nothing
  const unsigned ldo = P.ldo;
  // A buffer per row block, so that 32-bit offsets reach rows of any number (conv_dl_eligible): rows of the block that the matrix has.  All of it is
  // uniform, and said to be: with a word of the descriptor in a vector register (the compiler clamps there) every access is a loop over the
  // lanes' descriptors, 0.3 us of a 13 us launch.
  // The pointers are read up front, with everything else that is read of the problem.
  const int first_row = __builtin_amdgcn_readfirstlane(row0), M = P.M;
  const int64_t first_byte = 2 * (int64_t)first_row * ldo;
  auto place = [&](const void* p) { return const_cast<char*>(static_cast<const char*>(p)) + first_byte; };
  char* const out = place(P.out);
  char* const out2 = GELU && !MASK ? place(P.aux2) : out;
  char* const t0 = NT == 0 ? out : place(NSUM == 0 || FWD ? P.aux1 : P.aux0 ? P.aux0 : P.out);
  char* const t1 = NT < 2 ? out : place(NSUM == 2 ? P.out : P.aux1);
  char* const t2 = NT < 3 ? out : place(P.aux1);
  auto buffer = [&](char* p, int i) {
    const int rows = __builtin_amdgcn_readfirstlane(min(max(M - first_row - 32 * i, 0), 32));
    return __builtin_amdgcn_make_buffer_rsrc(p + 64 * (int64_t)i * ldo, (short)0, (unsigned)rows * ldo * 2u, 0x00020000);
  };
  unsigned off[NS];  // byte offset of the piece inside its block; columns past the matrix are sent past the buffer
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int c = col0 + 2 * VEC * s + VEC * hi;
    off[s] = c < P.N ? ((unsigned)l31 * ldo + c) * 2u : 0xfffffff0u;
  }
  v4u x[NT ? AHEAD : 1][NT ? NT : 1][NS];
  auto request = [&](int i) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if constexpr (NT > 0) x[i % AHEAD][0][s] = __builtin_amdgcn_raw_buffer_load_b128(buffer(t0, i), off[s], 0, 0);
      if constexpr (NT > 1) x[i % AHEAD][1][s] = __builtin_amdgcn_raw_buffer_load_b128(buffer(t1, i), off[s], 0, 0);
      if constexpr (NT > 2) x[i % AHEAD][2][s] = __builtin_amdgcn_raw_buffer_load_b128(buffer(t2, i), off[s], 0, 0);
    }
  };
  if constexpr (NT > 0 && AHEAD == 2) request(0);
  // The bias of this lane's columns, in one round; none is -0, which changes no value it is added to.  (Waited for here: where it is used the compiler
  // would wait again, for the stores too.  Added to the accumulators ahead of everything, 256 x 256 tiles spilled 66 registers, with a GELU 200:
  // us so / now, 25088 x 2048 x 2048 with bias, residual and ReLU 276 / 248, GELU 268 / 250.  EARLY: small tiles with a GELU do it all the same, the
  // pieces then have no branch: 3000 x 256 x 96 4.65 / 4.59, 25088 x 128 x 1152 with a bias 16.5 / 16.2.)
  typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
  constexpr bool EARLY = FWD && GELU && MI * NI <= 4;
  const bool biased = FWD && fwd && P.aux0, act_in = (biased && !EARLY) || relu;
  v4f bias[FWD ? NS : 1][2];
#pragma unroll
  for (int s = 0; s < (FWD ? NS : 1); ++s) bias[s][0] = bias[s][1] = v4f{-0.f, -0.f, -0.f, -0.f};
  if (EARLY && biased) {  // 32 j + 8 q + 4 hi are the columns of this lane as the products leave them
    v4f b[NI][4];
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) b[j][q] = *reinterpret_cast<const v4f*>(static_cast<const float*>(P.aux0) + min(col0 + 32 * j + 8 * q + 4 * hi, P.N - 4));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += b[j][q][e];
    __builtin_amdgcn_sched_barrier(0);
  }
  if (!EARLY && biased) {
#pragma unroll
    for (int s = 0; s < (FWD ? NS : 0); ++s) {
      const float* const from = static_cast<const float*>(P.aux0) + min(col0 + 2 * VEC * s + VEC * hi, P.N - VEC);  // N is a multiple of VEC on these paths
      bias[s][0] = *reinterpret_cast<const v4f*>(from);
      bias[s][1] = *reinterpret_cast<const v4f*>(from + 4);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if constexpr (NT > 0) {
      if (AHEAD == 1) request(i);
      else if (i + 1 < MI) request(i + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float val[VEC];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][s >> 1][8 * (s & 1) + e]),
                                                        __float_as_uint(acc[i][s >> 1][8 * (s & 1) + 4 + e]), false, false);
        val[e] = __uint_as_float(y[0]);
        val[4 + e] = __uint_as_float(y[1]);
      }
      if (act_in) {  // one branch for what a plain result has not
#pragma unroll
        for (int e = 0; e < VEC; ++e) val[e] += bias[FWD ? s : 0][e >> 2][e & 3];
        if (NSUM == 0 && relu) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) val[e] = fmaxf(val[e], 0.f);
        }
      }
      Chunk16<uint16_t> a, b, c, res, act;
      if constexpr (NT > 0) a.v = __builtin_bit_cast(uint4, x[i % AHEAD][0][s]);
      if constexpr (NT > 1) b.v = __builtin_bit_cast(uint4, x[i % AHEAD][1][s]);
      if constexpr (NT > 2) c.v = __builtin_bit_cast(uint4, x[i % AHEAD][2][s]);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        if constexpr (NSUM > 0) val[e] += E::to_f32(a.e[e]);
        if constexpr (NSUM > 1) val[e] += E::to_f32(b.e[e]);
      }
      if (NSUM > 0 && relu) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) val[e] = fmaxf(val[e], 0.f);
      }
      if constexpr (MASK) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float m = E::to_f32(NSUM == 0 ? a.e[e] : NSUM == 1 ? b.e[e] : c.e[e]);
          if constexpr (GELU) val[e] = E::to_f32(E::from_f32(val[e])) * gelu_df<uint16_t>(m);
          else if (!(m > 0.f)) val[e] = 0.f;
        }
      }
#pragma unroll
      for (int e = 0; e < VEC; ++e) res.e[e] = E::from_f32(val[e]);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, res.v), buffer(out, i), off[s], 0, 0);
      if constexpr (GELU && !MASK) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) act.e[e] = E::from_f32(gelu_f<uint16_t>(E::to_f32(res.e[e])));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, act.v), buffer(out2, i), off[s], 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}
template <int MI, int NI, bool GELU>  // GELU: the launch may hold problems with GF_GELU
__device__ __forceinline__ void conv_epilogue(const GemmProb& P, v16f_t (&acc)[MI][NI], int row0, int col0, int lane) {
  if (P.epi == EPI_FWD) {
    if constexpr (GELU) {
      if (P.flags & GF_GELU) {
        if (P.aux1) return conv_epilogue_as<MI, NI, true, 1, false, true>(P, acc, row0, col0, lane);
        return conv_epilogue_as<MI, NI, true, 0, false, true>(P, acc, row0, col0, lane);
      }
    }
    if (P.aux1) return conv_epilogue_as<MI, NI, true, 1, false, false>(P, acc, row0, col0, lane);
    return conv_epilogue_as<MI, NI, true, 0, false, false>(P, acc, row0, col0, lane);
  }
  const int nsum = (P.aux0 != nullptr) + ((P.flags & GF_ACCUM) != 0);
  if constexpr (GELU) {
    if (P.flags & GF_GELU) {
      if (nsum == 2) return conv_epilogue_as<MI, NI, false, 2, true, true>(P, acc, row0, col0, lane);
      if (nsum == 1) return conv_epilogue_as<MI, NI, false, 1, true, true>(P, acc, row0, col0, lane);
      return conv_epilogue_as<MI, NI, false, 0, true, true>(P, acc, row0, col0, lane);
    }
  }
  if (P.aux1) {
    if (nsum == 2) return conv_epilogue_as<MI, NI, false, 2, true, false>(P, acc, row0, col0, lane);
    if (nsum == 1) return conv_epilogue_as<MI, NI, false, 1, true, false>(P, acc, row0, col0, lane);
    return conv_epilogue_as<MI, NI, false, 0, true, false>(P, acc, row0, col0, lane);
  }
  if (nsum == 2) return conv_epilogue_as<MI, NI, false, 2, false, false>(P, acc, row0, col0, lane);
  if (nsum == 1) return conv_epilogue_as<MI, NI, false, 1, false, false>(P, acc, row0, col0, lane);
  return conv_epilogue_as<MI, NI, false, 0, false, false>(P, acc, row0, col0, lane);
}

// Through LDS, 32 rows at a time and in fp32: every instruction then moves whole rows.  `stage`: conv_stage_floats(NI) floats of
// the wave's own, which no wave reads any more.  NT tensors are read (the sums, then the mask).  Everything that is read - one tensor of all row
// blocks, two or three of as many chunks as the registers of one - is asked for in one round and waited for once, ahead of the stores, which count
// with the loads: a read on some path between two stores had every store wait for the one before, and a bias read element by element was eight
// round trips (us before / so: 100352 x 256 x 64 19.2 / 15.5, with bias, residual and ReLU 25.8 / 21.9; in fp32 6272 x 768 x 192 32.1 / 29.9).
constexpr int conv_stage_floats(int NI) { return 32 * (32 * NI + 4); }
template <typename T, int MI, int NI, bool FWD, int NT, bool GELU>
__device__ __forceinline__ void conv_epilogue_rows_as(const GemmProb& P, const v16f_t (&acc)[MI][NI], int row0, int col0, int lane, float* stage) {
  using E = Elem<T>;
  constexpr int VEC = E::VEC, SP = 32 * NI + 4;                // pitch: rows 4 banks apart
  constexpr int CPS = 32 * NI / VEC, NCH = 32 * CPS / 64;      // chunks per staged row, per lane and pass
  // Row blocks, and chunks of one, whose operands are held at once: no more registers than one tensor of all row blocks takes (or 32), or launches
  // that read nothing pay with their occupancy.
  constexpr int ROOM = MI * NCH > 8 ? MI * NCH : 8, BLOCKS = NT == 1 ? MI : 1;
  constexpr int HELD = NT * NCH <= ROOM || NT < 2 ? NCH : NT * NCH <= 2 * ROOM ? NCH / 2 : NCH / 4;
  static_assert(64 % CPS == 0, "a lane keeps its columns from chunk to chunk");
  const int l31 = lane & 31, hi = lane >> 5;
  const int c = col0 + (lane % CPS) * VEC;
  const bool relu = FWD && (P.flags & GF_RELU), masked = !FWD && P.aux1, accum = !FWD && (P.flags & GF_ACCUM);
  const int M = P.M, N = P.N, ldo = P.ldo;
  T* const out = static_cast<T*>(P.out);
  T* const out2 = GELU ? static_cast<T*>(const_cast<void*>(P.aux2)) : nullptr;
  const T* const t0 = static_cast<const T*>(FWD ? P.aux1 : P.aux0 ? P.aux0 : accum ? P.out : P.aux1);
  const T* const t1 = static_cast<const T*>(P.aux0 && accum ? P.out : P.aux1);
  const T* const t2 = static_cast<const T*>(P.aux1);
  uint4 x[NT ? NT : 1][BLOCKS][HELD];
  auto row = [&](int i, int t) { return row0 + i * 32 + (lane + 64 * t) / CPS; };
  auto request = [&](int i, int first) {  // rows and columns past the matrix repeat the last ones, which are not stored
#pragma unroll
    for (int t = 0; t < HELD; ++t) {
      const int64_t o = (int64_t)min(row(i, first + t), M - 1) * ldo + min(c, N - VEC);
      if constexpr (NT > 0) x[0][i % BLOCKS][t] = *reinterpret_cast<const uint4*>(t0 + o);
      if constexpr (NT > 1) x[1][i % BLOCKS][t] = *reinterpret_cast<const uint4*>(t1 + o);
      if constexpr (NT > 2) x[2][i % BLOCKS][t] = *reinterpret_cast<const uint4*>(t2 + o);
    }
  };
  if constexpr (NT == 1) {
#pragma unroll
    for (int i = 0; i < MI; ++i) request(i, 0);
  }
  const bool biased = FWD && P.aux0;
  float bias[VEC];
  if (biased) {
    typedef float vecf __attribute__((ext_vector_type(VEC), aligned(4)));
    const vecf b = *reinterpret_cast<const vecf*>(static_cast<const float*>(P.aux0) + min(c, N - VEC));
#pragma unroll
    for (int e = 0; e < VEC; ++e) bias[e] = b[e];
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if constexpr (NT > 1) request(i, 0);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the previous pass's reads are done
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(stage + l31 * SP + 32 * j + 8 * g + 4 * hi) = make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int t = 0; t < NCH; ++t) {
      if (NT > 1 && t > 0 && t % HELD == 0) request(i, t);
      if (t % HELD == 0 && (i == 0 || NT > 1)) {
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
      }
      float val[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) val[e] = stage[(lane + 64 * t) / CPS * SP + (lane % CPS) * VEC + e];
      if (biased) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) val[e] += bias[e];
      }
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        Chunk16<T> a;
        a.v = x[q][i % BLOCKS][t % HELD];
        if (q == NT - 1 && masked) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            const float m = E::to_f32(a.e[e]);
            if constexpr (GELU) val[e] = E::to_f32(E::from_f32(val[e])) * gelu_df<T>(m);
            else if (!(m > 0.f)) val[e] = 0.f;
          }
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) val[e] += E::to_f32(a.e[e]);
        }
      }
      if (relu) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) val[e] = fmaxf(val[e], 0.f);
      }
      Chunk16<T> res, act;
#pragma unroll
      for (int e = 0; e < VEC; ++e) res.e[e] = E::from_f32(val[e]);
      if (row(i, t) >= M || c >= N) continue;  // N is a multiple of VEC on these paths
      const int64_t o = (int64_t)row(i, t) * ldo + c;
      *reinterpret_cast<uint4*>(out + o) = res.v;
      if constexpr (GELU && FWD) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) act.e[e] = E::from_f32(gelu_f<T>(E::to_f32(res.e[e])));
        *reinterpret_cast<uint4*>(out2 + o) = act.v;
      }
    }
  }
}
template <typename T, int MI, int NI, bool GELU>  // GELU: the launch may hold problems with GF_GELU
__device__ __forceinline__ void conv_epilogue_rows(const GemmProb& P, const v16f_t (&acc)[MI][NI], int row0, int col0, int lane, float* stage) {
  const bool fwd = P.epi == EPI_FWD;
  const int nt = (P.aux1 != nullptr) + (!fwd && P.aux0) + (!fwd && (P.flags & GF_ACCUM));
  if constexpr (GELU) {
    if (P.flags & GF_GELU) {
      if (fwd) return nt ? conv_epilogue_rows_as<T, MI, NI, true, 1, true>(P, acc, row0, col0, lane, stage) : conv_epilogue_rows_as<T, MI, NI, true, 0, true>(P, acc, row0, col0, lane, stage);
      if (nt == 1) return conv_epilogue_rows_as<T, MI, NI, false, 1, true>(P, acc, row0, col0, lane, stage);
      if (nt == 2) return conv_epilogue_rows_as<T, MI, NI, false, 2, true>(P, acc, row0, col0, lane, stage);
      return conv_epilogue_rows_as<T, MI, NI, false, 3, true>(P, acc, row0, col0, lane, stage);
    }
  }
  if (fwd) return nt ? conv_epilogue_rows_as<T, MI, NI, true, 1, false>(P, acc, row0, col0, lane, stage) : conv_epilogue_rows_as<T, MI, NI, true, 0, false>(P, acc, row0, col0, lane, stage);
  if (nt == 0) return conv_epilogue_rows_as<T, MI, NI, false, 0, false>(P, acc, row0, col0, lane, stage);
  if (nt == 1) return conv_epilogue_rows_as<T, MI, NI, false, 1, false>(P, acc, row0, col0, lane, stage);
  if (nt == 2) return conv_epilogue_rows_as<T, MI, NI, false, 2, false>(P, acc, row0, col0, lane, stage);
  return conv_epilogue_rows_as<T, MI, NI, false, 3, false>(P, acc, row0, col0, lane, stage);
}

}  // namespace cdp
