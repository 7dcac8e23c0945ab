// Implicit-GEMM convolution passes of a CDP tick on gfx950, for channel counts that are whole 16-byte chunks, best
// multiples of the reduction slab (bf16: 32, fp32: 16); other shapes (the 3-channel stem) run on the generic kernel of
// gemm.hip.
//
//   conv_gemm_kernel   forward   y[(b,oh,ow)][o]  = sum_{tap,c} x[b][oh*s-p+kh][ow*s-p+kw][c] * wf[o][tap][c]
//                      data grad dx[(b,ih,iw)][c] = sum_{tap,o} dy[b][(ih+p-kh)/s][(iw+p-kw)/s][o] * wt[c][tap][o]
//     A slab of the reduction lies inside one tap, so the tap and its address delta are
//     wavefront-uniform; each thread keeps, per tile row it loads, one base offset and one
//     bit per tap (inside the image / on the stride lattice).  No division in the k-loop.
//   conv_wgrad_kernel  part[range][o][(tap,c)] = sum_{m in range} dy[m][o] * x[pos(m)+tap][c]
//     reduction over output positions, cut into ranges that write partial tiles with plain
//     stores; operands are staged as they lie in memory ([m][channels]) and MFMA fragments are
//     read transposed out of LDS; the per-position address decode is done once per workgroup
//     into an LDS table.  wgrad_reduce_kernel folds the ranges into G (scaled by gamma) and
//     produces d gamma and d beta.
#include <algorithm>

#include "../../include/cdp_kernels.h"
#include "conv_tile.h"
#include "elem.h"
#include "kernels.h"
#include "mfma_frag.h"

namespace cdp {

// Consecutive logical tiles that one XCD takes in a row (xcd_block_cyclic); measured on the ResNet-50 and ViT-B/16
// shaped workloads: 4, 8 and 16 within 0.5 % of each other in time, L2 misses of the forward / data-gradient
// kernel 26 % below the round-robin order.
constexpr int XCD_RUN = 8;

// ---------------------------------------------------------------------------------
// forward / data gradient: 128 x BN tile, waves 2 x 2, reduction slab BK (a divisor of the
// channel count).  Results, residuals and masks move as 16-byte vectors along the
// channel dimension (conv_epilogue).
// RAGGED: channel counts that are whole 16-byte chunks but not whole slabs.  A chunk still lies inside one tap, but a slab
// does not, so tap and address delta are the lane's own (all its rows load the same chunk column), found with a division
// per slab; the last slab may be partial.
// GELU: problems of the launch may have GF_GELU (conv_gelu_kernel).
template <typename T, int BM, int BN, int BK, bool DB, bool RAGGED, bool GELU>
__device__ __forceinline__ void conv_gemm_body(const GemmBatch& batch) {
  using E = Elem<T>;
  constexpr int VEC = E::VEC, LDP = BK + VEC;
  constexpr int WTM = BM / 2, MI = WTM / 32;   // wave tile WTM x WTN
  constexpr int CPR = BK / VEC;                // chunks per tile row
  constexpr int NA = BM * CPR / 256;           // A chunks per thread
  constexpr int NB = BN * CPR / 256;           // B chunks per thread
  constexpr int WTN = BN / 2, NI = WTN / 32;
  // one or two (DB) operand buffers; the staging areas of the epilogue reuse the space.
  // Size: conv_gemm_lds_bytes<T, BM, BN, BK, DB>().
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int BUF = (BM + BN) * LDP;  // elements per operand buffer
  T* const As0 = reinterpret_cast<T*>(smem);

  // runs of XCD_RUN neighbouring tiles (same rows, next columns; then the next rows, whose 3x3 halo they share) on one XCD
  const int tile = xcd_block_cyclic((int)blockIdx.x, batch.total_tiles, XCD_RUN);
  const GemmProb& P = batch.p[find_problem(batch, tile)];
  // a long reduction of a small launch is shared by P.splits workgroups (neighbours in the
  // tile list); the last of them to finish adds the partial tiles and runs the epilogue
  constexpr bool SPLIT = BM == 64 && BN == 64;  // the launcher splits only launches of the smallest tiles
  const int ks = SPLIT ? P.splits : 1, split = (tile - P.tile_begin) % ks;
  const int local = (tile - P.tile_begin) / ks;
  const int tn = local % P.tiles_n, tm = local / P.tiles_n;
  const int row0 = tm * BM, col0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const T* __restrict__ Ap = static_cast<const T*>(P.A);
  const T* __restrict__ Bp = static_cast<const T*>(P.B);
  const ConvGeom g = P.g;
  const int mode = P.a_mode;
  const int C = (mode == OP_PLAIN_K) ? P.K : g.C;  // channels per tap of the gathered tensor

  // per-row state of the A chunks this thread loads
  const int arow = tid / CPR, akc = (tid % CPR) * VEC;
  int abase[NA];
  unsigned amask[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int r = row0 + arow + i * (256 / CPR);
    abase[i] = 0;
    amask[i] = 0;
    if (r < P.M) {
      if (mode == OP_PLAIN_K) {
        abase[i] = r * P.lda;
        amask[i] = 1u;
      } else {
        conv_row(g, mode, r, abase[i], amask[i]);
      }
    }
  }
  const int brow = tid / CPR;
  int boff[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int r = col0 + brow + i * (256 / CPR);
    boff[i] = r < P.N ? r * P.ldb + akc : -1;
  }

  uint4 ra[NA], rb[NB];
  // wavefront-uniform position of the current slab: tap index, channel offset inside the tap
  const int nslab_all = RAGGED ? (P.K + BK - 1) / BK : P.K / BK, per = (nslab_all + ks - 1) / ks;
  const int s_begin = split * per, nslab = max(0, min(nslab_all, s_begin + per) - s_begin);
  const int kbeg = s_begin * BK;
  int tap = kbeg / C, c0 = kbeg - tap * C, kh = 0, kw = 0;
  if (mode != OP_PLAIN_K) { kh = tap / g.KW; kw = tap - kh * g.KW; }
  auto fetch = [&](int k0) {
    if constexpr (RAGGED) {
      const int k = k0 + akc, t = k / C, c = k - t * C;  // one tap when the operand is plain
      int d = c;
      if (mode != OP_PLAIN_K) {
        const int th = t / g.KW, tw = t - th * g.KW;
        if (mode == OP_CONV_FWD) d += (th * g.W + tw) * g.C;
        else if (g.stride == 1) d -= (th * g.W + tw) * g.C;
        else d -= ((th / g.stride) * g.W + (tw / g.stride)) * g.C;
      }
      const bool in = k < P.K;
#pragma unroll
      for (int i = 0; i < NA; ++i)
        ra[i] = in && ((amask[i] >> t) & 1u) ? *reinterpret_cast<const uint4*>(Ap + abase[i] + d) : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < NB; ++i) rb[i] = in && boff[i] >= 0 ? *reinterpret_cast<const uint4*>(Bp + boff[i] + k0) : make_uint4(0, 0, 0, 0);
      return;
    }
    int delta;
    if (mode == OP_PLAIN_K) delta = c0;
    else if (mode == OP_CONV_FWD) delta = (kh * g.W + kw) * g.C + c0;
    else delta = -((kh / g.stride) * g.W + (kw / g.stride)) * g.C + c0;
#pragma unroll
    for (int i = 0; i < NA; ++i)
      ra[i] = ((amask[i] >> tap) & 1u) ? *reinterpret_cast<const uint4*>(Ap + abase[i] + delta + akc) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NB; ++i) rb[i] = boff[i] >= 0 ? *reinterpret_cast<const uint4*>(Bp + boff[i] + k0) : make_uint4(0, 0, 0, 0);
    c0 += BK;
    if (c0 == C) {
      c0 = 0;
      ++tap;
      if (++kw == g.KW) { kw = 0; ++kh; }
    }
  };

  v16f_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  auto stash = [&](int buf) {  // registers -> operand buffer `buf`
    T* As = As0 + buf * BUF;
    T* Bs = As + BM * LDP;
#pragma unroll
    for (int i = 0; i < NA; ++i) *reinterpret_cast<uint4*>(As + (arow + i * (256 / CPR)) * LDP + akc) = ra[i];
#pragma unroll
    for (int i = 0; i < NB; ++i) *reinterpret_cast<uint4*>(Bs + (brow + i * (256 / CPR)) * LDP + akc) = rb[i];
  };
  auto contract = [&](const T* As) {
    const T* Bs = As + BM * LDP;
    const int kg = (lane >> 5) * E::KPL;
    const T* ap = As + (wm * WTM + (lane & 31)) * LDP + kg;
    const T* bp = Bs + (wn * WTN + (lane & 31)) * LDP + kg;
#pragma unroll
    for (int kk = 0; kk < BK; kk += E::MFMA_K) {
      if constexpr (sizeof(T) == 2) {
        uint4 a[MI], b[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) a[i] = *reinterpret_cast<const uint4*>(ap + i * 32 * LDP + kk);
#pragma unroll
        for (int j = 0; j < NI; ++j) b[j] = *reinterpret_cast<const uint4*>(bp + j * 32 * LDP + kk);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = mfma_bf16(b[j], a[i], acc[i][j]);  // transposed: see conv_epilogue
      } else {
        float a[MI], b[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) a[i] = ap[i * 32 * LDP + kk];
#pragma unroll
        for (int j = 0; j < NI; ++j) b[j] = bp[j * 32 * LDP + kk];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j], a[i], acc[i][j], 0, 0, 0);
      }
    }
  };
  if constexpr (DB) {
    // Two operand buffers (small problems, whose k-loop is a chain of latencies): while slab
    // `it` is contracted out of one buffer the loads of slab it+1 are in flight; they are
    // written to the other buffer after the contraction and the loads of slab it+2 are
    // issued.  One barrier per slab.
    if (nslab > 0) {
      fetch(kbeg);
      stash(0);
    }
    if (nslab > 1) fetch(kbeg + BK);
    __syncthreads();
    for (int it = 0; it < nslab; ++it) {
      contract(As0 + (it & 1) * BUF);
      if (it + 1 < nslab) {
        stash((it + 1) & 1);  // last read in iteration it-1, which every wave has left (barrier below)
        if (it + 2 < nslab) fetch(kbeg + (it + 2) * BK);
      }
      __syncthreads();
    }
  } else {
    // One operand buffer (large launches, where more workgroups per CU hide the latency):
    // the next slab's loads are in flight while the current one is contracted.
    if (nslab > 0) fetch(kbeg);
    for (int it = 0; it < nslab; ++it) {
      __syncthreads();
      stash(0);
      __syncthreads();
      if (it + 1 < nslab) fetch(kbeg + (it + 1) * BK);
      contract(As0);
    }
  }

  if (SPLIT && ks > 1) {
    // Partial tile -> this workgroup's slot of the workspace, in register order (lane-contiguous).
    // Partials and counter are device-scope atomics (they bypass the per-XCD L2) ordered by
    // waiting for the stores; the last arrival sums the slots in a fixed order.
    float* slot = batch.thin_ws + (int64_t)tile * (BM * BN);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          __hip_atomic_store(slot + ((i * NI + j) * 16 + v) * 256 + tid, acc[i][j][v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // every store above has been acknowledged before this wavefront reaches the barrier (a
    // workgroup-scope fence alone does not wait for global stores)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();  // also: the operand tiles are no longer read
    unsigned int* cnt = batch.thin_cnt + (tile - split);
    int* flag = reinterpret_cast<int*>(smem);
    if (tid == 0) {
      const unsigned int arrived = atomicAdd(cnt, 1u);
      *flag = arrived == (unsigned)(ks - 1);
      if (arrived == (unsigned)(ks - 1)) atomicExch(cnt, 0u);  // ready for the next launch
    }
    __syncthreads();
    if (!*flag) return;
    const float* first = batch.thin_ws + (int64_t)(tile - split) * (BM * BN);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    // one round trip per group of four slots: all their loads are issued together, then added in slot order
    constexpr int GS = 4, PE = MI * NI * 16;
    for (int sp = 0; sp < ks; sp += GS) {
      float part[GS][PE];
#pragma unroll
      for (int u = 0; u < GS; ++u) {
        const float* src = first + (int64_t)min(sp + u, ks - 1) * (BM * BN) + tid;  // (past the last slot: a harmless re-read)
#pragma unroll
        for (int e = 0; e < PE; ++e) part[u][e] = __hip_atomic_load(src + e * 256, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int u = 0; u < GS; ++u)
        if (sp + u < ks) {
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
              for (int v = 0; v < 16; ++v) acc[i][j][v] += part[u][(i * NI + j) * 16 + v];
        }
    }
  }

  __syncthreads();  // the operand tiles are consumed
  conv_epilogue_rows<T, MI, NI, GELU>(P, acc, row0 + wm * WTM, col0 + wn * WTN, lane, reinterpret_cast<float*>(smem) + wave * conv_stage_floats(NI));
}
// Four workgroups per CU of the 128 x 128 tiles in bf16 with slabs of 32, although epilogues that read spill a few of the 128 registers then (us, three /
// four: 100352 x 128 x 96 13.0 / 11.7, data gradient with mask and addend 20.2 / 19.2; 50176 x 136 x 96 11.2 / 10.1, with a mask 12.8 / 12.2).
template <typename T, int BM, int BN, int BK, bool DB, bool RAGGED>
__global__ __launch_bounds__(256, BM == 128 && BN == 128 ? (sizeof(T) == 2 && BK == 32 ? 4 : 3) : 4) void conv_gemm_kernel(const GemmBatch batch) {
  conv_gemm_body<T, BM, BN, BK, DB, RAGGED, false>(batch);
}
// A kernel of its own: with the second epilogue in conv_gemm_kernel its launches without a GELU lose 2 % (3x3 over 128 channels, three passes, 60.3 ->
// 62.6 us).
template <int BM, int BN, int BK, bool DB, bool RAGGED>
__global__ __launch_bounds__(256, BM == 128 && BN == 128 ? 3 : 4) void conv_gelu_kernel(const GemmBatch batch) {
  conv_gemm_body<uint16_t, BM, BN, BK, DB, RAGGED, true>(batch);
}

// ---------------------------------------------------------------------------------
// weight gradient.  Batch entry convention (as for the generic kernel): A = dy [Mpos][Cout]
// (OP_PLAIN_R, lda = Cout), B = x (OP_CONV_WGRAD geometry, or OP_PLAIN_R with ldb = Cin for a
// 1x1/stride-1 layer), out = G [Cout][taps*Cin] (ldo = taps*Cin), P.M = Cout, P.N = taps*Cin,
// P.K = Mpos, splits = number of reduction ranges.  Each range writes its partial tile with plain
// stores: out = partial sums f32 [splits][Cout][taps*Cin], aux3 = partial column sums of dy
// f32 [splits][Cout] or NULL.  wgrad_reduce_kernel folds the partials into the accumulators
// (device-wide atomics on a small hot array are an order of magnitude slower than this).
constexpr int WG_MAX_SLABS = 16;  // slabs per chunk of a workgroup's range (size of the LDS position table)
template <typename T> struct WgSlab { static constexpr int MB = sizeof(T) == 2 ? 64 : 32; };  // positions per slab
static inline int wg_slab(int dtype) { return dtype == DT_BF16 ? 64 : 32; }

// One tile (TO rows of the weight matrix x 128 columns, one reduction range) of problem P; Ds [MB][TO + PAD],
// Xs [MB][128 + PAD] and the two position tables [WG_MAX_SLABS * MB] are the workgroup's LDS.
template <typename T, int TO>
__device__ __forceinline__ void conv_wgrad_body(const GemmProb& P, int tile, T* __restrict__ Ds, T* __restrict__ Xs,
                                                int* __restrict__ pos_base, int* __restrict__ pos_hw) {
  using E = Elem<T>;
  constexpr int TC = 128, VEC = E::VEC, MB = WgSlab<T>::MB;
  constexpr int PAD = (sizeof(T) == 2) ? 16 : 4;  // bf16: pitch of 32 bytes modulo 128 for the transposing LDS read
  constexpr int PD = TO + PAD, PX = TC + PAD;  // LDS pitches (elements)
  constexpr int WAVES_O = TO / 64;             // 1 or 2
  constexpr int WAVES_C = 4 / WAVES_O;         // 4 or 2
  constexpr int WTC = TC / WAVES_C;            // 32 or 64 columns per wave
  constexpr int NI = WTC / 32;                 // 1 or 2
  const int row_tiles = (P.M + TO - 1) / TO, local = tile - P.tile_begin;
  const int tc = local % P.tiles_n, to = local / P.tiles_n % row_tiles, split = local / P.tiles_n / row_tiles;  // tiles of a range are neighbours
  const int o0 = to * TO, col0 = tc * TC;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wo = wave / WAVES_C, wc = wave % WAVES_C;
  const int Cout = P.M, Ncol = P.N, Mpos = P.K;
  const ConvGeom g = P.g;
  const bool gather = P.b_mode == OP_CONV_WGRAD;
  const int Cin = gather ? g.C : P.ldb;

  const int nslab_total = (Mpos + MB - 1) / MB;
  const int per = (nslab_total + P.splits - 1) / P.splits;
  const int s0 = split * per, s1 = min(nslab_total, s0 + per);
  const int nslab = max(0, s1 - s0);  // an empty range still writes its (zero) partial tile
  const int m_begin = s0 * MB, m_count = max(0, min(Mpos, s1 * MB) - m_begin);

  // this thread's chunks: dy columns (o) and x columns (tap, c) are fixed, rows advance
  constexpr int DCH = TO / VEC, XCH = TC / VEC;  // chunks per staged row
  constexpr int ND = MB * DCH / 256, NX = MB * XCH / 256;
  const int d_c = (tid % DCH) * VEC, d_m = tid / DCH;   // rows d_m + i * (256 / DCH)
  const int x_c = (tid % XCH) * VEC, x_m = tid / XCH;   // rows x_m + i * (256 / XCH)
  const int xcol = col0 + x_c;
  int x_kh = 0, x_kw = 0, x_delta = 0;
  const bool xcol_ok = xcol < Ncol;
  if (xcol_ok) {
    const int tap = xcol / Cin, c = xcol - tap * Cin;
    if (gather) {
      x_kh = tap / g.KW;
      x_kw = tap - x_kh * g.KW;
      x_delta = (x_kh * g.W + x_kw) * g.C + c;
    } else {
      x_delta = c;
    }
  }
  const T* __restrict__ Dp = static_cast<const T*>(P.A);
  const T* __restrict__ Xp = static_cast<const T*>(P.B);
  const bool dcol_ok = o0 + d_c < Cout;  // Cout is a multiple of VEC on this path

  uint4 rd[ND], rx[NX];
  int chunk_q0 = 0;  // first position (relative to m_begin) of the chunk the table describes
  auto fetch = [&](int s) {  // s = slab index inside the chunk; positions s*MB .. s*MB+MB-1 of the table
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int q = chunk_q0 + s * MB + d_m + i * (256 / DCH);
      rd[i] = (dcol_ok && q < m_count) ? *reinterpret_cast<const uint4*>(Dp + (int64_t)(m_begin + q) * P.lda + o0 + d_c)
                                       : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int q = s * MB + x_m + i * (256 / XCH);
      const int hw = pos_hw[q];
      const int ih = (hw >> 16) + x_kh, iw = (int)(short)(hw & 0xffff) + x_kw;
      const bool ok = xcol_ok && (!gather || (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W)) && hw != (int)0x80008000u;
      rx[i] = ok ? *reinterpret_cast<const uint4*>(Xp + pos_base[q] + x_delta) : make_uint4(0, 0, 0, 0);
    }
  };

  v16f_t acc[2][NI];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  const bool do_beta = tc == 0 && P.aux3 != nullptr && wc == 0;
  float bsum[2] = {0.f, 0.f};  // column sums of dy (bf16: out of the fragments that are multiplied anyway)

  // The range is walked in chunks of at most WG_MAX_SLABS slabs; per chunk the positions are
  // decoded once into the LDS table.
  for (int cs = 0; cs < nslab; cs += WG_MAX_SLABS) {
  const int cn = min(WG_MAX_SLABS, nslab - cs);
  chunk_q0 = cs * MB;
  __syncthreads();  // the previous chunk's table and operand tiles are consumed
  // position table: element offset of x[b][oh*s-p][ow*s-p][0] and the packed (ih0, iw0)
  for (int q = tid; q < cn * MB; q += 256) {
    int base = 0, hw = (int)0x80008000u;  // (ih0, iw0) = (-32768, -32768): every tap out of range
    if (chunk_q0 + q < m_count) {
      const int m = m_begin + chunk_q0 + q;
      if (gather) {
        const int b = m / (g.OH * g.OW);
        const int rem = m - b * (g.OH * g.OW);
        const int oh = rem / g.OW, ow = rem - oh * g.OW;
        const int ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
        base = ((b * g.H + ih0) * g.W + iw0) * g.C;
        hw = (int)(((unsigned)(ih0 & 0xffff) << 16) | (unsigned)(iw0 & 0xffff));
      } else {
        base = m * P.ldb;
        hw = 0;
      }
    }
    pos_base[q] = base;
    pos_hw[q] = hw;
  }
  __syncthreads();  // position table complete
  fetch(0);
  for (int s = 0; s < cn; ++s) {
    if (s > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      Chunk16<T> c;
      c.v = rd[i];
      uint2* dst = reinterpret_cast<uint2*>(Ds + (d_m + i * (256 / DCH)) * PD + d_c);
      dst[0] = c.h[0];
      dst[1] = c.h[1];
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      Chunk16<T> c;
      c.v = rx[i];
      uint2* dst = reinterpret_cast<uint2*>(Xs + (x_m + i * (256 / XCH)) * PX + x_c);
      dst[0] = c.h[0];
      dst[1] = c.h[1];
    }
    __syncthreads();
    if (s + 1 < cn) fetch(s + 1);
    const int gq = lane >> 5, l31 = lane & 31;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int kk = 0; kk < MB; kk += 16) {
        uint4 a[2], b[NI];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = frag_tr_bf16(Ds, PD, kk, wo * 64 + i * 32, lane);
#pragma unroll
        for (int j = 0; j < NI; ++j) b[j] = frag_tr_bf16(Xs, PX, kk, wc * WTC + j * 32, lane);
        if (do_beta) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            auto pair = [&](uint32_t w) { return __uint_as_float(w << 16) + __uint_as_float(w & 0xffff0000u); };
            bsum[i] += (pair(a[i].x) + pair(a[i].y)) + (pair(a[i].z) + pair(a[i].w));
          }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = mfma_bf16(a[i], b[j], acc[i][j]);
      }
    } else {
#pragma unroll 8
      for (int kk = 0; kk < MB; kk += 2) {
        float a[2], b[NI];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = Ds[(kk + gq) * PD + wo * 64 + i * 32 + l31];
#pragma unroll
        for (int j = 0; j < NI; ++j) b[j] = Xs[(kk + gq) * PX + wc * WTC + j * 32 + l31];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      // The column sums have a pass of their own: an addition per fragment between the products keeps the compiler from requesting the
      // x fragments of eight steps ahead, and every step then waits for its own (64 rows: 40 x 688 over 16530 positions 37.6 -> 42.2 us).
      if (do_beta) {
#pragma unroll 8
        for (int kk = 0; kk < MB; kk += 2)
#pragma unroll
          for (int i = 0; i < 2; ++i) bsum[i] += Ds[(kk + gq) * PD + wo * 64 + i * 32 + l31];
      }
    }
  }
  }

  // epilogue: acc rows = o, cols = (tap, c); plain stores into this range's partial buffer
  float* __restrict__ part = static_cast<float*>(P.out) + (int64_t)split * Cout * Ncol;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = o0 + wo * 64 + i * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
      if (r >= Cout) continue;
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int c = col0 + wc * WTC + j * 32 + (lane & 31);
        if (c < Ncol) part[(int64_t)r * Ncol + c] = acc[i][j][v];
      }
    }
  if (do_beta) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float sum = bsum[i] + __shfl_xor(bsum[i], 32, 64);
      const int r = o0 + wo * 64 + i * 32 + (lane & 31);
      if (lane < 32 && r < Cout) static_cast<float*>(P.aux3)[(int64_t)split * Cout + r] = sum;
    }
  }
}

template <typename T, int TO>
__global__ __launch_bounds__(256) void conv_wgrad_kernel(const GemmBatch batch) {
  constexpr int MB = WgSlab<T>::MB, PAD = (sizeof(T) == 2) ? 16 : 4;
  __shared__ __attribute__((aligned(16))) T Ds[MB * (TO + PAD)];
  __shared__ __attribute__((aligned(16))) T Xs[MB * (128 + PAD)];
  __shared__ int pos_base[WG_MAX_SLABS * MB];
  __shared__ int pos_hw[WG_MAX_SLABS * MB];
  const int tile = xcd_block_cyclic((int)blockIdx.x, batch.total_tiles, batch.xcd_run);
  conv_wgrad_body<T, TO>(batch.p[find_problem(batch, tile)], tile, Ds, Xs, pos_base, pos_hw);
}
// Tiles of both heights in one launch (the height is the problem's: 128 rows for matrices of 128 rows and more, 64
// below): the weight gradients of a tick are one launch instead of one per height, each of which alone is short
// of workgroups on the small ResNet configurations.
__host__ __device__ inline int conv_wgrad_rows(const GemmProb& p) { return p.M >= 128 ? 128 : 64; }
template <typename T>
__global__ __launch_bounds__(256) void conv_wgrad_mixed_kernel(const GemmBatch batch) {
  constexpr int MB = WgSlab<T>::MB, PAD = (sizeof(T) == 2) ? 16 : 4;
  __shared__ __attribute__((aligned(16))) T Ds[MB * (128 + PAD)];
  __shared__ __attribute__((aligned(16))) T Xs[MB * (128 + PAD)];
  __shared__ int pos_base[WG_MAX_SLABS * MB];
  __shared__ int pos_hw[WG_MAX_SLABS * MB];
  const int tile = xcd_block_cyclic((int)blockIdx.x, batch.total_tiles, batch.xcd_run);
  const GemmProb& P = batch.p[find_problem(batch, tile)];
  if (conv_wgrad_rows(P) == 128) conv_wgrad_body<T, 128>(P, tile, Ds, Xs, pos_base, pos_hw);
  else conv_wgrad_body<T, 64>(P, tile, Ds, Xs, pos_base, pos_hw);
}

// Fold of the partial sums.  A workgroup is 8 groups of 32 lanes; a lane owns 4 of the 128
// columns of its group's weight row.  Depending on the number of ranges, `rg` = 1, 2, 4 or 8
// groups share one row (each summing every rg-th range) and the workgroup covers 8/rg rows,
// so layers with few ranges still give every lane work and layers with hundreds of ranges
// still split the long sum.  The workgroups of all problems form one flat list.
//   s[c] = sum_ranges part[.][o][c];  G[o][c] += gamma[o]*s[c];
//   d gamma[o] += sum_c s[c]*Wplain[o][c]  (one atomic per 128 columns);
//   d beta[o]  += sum_ranges part_beta[.][o]  (first column chunk only).
//
// What bounds it is the chain of memory round trips of a workgroup (some 8 KB of traffic each, thousands of them in a launch), so
// everything it reads (its partial sums up to 8 per lane, the accumulator, weights, gamma) is asked for in one round, and the
// share of d gamma leaves ahead of the accumulator.  In ResNet-50-shaped training with 64 samples a micro-batch, us per launch with
// up to five rounds of reads / so: 4288 workgroups 67 / 42, 8768 workgroups 59 / 45, 704 workgroups 12.6 / 10.9.
template <typename T, bool VEC> __device__ __forceinline__ void wgrad_reduce_piece(const WReduceProb& P, float4 (&red)[8][32], int& last) {
  using E = Elem<T>;
  const int rg = P.rg, rows_per_wg = 8 / rg, splits = P.splits;
  const int chunks = (P.Ncol + 127) >> 7;
  const int local = (int)blockIdx.x - P.tile_begin;
  const int ob = local / chunks, chunk = local - ob * chunks, c0 = chunk * 128;
  const int cl = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int o = ob * rows_per_wg + grp / rg, q0 = grp % rg;
  const int c = c0 + cl * 4;
  const bool row_ok = o < P.Cout, owner = row_ok && q0 == 0;  // the owner group of 32 lanes finishes row o
  const int64_t row = (int64_t)o * P.Ncol, stride = (int64_t)P.Cout * P.Ncol;
  const bool beta = c0 == 0 && P.Gbeta, alone = P.Ggamma && chunks == 1;
  float gam = 1.f, sb = 0.f, gbeta = 0.f, ggamma = 0.f;
  float gold[4] = {0.f, 0.f, 0.f, 0.f};
  T wpl[4] = {};
  uint2 wpl_bits[sizeof(T) / 2] = {};  // the four of them as they lie in memory: unpacked here they would be waited for here
  if (owner) {
    if (P.gamma) gam = P.gamma[o];
    if (VEC) {
      if (c < P.Ncol) {
        if (!P.overwrite) *reinterpret_cast<float4*>(gold) = *reinterpret_cast<const float4*>(P.G + row + c);
        if (P.wplain) {
#pragma unroll
          for (int e = 0; e < (int)sizeof(T) / 2; ++e) wpl_bits[e] = reinterpret_cast<const uint2*>(static_cast<const T*>(P.wplain) + row + c)[e];
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < P.Ncol) {
          if (!P.overwrite) gold[e] = P.G[row + c + e];
          if (P.wplain) wpl[e] = static_cast<const T*>(P.wplain)[row + c + e];
        }
    }
    if (beta && cl < splits) sb = P.part_beta[(int64_t)cl * P.Cout + o];
    if (beta && cl == 0) gbeta = P.Gbeta[o];
    if (alone && cl == 0) ggamma = P.Ggamma[o];
  }
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  if (row_ok && VEC) {
    if (c < P.Ncol) {
      const float* src = P.part + row + c;
      float4 s1 = sum, s2 = sum, s3 = sum;
      for (int q = q0; q < splits; q += 8 * rg) {
        float4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = q + j * rg < splits ? *reinterpret_cast<const float4*>(src + (q + j * rg) * stride) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
          if (q + (h + 3) * rg < splits) {  // four running sums; what is left at the end goes to the first
            sum.x += v[h].x; sum.y += v[h].y; sum.z += v[h].z; sum.w += v[h].w;
            s1.x += v[h + 1].x; s1.y += v[h + 1].y; s1.z += v[h + 1].z; s1.w += v[h + 1].w;
            s2.x += v[h + 2].x; s2.y += v[h + 2].y; s2.z += v[h + 2].z; s2.w += v[h + 2].w;
            s3.x += v[h + 3].x; s3.y += v[h + 3].y; s3.z += v[h + 3].z; s3.w += v[h + 3].w;
          } else {
#pragma unroll
            for (int j = h; j < h + 3; ++j) { sum.x += v[j].x; sum.y += v[j].y; sum.z += v[j].z; sum.w += v[j].w; }
          }
        }
      }
      sum.x += (s1.x + s2.x) + s3.x; sum.y += (s1.y + s2.y) + s3.y;
      sum.z += (s1.z + s2.z) + s3.z; sum.w += (s1.w + s2.w) + s3.w;
    }
  } else if (row_ok) {
    for (int q = q0; q < splits; q += 4 * rg) {
      float v[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][e] = q + j * rg < splits && c + e < P.Ncol ? P.part[(q + j * rg) * stride + row + c + e] : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) { sum.x += v[j][0]; sum.y += v[j][1]; sum.z += v[j][2]; sum.w += v[j][3]; }
    }
  }
  float tot[4] = {0.f, 0.f, 0.f, 0.f};
  if (rg > 1) {
    red[grp][cl] = sum;
    __syncthreads();
    if (owner)
      for (int k = 0; k < rg; ++k) {
        const float4 v = red[grp + k][cl];
        tot[0] += v.x; tot[1] += v.y; tot[2] += v.z; tot[3] += v.w;
      }
  } else if (owner) {
    tot[0] += sum.x; tot[1] += sum.y; tot[2] += sum.z; tot[3] += sum.w;
  }
  if (VEC) __builtin_memcpy(wpl, wpl_bits, sizeof(wpl));
  auto finish = [&]() {
    if (!owner) return;
    if (VEC) {
      if (c < P.Ncol)
        *reinterpret_cast<float4*>(P.G + row + c) = make_float4(gold[0] + gam * tot[0], gold[1] + gam * tot[1], gold[2] + gam * tot[2], gold[3] + gam * tot[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < P.Ncol) P.G[row + c + e] = gold[e] + gam * tot[e];
    }
    if (beta) {
      for (int q = cl + 32; q < splits; q += 32) sb += P.part_beta[(int64_t)q * P.Cout + o];
#pragma unroll
      for (int off = 16; off >= 1; off >>= 1) sb += __shfl_xor(sb, off, 64);
      if (cl == 0) P.Gbeta[o] = gbeta + sb;
    }
  };
  if (!P.Ggamma) {  // uniform over the workgroup
    finish();
    return;
  }
  float dg = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) dg += tot[e] * E::to_f32(wpl[e]);  // zeros past the end and in lanes of other groups
  // the 32 lanes of a group (shuffles stay inside a half wavefront)
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) dg += __shfl_xor(dg, off, 64);
  if (chunks == 1) {
    if (owner && cl == 0) P.Ggamma[o] = ggamma + dg;
    finish();
    return;
  }
  if (!P.gpart || !P.cnt) {
    if (owner && cl == 0) atomicAdd(P.Ggamma + o, dg);
    finish();
    return;
  }
  // share of this chunk -> workspace; the last workgroup of the row block to get here adds the shares of
  // every row of the block in chunk order.  Shares and counter are device-scope atomics ordered by waiting
  // for the stores' acknowledgement before the barrier (as in the split contraction tiles).
  if (owner && cl == 0) __hip_atomic_store(P.gpart + (int64_t)o * chunks + chunk, dg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  unsigned int arrived = 0;
  if (threadIdx.x == 0) arrived = atomicAdd(P.cnt + ob, 1u);
  finish();
  if (threadIdx.x == 0) {
    last = arrived == (unsigned)(chunks - 1);
    if (last) atomicExch(P.cnt + ob, 0u);  // ready for the next launch
  }
  __syncthreads();
  if (!last) return;
  if ((int)threadIdx.x < rows_per_wg) {
    const int orow = ob * rows_per_wg + (int)threadIdx.x;
    if (orow < P.Cout) {
      const float old = P.Ggamma[orow];
      float total = 0.f;
      for (int k = 0; k < chunks; k += 8) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = k + j < chunks ? __hip_atomic_load(P.gpart + (int64_t)orow * chunks + k + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) total += v[j];
      }
      P.Ggamma[orow] = old + total;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const WReduceBatch batch) {
  __shared__ float4 red[8][32];
  __shared__ int last;
  const WReduceProb& P = batch.p[tile_starts_find(batch.starts, batch.n, (int)blockIdx.x)];
  // rows of the partial buffers are 16-byte aligned where they are whole groups of four
  if ((P.Ncol & 3) == 0 && (reinterpret_cast<uintptr_t>(P.G) & 15) == 0 && (reinterpret_cast<uintptr_t>(P.wplain) & 7) == 0)
    wgrad_reduce_piece<T, true>(P, red, last);
  else
    wgrad_reduce_piece<T, false>(P, red, last);
}

// The same fold for layers with at most 8 ranges and rows of whole 16-byte groups, by rows: a group of 32 lanes
// walks all 128-column chunks of one weight row (eight rows per workgroup), so a row's d gamma is complete inside
// its group - no shares in a workspace, no counters, no barriers - and a workgroup moves 8 whole rows instead of
// 4 KB of the accumulator.  Every sum is associated as wgrad_reduce_kernel associates it (ranges: groups of four
// into four running sums, the rest into the first; a chunk's d gamma share: the lane's four products in order,
// then the 32-lane exchange tree; shares in chunk order), so the two kernels give the same bits.
template <typename T>
__global__ __launch_bounds__(256) void wgrad_fold_rows_kernel(const WReduceBatch batch) {
  using E = Elem<T>;
  const WReduceProb& P = batch.p[tile_starts_find(batch.starts, batch.n, (int)blockIdx.x)];
  const int cl = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int o = ((int)blockIdx.x - P.tile_begin) * 8 + grp;
  if (o >= P.Cout) return;  // whole 32-lane groups leave: the exchanges below stay inside a group
  const int splits = P.splits, chunks = (P.Ncol + 127) >> 7;
  const int64_t row = (int64_t)o * P.Ncol, stride = (int64_t)P.Cout * P.Ncol;
  const float gam = P.gamma ? P.gamma[o] : 1.f;
  const T* __restrict__ wplain = static_cast<const T*>(P.wplain);
  float dgsum = 0.f;
  for (int chunk = 0; chunk < chunks; ++chunk) {
    const int c = chunk * 128 + cl * 4;
    float dg = 0.f;
    if (c < P.Ncol) {
      const float* src = P.part + row + c;
      float4 v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = q < splits ? *reinterpret_cast<const float4*>(src + q * stride) : make_float4(0.f, 0.f, 0.f, 0.f);
      const float4 gold = P.overwrite ? make_float4(0.f, 0.f, 0.f, 0.f) : *reinterpret_cast<const float4*>(P.G + row + c);
      float wpl[4] = {0.f, 0.f, 0.f, 0.f};
      if (wplain) {
#pragma unroll
        for (int e = 0; e < 4; ++e) wpl[e] = E::to_f32(wplain[row + c + e]);
      }
      float4 sum = make_float4(0.f, 0.f, 0.f, 0.f), s1 = sum, s2 = sum, s3 = sum;
      const int full = splits & ~3;
#pragma unroll
      for (int q = 0; q < 8; q += 4)
        if (q + 3 < splits) {
          sum.x += v[q].x; sum.y += v[q].y; sum.z += v[q].z; sum.w += v[q].w;
          s1.x += v[q + 1].x; s1.y += v[q + 1].y; s1.z += v[q + 1].z; s1.w += v[q + 1].w;
          s2.x += v[q + 2].x; s2.y += v[q + 2].y; s2.z += v[q + 2].z; s2.w += v[q + 2].w;
          s3.x += v[q + 3].x; s3.y += v[q + 3].y; s3.z += v[q + 3].z; s3.w += v[q + 3].w;
        }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q >= full && q < splits) { sum.x += v[q].x; sum.y += v[q].y; sum.z += v[q].z; sum.w += v[q].w; }
      sum.x += (s1.x + s2.x) + s3.x; sum.y += (s1.y + s2.y) + s3.y;
      sum.z += (s1.z + s2.z) + s3.z; sum.w += (s1.w + s2.w) + s3.w;
      const float tot[4] = {0.f + sum.x, 0.f + sum.y, 0.f + sum.z, 0.f + sum.w};
      *reinterpret_cast<float4*>(P.G + row + c) =
          make_float4(gold.x + gam * tot[0], gold.y + gam * tot[1], gold.z + gam * tot[2], gold.w + gam * tot[3]);
#pragma unroll
      for (int e = 0; e < 4; ++e) dg += tot[e] * wpl[e];
    }
    if (chunk == 0 && P.Gbeta) {
      float sb = 0.f;
      for (int q = cl; q < splits; q += 32) sb += P.part_beta[(int64_t)q * P.Cout + o];
#pragma unroll
      for (int off = 16; off >= 1; off >>= 1) sb += __shfl_xor(sb, off, 64);
      if (cl == 0) P.Gbeta[o] += sb;
    }
    if (P.Ggamma) {
#pragma unroll
      for (int off = 16; off >= 1; off >>= 1) dg += __shfl_xor(dg, off, 64);
      dgsum += dg;
    }
  }
  if (P.Ggamma && cl == 0) P.Ggamma[o] += dgsum;
}

hipError_t launch_wgrad_reduce(WReduceBatch& b, int dtype, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > WREDUCE_MAX_PROBS) return hipErrorInvalidValue;
  {
    // by rows where every problem allows it and the launch still has a few workgroups per compute unit
    bool rows_ok = true;
    int64_t wgs = 0;
    for (int i = 0; i < b.n && rows_ok; ++i) {
      const WReduceProb& p = b.p[i];
      rows_ok = p.splits >= 1 && p.splits <= 8 && p.Cout > 0 && p.Ncol > 0 && p.Ncol % 4 == 0 &&
                reinterpret_cast<uintptr_t>(p.part) % 16 == 0 && reinterpret_cast<uintptr_t>(p.G) % 16 == 0 && (!p.Gbeta || p.part_beta);
      wgs += (p.Cout + 7) / 8;
    }
    if (rows_ok && wgs >= 512 && wgs < (1ll << 31)) {
      int total = 0;
      for (int i = 0; i < b.n; ++i) {
        b.p[i].tile_begin = total;
        total += (b.p[i].Cout + 7) / 8;
      }
      tile_starts_set(b.starts, b.p, b.n);
      if (dtype == DT_BF16) hipLaunchKernelGGL((wgrad_fold_rows_kernel<uint16_t>), dim3((unsigned)total), dim3(256), 0, stream, b);
      else hipLaunchKernelGGL((wgrad_fold_rows_kernel<float>), dim3((unsigned)total), dim3(256), 0, stream, b);
      return hipGetLastError();
    }
  }
  int64_t total = 0;
  for (int i = 0; i < b.n; ++i) {
    WReduceProb& p = b.p[i];
    if (p.Cout <= 0 || p.Ncol <= 0 || p.splits <= 0) return hipErrorInvalidValue;
    if ((p.gpart == nullptr) != (p.cnt == nullptr)) return hipErrorInvalidValue;
    p.rg = p.splits <= 8 ? 1 : p.splits <= 16 ? 2 : p.splits <= 32 ? 4 : 8;
    const int rows_per_wg = 8 / p.rg;
    p.tile_begin = (int)total;
    total += (int64_t)((p.Cout + rows_per_wg - 1) / rows_per_wg) * ((p.Ncol + 127) / 128);
    if (total >= (1ll << 31)) return hipErrorInvalidValue;
  }
  tile_starts_set(b.starts, b.p, b.n);
  dim3 grid((unsigned)total), block(256);
  if (dtype == DT_BF16) hipLaunchKernelGGL((wgrad_reduce_kernel<uint16_t>), grid, block, 0, stream, b);
  else hipLaunchKernelGGL((wgrad_reduce_kernel<float>), grid, block, 0, stream, b);
  return hipGetLastError();
}

int conv_wgrad_slab(int dtype) { return wg_slab(dtype); }

int conv_wgrad_splits(const GemmProb& p, int dtype, int wanted) {
  // Short ranges (one per WG_MAX_SLABS slabs) measured faster than few long ones as long as the
  // launch is short of workgroups, even though they write more partial sums; a layer with
  // enough tiles of its own does not need them.
  const int nslab = (p.K + wg_slab(dtype) - 1) / wg_slab(dtype);
  const int to = p.M >= 128 ? 128 : 64;
  const int tiles = ((p.M + to - 1) / to) * ((p.N + 127) / 128);
  const int min_splits = std::min((nslab + WG_MAX_SLABS - 1) / WG_MAX_SLABS, (1024 + tiles - 1) / tiles);
  return std::max(1, std::min(nslab, std::max(wanted, min_splits)));
}

// Ranges of a problem launched on its own, at most `room` of them: the cheapest by what the launch costs on conv_wgrad_kernel.  A workgroup's
// slab takes a chain of latencies alone on its CU and longer beside others; how much longer is matrix time, which depends on the type
// and on the height of the tile.  The workgroups run in rounds of as many as a CU holds, and every range writes its partial
// matrix once and the fold reads it once.  Fitted to 900 launches of that kernel (150 shapes of 1 to 310 tiles, 1 to 12544 slabs, 1 to 784
// ranges, rms 2.5 % in fp32 and 5 % in bf16) with the reduction ranges listed side by side.  It does not know the kernels that launches short
// of workgroups run on (conv_wgrad_small.hip), but its counts serve them: of 13 shapes timed with 3 to 11 counts, each on the kernel that it runs
// on, the chosen count is the fastest or within 4 % of it, but for fp32 128 x 576 over 800 (five ranges 11.9 us, four 11.1).  Against three
// ranges or one per 16 slabs, us:
//   bf16 3072 x 768 over 6272 rows 75.5 -> 68.7, 128 x 1152 over 25088 30.7 -> 29.5, 136 x 19800 over 15129 251 -> 252;
//   fp32 128 x 576 over 800 12.5 -> 11.9, 280 x 504 over 40656 175 -> 160, 56 x 792 over 39546 76.9 -> 64.7.
// A function of the shape where there is room for what it wants, which is what cdp_k_conv asks of its workspace and no more than
// the library's own array where one per 16 slabs or three fit that: cdp_k_conv and cdp_k_conv_wgrad_static then add
// in one order and give the same bits (128 x 1152 over 25088 in bf16 is 28 ranges so, 29.5 us; 49, 30.6 us, would not fit).
int conv_wgrad_splits_alone(const GemmProb& p, int dtype, int room) {
  // us per slab with 1, 2, .. workgroups on the CU: [fp32, bf16][tiles of 64, 128 rows]
  static const double SLAB_US[2][2][4] = {{{1.95, 2.9, 3.9, 4.85}, {3.1, 5.15, 7.1, 9.4}}, {{1.25, 1.5, 1.7, 0.0}, {1.45, 1.8, 2.05, 0.0}}};
  const bool bf16 = dtype == DT_BF16, tall = p.M >= 128;
  const double* slab_us = SLAB_US[bf16][tall];
  const int resident = bf16 ? 3 : 4, to = tall ? 128 : 64;
  const int64_t nslab = ((int64_t)p.K + wg_slab(dtype) - 1) / wg_slab(dtype);
  const int64_t tiles = (int64_t)((p.M + to - 1) / to) * ((p.N + 127) / 128);
  const double range_us = 2.0 * 4.0 * p.M * (double)p.N / (bf16 ? 6e6 : 7e6);
  int64_t most = std::max<int64_t>(1, std::min<int64_t>(room, (int64_t)p.K / 512 + 4));
  const int64_t own = (int64_t)CDP_STATIC_SCRATCH_BYTES / (4ll * p.M * p.N);
  if (conv_wgrad_splits(p, dtype, 3) <= own) most = std::min(most, own);
  int64_t best = 1;
  double best_us = 1e30;
  for (int64_t len = 1; len <= nslab; len += 1 + len / 16) {  // slabs per range
    const int64_t s = (nslab + len - 1) / len;
    if (s > most) continue;
    const int64_t rounds = tiles * s / (256 * resident), rest = tiles * s - rounds * 256 * resident;
    const double us = len * (rounds * slab_us[resident - 1] + (rest ? slab_us[(rest - 1) / 256] : 0.0)) + s * range_us;
    if (us < best_us) { best_us = us; best = s; }
  }
  return (int)best;
}

// ---------------------------------------------------------------------------------
bool conv_fast_eligible(const GemmProb& p, int dtype) {
  const int vec = dtype == DT_BF16 ? 8 : 4;
  if (p.epi == EPI_WGRAD) {
    if (p.a_mode != OP_PLAIN_R) return false;
    if (p.b_mode == OP_CONV_WGRAD) {
      if (p.g.C % vec || p.g.KH * p.g.KW > 32 || p.g.H >= 32768 || p.g.W >= 32768) return false;
    } else if (p.b_mode == OP_PLAIN_R) {
      if (p.ldb % vec || p.N > p.ldb) return false;
    } else {
      return false;
    }
    return (p.M % vec) == 0 && (p.lda % vec) == 0;
  }
  if (p.b_mode != OP_PLAIN_K || p.ldb != p.K || (p.K % vec)) return false;
  if ((p.flags & GF_OUT_F32) || (p.N % vec) || (p.ldo % vec)) return false;
  const int C = p.a_mode == OP_PLAIN_K ? p.K : p.g.C;
  if (C % (dtype == DT_BF16 ? 32 : 16)) {  // the ragged kernel: pieces of 16 bytes at 32-bit offsets
    const uintptr_t at = reinterpret_cast<uintptr_t>(p.A) | reinterpret_cast<uintptr_t>(p.B) | reinterpret_cast<uintptr_t>(p.out) |
                         reinterpret_cast<uintptr_t>(p.aux1) | (p.epi == EPI_DGRAD ? reinterpret_cast<uintptr_t>(p.aux0) : 0);
    const int64_t a_elems = p.a_mode == OP_PLAIN_K ? (int64_t)p.M * p.lda : (int64_t)(p.M / (p.g.OH * p.g.OW) + 1) * p.g.H * p.g.W * p.g.C;
    if ((at & 15) || a_elems >= (1ll << 31) || (int64_t)p.N * p.ldb >= (1ll << 31)) return false;
  }
  if (p.a_mode == OP_PLAIN_K) return p.lda == p.K;
  if (p.a_mode == OP_CONV_FWD || p.a_mode == OP_CONV_DGRAD) return (p.g.C % vec) == 0 && p.g.KH * p.g.KW <= 32;
  return false;
}

template <typename T, int BM, int BN, int BK, bool DB>
constexpr int conv_gemm_lds_bytes() {
  constexpr int oper = (DB ? 2 : 1) * (BM + BN) * (BK + 16 / (int)sizeof(T)) * (int)sizeof(T), stage = 4 * conv_stage_floats(BN / 64) * 4;
  return oper > stage ? oper : stage;
}

// fp32, few tiles: a workgroup per 32 x 32 tile of the result, its four wavefronts take every fourth slab of 32 of the reduction
// with both operands straight from memory (16-byte pieces of 32 rows, both sides' columns in the same order), and add their tiles
// through LDS in wavefront order.  Bound by the latency of memory: the zeros of a tap outside the image are put in right behind the
// request, a use, so that the products of a slab wait for the gathered pieces of the next one, a round trip per slab of a wavefront.
// 162 tiles, 1152 deep (3x3, stride 2, data gradient of 32 x 9 x 9 x 64: nine slabs each) 38.6 us as 41 tiles of 64 x 64,
// 12.6 us so; 100 tiles, 576 deep (five) 20.6 -> 8.8 us.
__global__ __launch_bounds__(256, 2) void conv_gemm_few_kernel(const GemmBatch batch) {
  __shared__ float red[4 * 16 * 64];
  const int tile = blockIdx.x;
  const GemmProb& P = batch.p[find_problem(batch, tile)];
  const int local = tile - P.tile_begin, tn = local % P.tiles_n, tm = local / P.tiles_n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l31 = lane & 31, hi = lane >> 5;
  const int r = tm * 32 + l31, col0 = tn * 32;
  const ConvGeom g = P.g;
  const int mode = P.a_mode, C = mode == OP_PLAIN_K ? P.K : g.C;
  int base = 0;
  unsigned mask = 0;
  if (r < P.M) {
    if (mode == OP_PLAIN_K) {
      base = r * P.lda;
      mask = 1u;
    } else {
      conv_row(g, mode, r, base, mask);
    }
  }
  const float* Ap = static_cast<const float*>(P.A) + 4 * hi;
  const float* Bp = static_cast<const float*>(P.B) + (int64_t)min(col0 + l31, P.N - 1) * P.ldb + 4 * hi;
  auto load = [&](float4 (&a)[4], float4 (&b)[4], int k) {
    const int tap = k / C, c0 = k - tap * C;
    int delta = c0;
    if (mode != OP_PLAIN_K) {
      const int kh = tap / g.KW, kw = tap - kh * g.KW;
      if (mode == OP_CONV_FWD) delta += (kh * g.W + kw) * g.C;
      else delta -= ((kh / g.stride) * g.W + (kw / g.stride)) * g.C;
    }
    const bool in = (mask >> tap) & 1u;
    const float* p = Ap + (in ? base + delta : 0);  // a select, no branch: the loads go out together
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      a[s] = *reinterpret_cast<const float4*>(p + 8 * s);
      b[s] = *reinterpret_cast<const float4*>(Bp + k + 8 * s);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      a[s].x = in ? a[s].x : 0.f;
      a[s].y = in ? a[s].y : 0.f;
      a[s].z = in ? a[s].z : 0.f;
      a[s].w = in ? a[s].w : 0.f;
    }
  };
  v16f_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  auto contract = [&](const float4 (&a)[4], const float4 (&b)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {  // transposed: see conv_epilogue
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[s].x, a[s].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[s].y, a[s].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[s].z, a[s].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[s].w, a[s].w, acc, 0, 0, 0);
    }
  };
  constexpr int STEP = 4 * 32;
  float4 a0[4], b0[4], a1[4], b1[4];
  int k = 32 * wave;
  if (k < P.K) load(a0, b0, k);
  for (; k < P.K; k += 2 * STEP) {
    if (k + STEP < P.K) load(a1, b1, k + STEP);
    contract(a0, b0);
    if (k + STEP >= P.K) break;
    if (k + 2 * STEP < P.K) load(a0, b0, k + 2 * STEP);
    contract(a1, b1);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = acc[v];
  __syncthreads();
  const int c = col0 + 8 * wave + 4 * hi;  // each wavefront finishes four columns per lane half
  if (r >= P.M || c >= P.N) return;
  const int64_t o = (int64_t)r * P.ldo + c;
  const bool fwd = P.epi == EPI_FWD, biased = fwd && P.aux0, added = !fwd && P.aux0, accum = !fwd && (P.flags & GF_ACCUM);
  float* const out = static_cast<float*>(P.out) + o;
  typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
  const v4f none = {0.f, 0.f, 0.f, 0.f};  // all that is read, in one round
  const v4f bias = biased ? *reinterpret_cast<const v4f*>(static_cast<const float*>(P.aux0) + c) : none;
  const v4f x1 = P.aux1 ? *reinterpret_cast<const v4f*>(static_cast<const float*>(P.aux1) + o) : none;
  const v4f x0 = added ? *reinterpret_cast<const v4f*>(static_cast<const float*>(P.aux0) + o) : none;
  const v4f old = accum ? *reinterpret_cast<const v4f*>(out) : none;
  v4f val;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float* x = red + (4 * wave + e) * 64 + lane;
    val[e] = (x[0] + x[1024]) + (x[2048] + x[3072]);
  }
  if (fwd) {
    if (biased) val += bias;
    if (P.aux1) val += x1;
    if (P.flags & GF_RELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) val[e] = fmaxf(val[e], 0.f);
    }
  } else {
    if (added) val += x0;
    if (accum) val += old;
    if (P.aux1) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!(x1[e] > 0.f)) val[e] = 0.f;
    }
  }
  *reinterpret_cast<v4f*>(out) = val;
}

template <typename T, int BM, int BN, int BK, bool DB, bool RAGGED>
static hipError_t launch_conv_gemm_inst(const GemmBatch& b, dim3 grid, hipStream_t stream) {
  constexpr int lds = conv_gemm_lds_bytes<T, BM, BN, BK, DB>();
  static_assert(lds <= 64 * 1024, "stays within the default dynamic LDS limit");
  if constexpr (sizeof(T) == 2 && !(BM == 128 && BN == 64)) {  // (a GELU's contractions are more than 64 columns wide)
    if (conv_has_gelu(b)) {
      hipLaunchKernelGGL((conv_gelu_kernel<BM, BN, BK, DB, RAGGED>), grid, dim3(256), lds, stream, b);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((conv_gemm_kernel<T, BM, BN, BK, DB, RAGGED>), grid, dim3(256), lds, stream, b);
  return hipGetLastError();
}

template <typename T, int BK, bool RAGGED = false>
static hipError_t launch_conv_gemm_typed(const GemmBatch& b, int bm, int bn, dim3 grid, hipStream_t stream) {
  if (bm == 128 && bn == 128) return launch_conv_gemm_inst<T, 128, 128, BK, false, RAGGED>(b, grid, stream);
  if (bm == 128) return launch_conv_gemm_inst<T, 128, 64, BK, false, RAGGED>(b, grid, stream);
  if (bn == 128) return launch_conv_gemm_inst<T, 64, 128, BK, true, RAGGED>(b, grid, stream);
  return launch_conv_gemm_inst<T, 64, 64, BK, true, RAGGED>(b, grid, stream);
}

// Tile shape for the forward / data-gradient problems of one launch: the largest of
// 128x128, 64x128, 64x64 (128x64, 64x64 when every output is at most 64 wide) that still
// yields enough workgroups over the whole launch.
void conv_gemm_tile(const GemmProb* p, int n, int* bm, int* bn) {
  const int want = 384;
  bool narrow = true;
  for (int i = 0; i < n; ++i) narrow = narrow && p[i].N <= 64;
  auto tiles = [&](int tm, int tn) {
    int t = 0;
    for (int i = 0; i < n; ++i) t += ((p[i].M + tm - 1) / tm) * ((p[i].N + tn - 1) / tn);
    return t;
  };
  if (narrow) {
    *bn = 64;
    *bm = tiles(128, 64) >= want ? 128 : 64;
  } else if (tiles(128, 128) >= want) {
    *bm = 128; *bn = 128;
  } else if (tiles(64, 128) >= want) {
    *bm = 64; *bn = 128;
  } else {
    *bm = 64; *bn = 64;
  }
}

// Launches of conv_gemm_few_kernel: fp32, up to three workgroups per CU, and no workspace in which 64 x 64 tiles could share
// their reductions over workgroups (with it those are the faster ones: a ResNet-18-shaped fp32 step of 4 samples 3.03 against
// 3.38 ms).  64 x 64 tiles without it against these, us: 256 tiles, 4608 deep 130 / 37; 512 tiles, 2304 deep 68 / 36; 600
// tiles, 768 deep 27 / 23; 1024 tiles, 1152 deep 39 / 40; 1568 tiles, 64 deep 8.9 / 9.3.
static bool conv_few_tiles(const GemmBatch& b, int dtype) {
  if (dtype != DT_F32 || b.thin_ws) return false;
  const GemmProb* p = b.p;
  int64_t tiles = 0;
  for (int i = 0; i < b.n; ++i) {
    if (p[i].M <= 0 || p[i].N <= 0 || p[i].K <= 0 || p[i].epi == EPI_WGRAD || !conv_fast_eligible(p[i], dtype)) return false;
    if ((p[i].a_mode == OP_PLAIN_K ? p[i].K : p[i].g.C) % 32) return false;
    tiles += (int64_t)((p[i].M + 31) / 32) * ((p[i].N + 31) / 32);
  }
  return tiles <= 768;
}

// The tile is a wish: bf16 launches whose channels are whole slabs run on the direct-to-LDS tiles (conv_launch_tile) unless they share reductions or have
// many tiles of at most 64 columns, fp32
// launches of few tiles without a workspace on conv_gemm_few_kernel.  What is left for 64 x 64 tiles here is shared reductions, ragged
// channel counts and fp32; for 64 x 128, ragged, fp32, and operands that are not 16-byte aligned or need 64-bit offsets.
hipError_t launch_conv_gemm(GemmBatch& b, int dtype, int bm, int bn, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > GEMM_MAX_PROBS) return hipErrorInvalidValue;
  if ((bm != 64 && bm != 128) || (bn != 64 && bn != 128)) return hipErrorInvalidValue;
  const int bk = dtype == DT_BF16 ? 32 : 16;
  int total = 0;
  if (!conv_gelu_valid(b, dtype) || (conv_has_gelu(b) && bm == 128 && bn == 64)) return hipErrorInvalidValue;
  if (const int dl = conv_launch_tile(b.p, b.n, dtype, b.thin_ws && b.thin_cnt)) return launch_conv_dl(b, dtype, dl, stream);
  if (conv_few_tiles(b, dtype)) {
    for (int i = 0; i < b.n; ++i) {
      GemmProb& p = b.p[i];
      p.splits = 1;
      p.tiles_n = (p.N + 31) / 32;
      p.tile_begin = total;
      total += ((p.M + 31) / 32) * p.tiles_n;
    }
    b.total_tiles = total;
    tile_starts_set(b.starts, b.p, b.n);
    hipLaunchKernelGGL(conv_gemm_few_kernel, dim3(total), dim3(256), 0, stream, b);
    return hipGetLastError();
  }
  bool deep = true;  // every problem allows the double-depth slab
  // One problem whose channels are not whole slabs takes the whole launch to the RAGGED kernel.  Ragged problems in a launch of their own
  // (with the others on the direct-to-LDS tiles), ms per step of ResNets on 4 micro-batches, one launch / two: width 16 (one stage in four ragged) of 16
  // samples 1.51 / 1.60, width 24 (two in four) 1.70 / 1.66, in fp32 2.47 / 2.59, width 40 of 32 samples 2.27 / 2.35, width 80 of 8 3.08 / 2.89, ResNet-50 of width 16
  // 4.78 / 4.62: a launch fewer per level is worth more on most.  (All on the element-by-element kernel: 2.57, 3.80, 3.86, 7.15, 6.57, 6.73.)
  bool ragged = false;
  for (int i = 0; i < b.n; ++i) {
    GemmProb& p = b.p[i];
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || p.epi == EPI_WGRAD || !conv_fast_eligible(p, dtype)) return hipErrorInvalidValue;
    const int C = p.a_mode == OP_PLAIN_K ? p.K : p.g.C;
    if (C % (2 * bk)) deep = false;
    if (C % bk) ragged = true;
    p.splits = 1;
    p.tiles_n = (p.N + bn - 1) / bn;
    p.tile_begin = total;
    total += ((p.M + bm - 1) / bm) * p.tiles_n;
  }
  // A launch short of workgroups shares its long reductions: about 640 workgroups in all,
  // ranges of at least 4 slabs, at most 8 per tile, while the partial tiles fit the workspace.
  // (64 x 64 tiles only: the partial tile of a larger one costs more than the shorter chain saves)
  if (b.thin_ws && b.thin_cnt && total < 512 && bm == 64 && bn == 64) {
    const int slab = deep || ragged ? 2 * bk : bk, want = (640 + total - 1) / total;
    int split_total = 0;
    for (int i = 0; i < b.n; ++i) {
      GemmProb& p = b.p[i];
      p.splits = std::max(1, std::min(std::min(want, 8), p.K / slab / 4));
      split_total += ((p.M + bm - 1) / bm) * p.tiles_n * p.splits;
    }
    if (split_total <= CONV_SPLIT_SLOTS && (int64_t)split_total * bm * bn * 4 <= CONV_SPLIT_WS_BYTES) {
      total = 0;
      for (int i = 0; i < b.n; ++i) {
        b.p[i].tile_begin = total;
        total += ((b.p[i].M + bm - 1) / bm) * b.p[i].tiles_n * b.p[i].splits;
      }
    } else {
      for (int i = 0; i < b.n; ++i) b.p[i].splits = 1;
    }
  }
  b.total_tiles = total;
  tile_starts_set(b.starts, b.p, b.n);
  dim3 grid(total);
  if (ragged) return dtype == DT_BF16 ? launch_conv_gemm_typed<uint16_t, 64, true>(b, bm, bn, grid, stream)
                                      : launch_conv_gemm_typed<float, 32, true>(b, bm, bn, grid, stream);
  if (dtype == DT_BF16) return deep ? launch_conv_gemm_typed<uint16_t, 64>(b, bm, bn, grid, stream)
                                    : launch_conv_gemm_typed<uint16_t, 32>(b, bm, bn, grid, stream);
  return deep ? launch_conv_gemm_typed<float, 32>(b, bm, bn, grid, stream)
              : launch_conv_gemm_typed<float, 16>(b, bm, bn, grid, stream);
}

// Neighbouring weight-gradient tiles that go to one XCD (xcd_block_cyclic: whole blocks of eight such runs, what is left keeps its place).  The
// tiles of a range read the same rows of dy and x, so an XCD that holds many of them finds those rows in its L2; dealt one by one every
// XCD reads every row.  Launches of several shapes take shorter runs: their tiles are of different lengths and long runs leave an
// XCD with the longest ones.  us with 1 / 8 / 16 / 32 / 64:
//   six ResNet stages, 11 layers (about 1400 tiles)     145.5 / 141.6 / 141.5 / 143.4 / 165.8
//   16 ViT layers of 6272 rows, two ranges (3456)       556.6 / 547.8 / 543.1 / 538.1 / 531.0
//   3072 x 768 over 6272 rows, five ranges (720)         57.9 /  54.8 /  53.6 /  53.1 /  52.2
// (170, 589 and 58.1 with the ranges as neighbours and the column sums of dy read back out of LDS row by row: what the first column is better is
// those two together, the rest the XCDs.)
// Short ranges of many tiles in one round (bf16: 768 workgroups are resident) have little to share, and there what counts is that the work
// starts spread out: us with 1 / 4 / 32, bf16,
//   648 x 576 over 3200, ten ranges (300 tiles)     22.6 / 25.4 / 25.9      1984 x 648 over 1088, three (288)    24.5 / 26.1 / 27.7
//   104 x 5688 over 2048, seven (630)               21.9 / 22.0 / 24.3      40 x 8424 over 2448, eight (528)     18.6 / 18.6 / 20.8
//   776 x 120 over 85050, 103 (721: long ranges)    78.8 / 54.4 / 54.1      272 x 368 over 18432, 36 (324: few tiles) 29.7 / 27.4 / 27.5
// 411 launches of 250 to 2000 tiles: 6.3 % faster than ranges as neighbours, 5.9 % with runs of 32 throughout (the slowest 0.95 and 0.87).
int conv_wgrad_xcd_run(const GemmBatch& b) {
  if (b.n > 1) return b.total_tiles >= 2048 ? 32 : 16;
  const int ranges = b.p[0].splits, tiles = b.total_tiles / ranges;
  if (b.total_tiles <= 768 && b.p[0].K / ranges <= 600 && tiles >= (b.total_tiles <= 512 ? 28 : 40)) return b.total_tiles <= 512 ? 1 : 4;
  return 32;
}

hipError_t launch_conv_wgrad_mixed(GemmBatch& b, int dtype, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > GEMM_MAX_PROBS) return hipErrorInvalidValue;
  int total = 0;
  for (int i = 0; i < b.n; ++i) {
    GemmProb& p = b.p[i];
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || p.epi != EPI_WGRAD || !conv_fast_eligible(p, dtype)) return hipErrorInvalidValue;
    if (p.splits < 1 || p.splits > (p.K + wg_slab(dtype) - 1) / wg_slab(dtype)) return hipErrorInvalidValue;  // the caller sized the partial buffer
  }
  if (conv_wgrad_small_wanted(b, dtype)) return launch_conv_wgrad_small(b, dtype, stream);
  for (int i = 0; i < b.n; ++i) {
    GemmProb& p = b.p[i];
    const int to = conv_wgrad_rows(p);
    p.tiles_n = (p.N + 127) / 128;
    p.tile_begin = total;
    total += ((p.M + to - 1) / to) * p.tiles_n * p.splits;
  }
  b.total_tiles = total;
  tile_starts_set(b.starts, b.p, b.n);
  b.xcd_run = conv_wgrad_xcd_run(b);
  if (dtype == DT_BF16) hipLaunchKernelGGL((conv_wgrad_mixed_kernel<uint16_t>), dim3(total), dim3(256), 0, stream, b);
  else hipLaunchKernelGGL((conv_wgrad_mixed_kernel<float>), dim3(total), dim3(256), 0, stream, b);
  return hipGetLastError();
}

hipError_t launch_conv_wgrad(GemmBatch& b, int dtype, bool wide, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > GEMM_MAX_PROBS) return hipErrorInvalidValue;
  const int to = wide ? 128 : 64;
  int total = 0;
  for (int i = 0; i < b.n; ++i) {
    GemmProb& p = b.p[i];
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || p.epi != EPI_WGRAD || !conv_fast_eligible(p, dtype)) return hipErrorInvalidValue;
    if (p.splits < 1 || p.splits > (p.K + wg_slab(dtype) - 1) / wg_slab(dtype)) return hipErrorInvalidValue;  // the caller sized the partial buffer
  }
  if (conv_wgrad_small_wanted(b, dtype)) return launch_conv_wgrad_small(b, dtype, stream);
  for (int i = 0; i < b.n; ++i) {
    GemmProb& p = b.p[i];
    p.tiles_n = (p.N + 127) / 128;
    p.tile_begin = total;
    total += ((p.M + to - 1) / to) * p.tiles_n * p.splits;
  }
  b.total_tiles = total;
  tile_starts_set(b.starts, b.p, b.n);
  b.xcd_run = conv_wgrad_xcd_run(b);
  dim3 grid(total), block(256);
  if (dtype == DT_BF16) {
    if (wide) hipLaunchKernelGGL((conv_wgrad_kernel<uint16_t, 128>), grid, block, 0, stream, b);
    else hipLaunchKernelGGL((conv_wgrad_kernel<uint16_t, 64>), grid, block, 0, stream, b);
  } else {
    if (wide) hipLaunchKernelGGL((conv_wgrad_kernel<float, 128>), grid, block, 0, stream, b);
    else hipLaunchKernelGGL((conv_wgrad_kernel<float, 64>), grid, block, 0, stream, b);
  }
  return hipGetLastError();
}

}  // namespace cdp
