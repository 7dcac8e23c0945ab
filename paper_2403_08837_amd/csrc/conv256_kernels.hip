// Implicit-GEMM convolution / token-wise linear passes for bf16 on gfx950 with operands loaded straight into LDS: 256 x 256
// outputs per workgroup for large launches with long reductions, smaller tiles with a deeper prefetch for launches short
// of workgroups (conv_dl_tile).
//
// What is different from conv_gemm_kernel (128 x 128, four wavefronts):
//   * operands go from global memory straight into LDS (global_load_lds_dwordx4, 16 bytes per lane, no
//     register round trip and no LDS store instructions); a lane whose chunk is a structural zero (a tap
//     outside the image, a row past the matrix) reads 16 zero bytes from a small device array instead;
//   * one such instruction fills 1 KB of LDS lane by lane, so a tile row is BK unpadded elements and bank
//     conflicts are avoided by an XOR swizzle: 16-byte chunk c of tile row r sits in slot c ^ ((r >> 1) & 7) (slabs of 64;
//     c ^ ((r >> 2) & 3) for slabs of 32; the loading lane picks the global chunk that belongs in its slot); a fragment
//     read of 16 rows x 16 bytes then covers all 64 banks once;
//   * two to four LDS stages: the loads of the next STAGES - 1 slabs are in flight while one is contracted, one
//     barrier per slab.  The stages are separate __shared__ arrays on purpose: the compiler orders an
//     LDS read after every outstanding LDS-writing load it cannot prove disjoint, and a single array would
//     make it wait for the prefetch before the first fragment read;
//   * the fragments of the next 16-deep step are read between the products of the current one (a fixed schedule: left to
//     itself the compiler reads, waits, multiplies);
//   * results leave out of the registers (conv_epilogue).
// Fixed schedule and register epilogue, 256 x 256 tiles: 8192^3 1057 -> 950 us (1160 TFLOP/s), 3x3 over 512 channels,
// 25088 rows, 132 -> 115 us.  LDS bandwidth is the next wall there: wave tiles of 128 x 64 read and the loads write about what
// the LDS of a CU moves in the cycles of their products.
// Same problem descriptors, same epilogues (bias, residual, ReLU; data gradient: addend, accumulate, mask).
#include <algorithm>
#include <type_traits>

#include "conv_tile.h"
#include "elem.h"
#include "kernels.h"

namespace cdp {

namespace {

__device__ uint4 g_zero_chunk[4];  // zero-initialised; source of structural zeros

typedef __attribute__((address_space(3))) void* lds_ptr;

}  // namespace

// BM x BN outputs per workgroup of WAVES_M x WAVES_N wavefronts, slabs of BK, STAGES of them in LDS; WPS: wavefronts per SIMD
// that LDS allows (said to the compiler, which otherwise copies the accumulators between the two register files).
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, bool GELU>
__device__ __forceinline__ void conv_gemm_dl_body(const GemmBatch& batch) {
  constexpr int NWAVE = WAVES_M * WAVES_N;
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;  // wave tile
  constexpr int MI = WTM / 32, NI = WTN / 32;            // MFMA tiles per wave
  constexpr int ROW = BK * 2, CPR = ROW / 16, RPB = 1024 / ROW;  // bytes and chunks of a tile row, rows per 1 KB block
  constexpr int STAGE_BYTES = (BM + BN) * ROW;           // one LDS stage
  constexpr int LPA = BM / RPB / NWAVE, LPB = BN / RPB / NWAVE;  // 1 KB blocks a wave loads per operand and slab
  static_assert(LPA * RPB * NWAVE == BM && LPB * RPB * NWAVE == BN, "tile rows are dealt to the waves in 1 KB blocks");
  static_assert(STAGES >= 2 && STAGES <= 4, "");
  __shared__ __attribute__((aligned(1024))) unsigned char smem0[STAGE_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char smem1[STAGE_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char smem2[STAGES > 2 ? STAGE_BYTES : 1];
  __shared__ __attribute__((aligned(1024))) unsigned char smem3[STAGES > 3 ? STAGE_BYTES : 1];
  constexpr int VEC = 8;
  // 16-byte chunk c of tile row r sits in slot c ^ swz(r) of the row
  auto swz = [](int r) { return BK == 64 ? (r >> 1) & 7 : (r >> 2) & 3; };
  const int tile = xcd_block_cyclic((int)blockIdx.x, batch.total_tiles, 8);
  const GemmProb& P = batch.p[find_problem(batch, tile)];
  const int local = tile - P.tile_begin;
  const int tn = local % P.tiles_n, tm = local / P.tiles_n;
  const int row0 = tm * BM, col0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const uint16_t* __restrict__ Ap = static_cast<const uint16_t*>(P.A);
  const uint16_t* __restrict__ Bp = static_cast<const uint16_t*>(P.B);
  const uint16_t* const zero = reinterpret_cast<const uint16_t*>(g_zero_chunk);
  const ConvGeom g = P.g;
  const int mode = P.a_mode;
  const int C = (mode == OP_PLAIN_K) ? P.K : g.C;  // channels per tap of the gathered tensor

  // rows this lane loads: block (wave * LPA + i) of RPB rows, row lane / CPR of it, slot lane % CPR
  const int lr = lane / CPR, ls = lane % CPR;
  int abase[LPA], boff[LPB];
  unsigned amask[LPA];
#pragma unroll
  for (int i = 0; i < LPA; ++i) {
    const int tr = (wave * LPA + i) * RPB + lr;   // tile row
    const int chunk = ls ^ swz(tr);               // the global chunk whose place is slot ls
    const int r = row0 + tr;
    abase[i] = 0;
    amask[i] = 0;
    if (r < P.M) {
      if (mode == OP_PLAIN_K) {
        abase[i] = r * P.lda + chunk * VEC;
        amask[i] = 1u;
      } else {
        conv_row(g, mode, r, abase[i], amask[i]);
        abase[i] += chunk * VEC;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < LPB; ++i) {
    const int tr = (wave * LPB + i) * RPB + lr, c = col0 + tr;
    boff[i] = c < P.N ? c * P.ldb + (ls ^ swz(tr)) * VEC : -1;
  }

  // wavefront-uniform position of the next slab to load: tap index, its address delta, channel offset inside the tap
  int tap = 0, tdelta = 0, c0 = 0, kh = 0, kw = 0, kload = 0;
  auto issue = [&](unsigned char* stage) {
    const int delta = tdelta + c0;
#pragma unroll
    for (int i = 0; i < LPA; ++i) {
      const uint16_t* pa = ((amask[i] >> tap) & 1u) ? Ap + abase[i] + delta : zero;
      __builtin_amdgcn_global_load_lds(pa, (lds_ptr)(stage + (wave * LPA + i) * 1024), 16, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < LPB; ++i) {
      const uint16_t* pb = boff[i] >= 0 ? Bp + boff[i] + kload : zero;
      __builtin_amdgcn_global_load_lds(pb, (lds_ptr)(stage + BM * ROW + (wave * LPB + i) * 1024), 16, 0, 0);
    }
    kload += BK;
    c0 += BK;
    if (c0 == C) {
      c0 = 0;
      ++tap;
      if (++kw == g.KW) { kw = 0; ++kh; }
      tdelta = mode == OP_CONV_FWD ? (kh * g.W + kw) * g.C : -((kh / g.stride) * g.W + (kw / g.stride)) * g.C;
    }
  };

  v16f_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // fragments: row = base + lane % 32, chunk = 2 * kk + lane / 32
  const int l31 = lane & 31, hi = lane >> 5;
  int offa[MI], offb[NI], swa[MI], swb[NI];
#pragma unroll
  for (int i = 0; i < MI; ++i) { const int r = wm * WTM + i * 32 + l31; offa[i] = r * ROW; swa[i] = swz(r); }
#pragma unroll
  for (int j = 0; j < NI; ++j) { const int r = wn * WTN + j * 32 + l31; offb[j] = BM * ROW + r * ROW; swb[j] = swz(r); }
  auto contract = [&](const unsigned char* stage) {
    constexpr int KK = BK / 16;
    uint4 a[2][MI], b[2][NI];
    auto frags = [&](int kk, int buf) {
#pragma unroll
      for (int i = 0; i < MI; ++i) a[buf][i] = *reinterpret_cast<const uint4*>(stage + offa[i] + (((kk * 2 + hi) ^ swa[i]) << 4));
#pragma unroll
      for (int j = 0; j < NI; ++j) b[buf][j] = *reinterpret_cast<const uint4*>(stage + offb[j] + (((kk * 2 + hi) ^ swb[j]) << 4));
    };
    frags(0, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk + 1 < KK) frags(kk + 1, (kk + 1) & 1);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = mfma_bf16(b[kk & 1][j], a[kk & 1][i], acc[i][j]);  // transposed: see the epilogue
    }
    {  // fragments of the next 16-deep step between the products of the current one
      __builtin_amdgcn_sched_group_barrier(0x100, MI + NI, 0);
#pragma unroll
      for (int kk = 0; kk + 1 < KK; ++kk) {
#pragma unroll
        for (int e = 0; e < MI * NI; ++e) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          if (e < MI + NI) __builtin_amdgcn_sched_group_barrier(0x100, (MI + NI + MI * NI - 1) / (MI * NI), 0);
        }
      }
      __builtin_amdgcn_sched_group_barrier(0x8, MI * NI, 0);
    }
  };

  // Slab t is waited for (every load of this wave but those of the slabs requested after it), the barrier makes it whole
  // and says that every wave is done with slab t - 1, whose stage slab t + STAGES - 1 is then requested into.
  // The compiler keeps its own account of loads that write LDS and of the waits it sees, and merges it over branches in
  // the most careful way: with the wait in assembly, or with a guarded request anywhere before it, it waits for every
  // load at the first fragment read and the deeper prefetch gains nothing.  Hence builtins, and straight-line code for
  // every number of slabs that the unrolled loop leaves.
  const int nslab = P.K / BK;
  unsigned char* const st[4] = {smem0, smem1, smem2, smem3};
  auto wait_slabs = [&](auto n) {  // all but the newest n slabs
    constexpr int N = decltype(n)::value * (LPA + LPB);
    static_assert(N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));  // vmcnt(N) lgkmcnt(0)
  };
  auto barrier = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // slabs 0 .. R - 1 of a row of slabs that starts in stage 0, the first min(R, STAGES - 1) requested already
  auto finish = [&](auto rem) {
    constexpr int R = decltype(rem)::value;
    static_for<R>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      wait_slabs(std::integral_constant<int, (STAGES - 2 < R - 1 - j ? STAGES - 2 : R - 1 - j)>{});
      barrier();
      if constexpr (j + STAGES - 1 < R) issue(st[(j + STAGES - 1) % STAGES]);
      contract(st[j % STAGES]);
    });
  };
  if constexpr (STAGES == 2) {
    issue(smem0);
    __builtin_amdgcn_s_waitcnt(0);
    barrier();
    for (int t = 0; t < nslab; t += 2) {
      if (t + 1 < nslab) issue(smem1);
      contract(smem0);
      __builtin_amdgcn_s_waitcnt(0);
      barrier();
      if (t + 1 >= nslab) break;
      if (t + 2 < nslab) issue(smem0);
      contract(smem1);
      __builtin_amdgcn_s_waitcnt(0);
      barrier();
    }
  } else if (nslab >= STAGES - 1) {
#pragma unroll
    for (int q = 0; q < STAGES - 1; ++q) issue(st[q]);
    int t = 0;
    for (; t + 2 * STAGES - 2 < nslab; t += STAGES) {
#pragma unroll
      for (int q = 0; q < STAGES; ++q) {
        wait_slabs(std::integral_constant<int, STAGES - 2>{});
        barrier();
        issue(st[(q + STAGES - 1) % STAGES]);
        contract(st[q]);
      }
    }
    static_for<STAGES>([&](auto k) {  // STAGES - 1 .. 2 STAGES - 2 slabs are left
      if (nslab - t == STAGES - 1 + decltype(k)::value) finish(std::integral_constant<int, STAGES - 1 + decltype(k)::value>{});
    });
  } else {
    static_for<STAGES - 2>([&](auto k) {
      constexpr int R = 1 + decltype(k)::value;
      if (nslab == R) {
#pragma unroll
        for (int q = 0; q < R; ++q) issue(st[q]);
        finish(std::integral_constant<int, R>{});
      }
    });
  }
  conv_epilogue<uint16_t, MI, NI, GELU>(P, acc, row0 + wm * WTM, col0 + wn * WTN, lane);
}
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, int WPS>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64, WPS) void conv_gemm_dl_kernel(const GemmBatch batch) {
  conv_gemm_dl_body<BM, BN, WAVES_M, WAVES_N, BK, STAGES, false>(batch);
}
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, int WPS>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64, WPS) void conv_gelu_dl_kernel(const GemmBatch batch) {
  conv_gemm_dl_body<BM, BN, WAVES_M, WAVES_N, BK, STAGES, true>(batch);
}
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, int WPS>
static void launch_dl(const GemmBatch& b, dim3 grid, hipStream_t stream) {
  if (conv_has_gelu(b)) hipLaunchKernelGGL((conv_gelu_dl_kernel<BM, BN, WAVES_M, WAVES_N, BK, STAGES, WPS>), grid, dim3(WAVES_M * WAVES_N * 64), 0, stream, b);
  else hipLaunchKernelGGL((conv_gemm_dl_kernel<BM, BN, WAVES_M, WAVES_N, BK, STAGES, WPS>), grid, dim3(WAVES_M * WAVES_N * 64), 0, stream, b);
}

// A forward / data-gradient problem these tiles take: bf16, every reduction slab of `bk` inside one tap, 16-byte aligned
// operands, 32-bit element offsets.
static bool conv_dl_eligible(const GemmProb& p, int dtype, int bk) {
  if (dtype != DT_BF16 || p.epi == EPI_WGRAD || !conv_fast_eligible(p, dtype)) return false;
  const int C = p.a_mode == OP_PLAIN_K ? p.K : p.g.C;
  if (p.K % bk || C % bk) return false;
  if ((reinterpret_cast<uintptr_t>(p.A) | reinterpret_cast<uintptr_t>(p.B) | reinterpret_cast<uintptr_t>(p.out)) & 15) return false;
  if ((p.aux1 && (reinterpret_cast<uintptr_t>(p.aux1) & 15)) || (p.epi == EPI_DGRAD && p.aux0 && (reinterpret_cast<uintptr_t>(p.aux0) & 15)))
    return false;
  const int64_t a_elems = p.a_mode == OP_PLAIN_K ? (int64_t)p.M * p.lda : (int64_t)(p.M / (p.g.OH * p.g.OW) + 1) * p.g.H * p.g.W * p.g.C;
  return a_elems < (1ll << 31) && (int64_t)p.N * p.ldb < (1ll << 31);
}
bool conv_gemm256_eligible(const GemmProb& p, int dtype) { return conv_dl_eligible(p, dtype, 64); }

// Worth it for long reductions (the tile's prologue and epilogue are paid once per 256 x 256 outputs), mostly full tiles, and a tile count
// that rounds well to the CUs.  us, conv_gemm_kernel / 256 x 256 / 256 x 128 / 192 x 128: 8192^3 1206 / 926 / 1024 / 1092, 3x3 over 512 channels with 25088
// rows 173 / 114 / 133 / 162, 25088 x 1024 x 2304 151 / 128 / 150 / 149; nothing lost where three rounds are not full: 25088 x 2048 x 2048 (784 tiles, 3.06
// rounds) 249 / 246 / 245 / 248, 50176 x 1024 x 2048 257 / 261 / 255 / 261, 100352 x 512 x 2304 277 / 266 / 266 / 269.
bool conv_gemm256_wanted(const GemmProb* p, int n, int dtype) {
  constexpr int BM = 256, BN = 256, BK = 64;
  int64_t tiles = 0;
  double useful = 0;
  for (int i = 0; i < n; ++i) {
    if (!conv_gemm256_eligible(p[i], dtype) || p[i].K < 32 * BK) return false;
    tiles += (int64_t)((p[i].M + BM - 1) / BM) * ((p[i].N + BN - 1) / BN);
    useful += (double)p[i].M * p[i].N;
  }
  if (tiles < 192) return false;
  const int64_t rounds = (tiles + 255) / 256;
  return useful / ((double)rounds * 256 * BM * BN) >= 0.75;
}

// Launches of one round or two, and long reductions.  conv_gemm_kernel is one slab ahead and needs its three workgroups per CU to
// cover for each other; the tiles here, one workgroup of eight wavefronts per CU with two slabs on their way, do not, so what counts is how
// full the rounds of 256 tiles are: the smallest of the three whose count fits one round.  us, conv_gemm_kernel / 256 x 128 / 192 x 128 / 128 x 128
// (64 x 128 with four wavefronts, the tile of one round before):
//   25088 x 128 x 1152   24.9 / 21.9 / 18.0 / 14.6 (17.1)     8503 x 344 x 3072    45.1 / 43.7 / 34.5 / 27.5 (31.3)
//   2725 x 928 x 128      7.8 /  8.3 /  7.3 /  6.2 (6.4)      3457 x 984 x 1536    26.3 / 25.8 / 21.3 / 17.7 (19.2)
//   6272 x 768 x 3072    54.2 / 44.3 / 37.3 / 53.2            6272 x 768 x 768     19.9 / 17.1 / 14.2 / 19.4
//   20091 x 256 x 128     9.8 /  9.2 /  8.1 / 10.4            5684 x 768 x 2304    43.4 / 36.0 / 29.7 / 42.1
//   12544 x 512 x 1024   24.5 / 21.3 / 30.8 / 23.3 (264 tiles of 192 x 128: two rounds)
// Past two rounds of 128 x 128 and for reductions of 1024 and more the time is counted in rounds of 256 x 128: one of 192 x 128 is 0.835 of it;
// conv_gemm_kernel, whose workgroups are not in rounds but pile up on the CUs, takes 0.562 - 100 / K for each tile of 128 x 128 that a CU gets, and 0.34.
// (Fitted to 238 products of 512 to 4970 tiles, K 1024 to 4032, rms 3.4 %.  Counted as 0.0027 per tile whatever K and the rounding, 17 of
// them were 2 to 9 % slower than conv_gemm_kernel, now 3, the slowest 0.95; all of them 8.1 % faster than it, 7.1 % with that count.)
//   us, conv_gemm_kernel / 256 x 128 / 192 x 128: 66517 x 824 x 1024 164 / 176 / 176, 68436 x 360 x 1216 94 / 101 / 101, 23232 x 2088 x 1152 159 / 170 / 175,
//   16735 x 1944 x 1344 126 / 132 / 127; 800 tiles of K 2944 121 / 96 / 112, 518 of 3456 101 / 104 / 85, 1524 of 3456 205 / 175 / 184.
//   9673 x 1024 x 1024 35.5 / - / 31.2, 14518 x 768 x 2304 72.9 / - / 62.8, 9209 x 1024 x 4608 127 / - / 106; x 768 30.4 / - / 30.9;
//   eight problems of 6272 x 768 x 3072 306 / 278 / -; four of 6272 x 768 x 2304 110 / 111 / -, left where they are.
// 64 x 64 (below 150 tiles of 128 x 128): slabs of 64 for long reductions, of 32 (twice the workgroups per CU) for short ones
// (6272 x 1024 x 256 13.5 against 11.9, 1568 x 512 x 4608 23.8 against 25.5) and for channel counts that are odd multiples of 32.
//   6272 x 256 x 2304 23 / 17 (conv_gemm_kernel / here)     1568 x 512 x 4608 40 / 24     6272 x 256 x 1024  12.9 / 9.5
// At most 64 output columns: the same two tiles up to 384 rows of 128; past two workgroups per CU very long reductions are
// conv_gemm_kernel's (us, that / slabs of 64 / of 32: 34848 x 64 x 5184 58 / 55 / 67, 34848 x 64 x 9216 100 / 109 / 123, 45000 x 64 x 576 11.5 / 10.1 / 10.1).
// `shared`: there is a workspace in which workgroups can share a reduction.  A long reduction of few tiles is cut there (64 x 64
// tiles of conv_gemm_kernel, up to eight workgroups each) where here it is one chain: the longer it is, the more tiles it takes before
// the chip is busy with chains.  us, shared / here: 49 x 512 x 4608 10.9 / 22.5, 784 x 512 x 4608 17.8 / 22.7, 1568 x 512 x 4608 24.4 / 22.8;
// 784 x 256 x 2304 11.5 / 13.5, 1568 x 256 x 2304 14.3 / 13.4; 392 x 512 x 2048 10.0 / 11.7, 784 x 512 x 2048 15.0 / 11.7; 1568 x 128 x 1152
// 8.5 / 8.9, 3136 x 128 x 1152 10.3 / 9.0; 256 x 64 x 576 7.9 / 6.4.
int conv_dl_tile(const GemmProb* p, int n, int dtype, bool shared) {
  int64_t t256 = 0, t192 = 0, t128 = 0, t64 = 0, narrow = 0, kmax = 0, kmin = INT64_MAX;
  bool slab64 = true, all_narrow = true;
  for (int i = 0; i < n; ++i) {
    if (!conv_dl_eligible(p[i], dtype, 32)) return 0;
    slab64 = slab64 && conv_dl_eligible(p[i], dtype, 64);
    all_narrow = all_narrow && p[i].N <= 64;
    t128 += (int64_t)((p[i].M + 127) / 128) * ((p[i].N + 127) / 128);
    t192 += (int64_t)((p[i].M + 191) / 192) * ((p[i].N + 127) / 128);
    t256 += (int64_t)((p[i].M + 255) / 256) * ((p[i].N + 127) / 128);
    t64 += (int64_t)((p[i].M + 63) / 64) * ((p[i].N + 63) / 64);
    narrow += (int64_t)((p[i].M + 127) / 128);
    kmax = std::max<int64_t>(kmax, p[i].K);
    kmin = std::min<int64_t>(kmin, p[i].K);
  }
  if (shared && kmax >= 1024 && t64 <= std::min<int64_t>(kmax / 24, 256)) return 0;
  const int t6464 = slab64 && kmax >= 1024 ? DL_64x64 : DL_64x64_SHORT;
  if (all_narrow) return narrow < 384 && !(t64 > 512 && kmax > 7168) ? t6464 : 0;
  if (!slab64) return t128 >= 512 ? 0 : t6464;
  if (t128 < 150) return t6464;
  if (t128 <= 256) return DL_128x128;
  if (t128 < 512) return t192 <= 256 ? DL_192x128 : DL_256x128;
  if (kmin < 1024) return 0;
  const double by256 = (double)((t256 + 255) / 256), by192 = 0.835 * ((t192 + 255) / 256);
  const double other = ((t128 + 255) / 256) * (0.562 - 100.0 / kmin) + 0.34;
  return std::min(by256, by192) >= 0.97 * other ? 0 : by192 < by256 ? DL_192x128 : DL_256x128;
}

hipError_t launch_conv_dl(GemmBatch& b, int dtype, int tile, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > GEMM_MAX_PROBS || !conv_gelu_valid(b, dtype)) return hipErrorInvalidValue;
  int bm, bn;
  switch (tile) {
    case DL_256x256: bm = 256; bn = 256; break;
    case DL_256x128: bm = 256; bn = 128; break;
    case DL_192x128: bm = 192; bn = 128; break;
    case DL_128x128: bm = 128; bn = 128; break;
    case DL_64x64: case DL_64x64_SHORT: bm = 64; bn = 64; break;
    default: return hipErrorInvalidValue;
  }
  int64_t total = 0;
  for (int i = 0; i < b.n; ++i) {
    GemmProb& p = b.p[i];
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || !conv_dl_eligible(p, dtype, tile == DL_64x64_SHORT ? 32 : 64)) return hipErrorInvalidValue;
    p.splits = 1;
    p.tiles_n = (p.N + bn - 1) / bn;
    p.tile_begin = (int)total;
    total += (int64_t)((p.M + bm - 1) / bm) * p.tiles_n;
    if (total >= (1ll << 31)) return hipErrorInvalidValue;
  }
  b.total_tiles = (int)total;
  tile_starts_set(b.starts, b.p, b.n);
  const dim3 grid((unsigned)total);
  switch (tile) {
    case DL_256x256: launch_dl<256, 256, 2, 4, 64, 2, 2>(b, grid, stream); break;
    case DL_256x128: launch_dl<256, 128, 4, 2, 64, 3, 2>(b, grid, stream); break;
    case DL_192x128: launch_dl<192, 128, 2, 4, 64, 3, 2>(b, grid, stream); break;
    case DL_128x128: launch_dl<128, 128, 4, 2, 64, 3, 2>(b, grid, stream); break;
    case DL_64x64: launch_dl<64, 64, 2, 2, 64, 3, 3>(b, grid, stream); break;
    default: launch_dl<64, 64, 2, 2, 32, 4, 4>(b, grid, stream); break;
  }
  return hipGetLastError();
}

}  // namespace cdp
