// Implicit-GEMM convolution / token-wise linear passes for bf16 on gfx950 with operands loaded straight into LDS: 256 x 256
// outputs per workgroup for large launches with long reductions, smaller tiles with a deeper prefetch for launches short
// of workgroups (conv_dl_tile).
//
// What is different from conv_gemm_kernel (128 x 128, four wavefronts):
//   * operands go from global memory straight into LDS (16 bytes per lane, no register round trip and no LDS store
//     instructions), as buffer loads: a lane whose chunk is a structural zero (a tap outside the image) asks for an offset past the
//     buffer and gets zeros, so that a slab costs no address arithmetic in the vector unit: the offsets change with the tap,
//     the scalar base with the slab;
//   * one such instruction fills 1 KB of LDS lane by lane, so a tile row is BK unpadded elements and bank
//     conflicts are avoided by an XOR swizzle: 16-byte chunk c of tile row r sits in slot c ^ ((r >> 1) & 7) (slabs of 64;
//     c ^ ((r >> 2) & 3) for slabs of 32; the loading lane picks the global chunk that belongs in its slot); a fragment
//     read of 16 rows x 16 bytes then covers all 64 banks once;
//   * two to four LDS stages: the loads of the next STAGES - 1 slabs are in flight while one is contracted, one barrier per slab.  The
//     loads are assembly without outputs: the compiler keeps an account of loads that write LDS and waits for all of them at fragment
//     reads it cannot tell apart from them (every second slab waited for the one just requested); here the waits are
//     those written down, and the barrier's fences keep the fragment reads between the barriers they belong to;
//   * the barrier stands before the last 16-deep step of a slab, whose fragments are in registers by then: the first fragments of the next
//     slab are read, and the loads into the stage just freed requested, between the products of that step.  With the barrier between two
//     slabs all eight wavefronts waited for their first fragments at once;
//   * fragments of the next 16-deep step are read between the products of the current one, in the order of the source (sched_barrier);
//   * results leave out of the registers (conv_epilogue).
// us, with compiler-ordered loads, the barrier between slabs and an epilogue whose stores waited for each other / so: 8192^3 936 / 804 (1367 TFLOP/s),
// 3x3 over 512 channels with 25088 rows 111 / 97 (256 x 256); 6272 x 768 x 3072 37.5 / 33.6 (192 x 128); 25088 x 128 x 1152 14.6 / 14.0 (128 x 128);
// 1568 x 512 x 4608 22.5 / 20.9, 6272 x 256 x 1024 9.4 / 8.6 (64 x 64).  Outputs bit for bit the same.
// Same problem descriptors, same epilogues (bias, residual, ReLU; data gradient: addend, accumulate, mask).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "conv_tile.h"
#include "elem.h"
#include "kernels.h"

namespace cdp {

namespace {

typedef __attribute__((address_space(3))) void* lds_ptr;

}  // namespace

// Slabs of one tile on their way into LDS: what conv_gemm_dl_kernel loads, and where it stands.  A wavefront fills LPA blocks of 1 KB of
// the gathered operand and LPB of the weights per slab.
template <int BM, int BN, int NWAVE, int BK>
struct SlabLoads {
  static constexpr int ROW = BK * 2, CPR = ROW / 16, RPB = 1024 / ROW;  // bytes and chunks of a tile row, rows per 1 KB block
  static constexpr int LPA = BM / RPB / NWAVE, LPB = BN / RPB / NWAVE, N = LPA + LPB;
  static_assert(LPA * RPB * NWAVE == BM && LPB * RPB * NWAVE == BN, "tile rows are dealt to the waves in 1 KB blocks");
  // 16-byte chunk c of tile row r sits in slot c ^ swz(r) of the row
  static __device__ __forceinline__ int swz(int r) { return BK == 64 ? (r >> 1) & 7 : (r >> 2) & 3; }

  ConvGeom g;
  int mode, C;                    // C: channels per tap of the gathered tensor
  int left, tap, c0, kh, kw;      // slabs left; position of the next one: tap, channel offset inside it
  const char *first, *pa, *pb;    // of the next slab, for offset 0; first: of tap (0, 0)
  unsigned records;               // bytes of either buffer: 0 once nothing is left
  unsigned abase[LPA], amask[LPA], aoff[LPA], boff[LPB];  // byte offsets; valid taps of a row, bit kh * KW + kw

  __device__ __forceinline__ void at_tap() {
#pragma unroll
    for (int i = 0; i < LPA; ++i) aoff[i] = (amask[i] >> tap) & 1u ? abase[i] : ~0u;
  }
  __device__ __forceinline__ void start(const GemmProb& P, int row0, int col0, int wave, int lane) {
    g = P.g;
    mode = P.a_mode;
    C = mode == OP_PLAIN_K ? P.K : g.C;
    left = P.K / BK;
    tap = c0 = kh = kw = 0;
    records = 0xfffffff0u;
    // offsets count from the lowest row's base (in the padding before the first image, or past its first positions)
    const int lowest = mode == OP_PLAIN_K ? 0 : mode == OP_CONV_FWD ? -(g.pad * g.W + g.pad) * g.C : ((g.pad / g.stride) * g.W + g.pad / g.stride) * g.C;
    pa = first = static_cast<const char*>(P.A) + 2 * (int64_t)lowest;
    pb = static_cast<const char*>(P.B);
    // block (wave * LPA + i) of RPB rows, row lane / CPR of it, slot lane % CPR; rows past the matrix repeat the last one: they only
    // reach results that are not stored
    const int lr = lane / CPR, ls = lane % CPR;
#pragma unroll
    for (int i = 0; i < LPA; ++i) {
      const int tr = (wave * LPA + i) * RPB + lr, r = min(row0 + tr, P.M - 1);
      int base;
      amask[i] = 1u;
      if (mode == OP_PLAIN_K) base = r * P.lda;
      else conv_row(g, mode, r, base, amask[i]);
      abase[i] = 2u * ((unsigned)base - (unsigned)lowest + (ls ^ swz(tr)) * 8);
    }
    at_tap();
#pragma unroll
    for (int i = 0; i < LPB; ++i) {
      const int tr = (wave * LPB + i) * RPB + lr, c = min(col0 + tr, P.N - 1);
      boff[i] = 2u * (unsigned)(c * P.ldb + (ls ^ swz(tr)) * 8);
    }
  }
  // Load e of the next slab into the stage whose rows of the gathered operand begin at LDS address `at` (those of the weights behind them).
  __device__ __forceinline__ void issue(unsigned at, int wave, int e) const {
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    const uintptr_t p = (uintptr_t)(e < LPA ? pa : pb);
    // (uniform; said so because the compiler at times keeps them in vector registers, which the instruction does not take)
    auto uniform = [](unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane((int)x); };
    const v4u buffer = {uniform((unsigned)p), uniform((unsigned)(p >> 32)), uniform(records), 0x00020000u};
    const unsigned lds = at + (e < LPA ? (wave * LPA + e) * 1024 : BM * ROW + (wave * LPB + e - LPA) * 1024);
    // The wait states of this are ours, the compiler does not look into assembly: one between the write of m0 and the load, five between a
    // write of a descriptor word by the vector unit (the readfirstlane above may be the instruction before) and the load that reads it.  The
    // s_mov_b32 is one and s_nop 3 four, whatever stands before.  (us so / with the words pinned in scalar registers a slab
    // ahead: 8192^3 801 / 806, 6272 x 3072 x 768 41.1 / 41.0, 25088 x 128 x 1152 14.0 / 13.8.)
    // Nothing is written to registers but m0, which the compiler reserves for itself and warns about: it is said so that no use of its own
    // is scheduled across.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(e < LPA ? aoff[e] : boff[e - LPA]), "s"(buffer) : "m0");
#pragma clang diagnostic pop
  }
  __device__ __forceinline__ void advance() {
    if (--left <= 0) {
      records = 0;  // the loads past the last slab, which the counted waits expect, read nothing
      return;
    }
    pa += 2 * BK;
    pb += 2 * BK;
    c0 += BK;
    if (c0 == C) {
      c0 = 0;
      ++tap;
      if (++kw == g.KW) { kw = 0; ++kh; }
      pa = first + 2 * (int64_t)(mode == OP_CONV_FWD ? (kh * g.W + kw) * g.C : -((kh / g.stride) * g.W + (kw / g.stride)) * g.C);
      at_tap();
    }
  }
};

// All but the newest N of this wave's loads and stores are done, and its LDS reads.
template <int N> __device__ __forceinline__ void wait_newest() {
  static_assert(N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}
__device__ __forceinline__ void slab_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// BM x BN outputs per workgroup of WAVES_M x WAVES_N wavefronts, slabs of BK, STAGES of them in LDS; WPS: wavefronts per SIMD
// that LDS allows (said to the compiler, which otherwise copies the accumulators between the two register files).
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, bool GELU>
__device__ __forceinline__ void conv_gemm_dl_body(const GemmBatch& batch) {
  using Loads = SlabLoads<BM, BN, WAVES_M * WAVES_N, BK>;
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;  // wave tile
  constexpr int MI = WTM / 32, NI = WTN / 32;            // MFMA tiles per wave
  constexpr int ROW = Loads::ROW, STAGE_BYTES = (BM + BN) * ROW, KK = BK / 16, LP = Loads::N;
  static_assert(STAGES >= 2 && STAGES <= 4, "");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[STAGES * STAGE_BYTES];
  const int tile = xcd_block_cyclic((int)blockIdx.x, batch.total_tiles, 8);
  // All of the descriptor in one round: read where they are used, the fields that choose the epilogue, and then those of the one chosen, are a chain of
  // reads behind the last slab (us so / read here: 2304 x 768 x 192 with a mask 5.23 / 5.00, 3000 x 256 x 96 3.77 / 3.53; 38 scalar registers).
  const GemmProb P = read_args(batch.p[__builtin_amdgcn_readfirstlane(find_problem(batch, tile))]);
  const int local = tile - P.tile_begin;
  const int tn = local % P.tiles_n, tm = local / P.tiles_n;
  const int row0 = tm * BM, col0 = tn * BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const unsigned lds = (unsigned)(uintptr_t)(lds_ptr)smem;

  Loads loads;
  loads.start(P, row0, col0, wave, lane);
  static_for<STAGES>([&](auto q) {
#pragma unroll
    for (int e = 0; e < LP; ++e) loads.issue(lds + decltype(q)::value * STAGE_BYTES, wave, e);
    loads.advance();
  });
  v16f_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // fragments: row = base + lane % 32, chunk = 2 * kk + lane / 32
  const int l31 = lane & 31, hi = lane >> 5, swa = Loads::swz(l31);  // rows 32 apart swizzle alike
  const unsigned char* const ra = smem + (wm * WTM + l31) * ROW;
  const unsigned char* const rb = smem + BM * ROW + (wn * WTN + l31) * ROW;
  uint4 fa[2][MI], fb[2][NI];
  auto frag = [&](int q, int kk, int buf, int e) {  // fragment e of MI + NI
    const int x = q * STAGE_BYTES + (((kk * 2 + hi) ^ swa) << 4);
    if (e < MI) fa[buf][e] = *reinterpret_cast<const uint4*>(ra + x + e * 32 * ROW);
    else fb[buf][e - MI] = *reinterpret_cast<const uint4*>(rb + x + (e - MI) * 32 * ROW);
  };
  wait_newest<(STAGES - 1) * LP>();
  slab_barrier();
#pragma unroll
  for (int e = 0; e < MI + NI; ++e) frag(0, 0, 0, e);
  auto step = [&](auto qc) {
    constexpr int q = decltype(qc)::value, next = (q + 1) % STAGES;
    constexpr int MN = MI * NI, RP = (MI + NI + MN - 1) / MN, IP = (LP + MN - 1) / MN;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const bool last = kk == KK - 1;
      if (last) {  // the next slab is whole, and every wave has read this one
        wait_newest<(STAGES - 2) * LP>();
        slab_barrier();
      }
#pragma unroll
      for (int e = 0; e < MN; ++e) {
        acc[e / NI][e % NI] = mfma_bf16(fb[kk & 1][e % NI], fa[kk & 1][e / NI], acc[e / NI][e % NI]);  // transposed: see the epilogue
#pragma unroll
        for (int r = 0; r < RP; ++r)
          if (e * RP + r < MI + NI) frag(last ? next : q, last ? 0 : kk + 1, (kk + 1) & 1, e * RP + r);
#pragma unroll
        for (int r = 0; r < IP; ++r)
          if (last && e * IP + r < LP) loads.issue(lds + q * STAGE_BYTES, wave, e * IP + r);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    loads.advance();
  };
  for (int t = P.K / BK;;) {
    step(std::integral_constant<int, 0>{});
    if (--t == 0) break;
    step(std::integral_constant<int, 1>{});
    if (--t == 0) break;
    if constexpr (STAGES > 2) {
      step(std::integral_constant<int, 2>{});
      if (--t == 0) break;
    }
    if constexpr (STAGES > 3) {
      step(std::integral_constant<int, 3>{});
      if (--t == 0) break;
    }
  }
  wait_newest<0>();  // no load is left that writes LDS when this workgroup gives it back
  conv_epilogue<MI, NI, GELU>(P, acc, row0 + wm * WTM, col0 + wn * WTN, lane);
}
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, int WPS>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64, WPS) void conv_gemm_dl_kernel(const GemmBatch batch) {
  conv_gemm_dl_body<BM, BN, WAVES_M, WAVES_N, BK, STAGES, false>(batch);
}
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, int WPS>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64, WPS) void conv_gelu_dl_kernel(const GemmBatch batch) {
  conv_gemm_dl_body<BM, BN, WAVES_M, WAVES_N, BK, STAGES, true>(batch);
}

// Launches of many tiles: 512 workgroups of four wavefronts, two per CU, walk tiles of 128 x 128 (wave tiles of 64 x 64, slabs of 64,
// two stages of 32 KB).  The loads run through the tiles without a break: behind the last slab of a tile the first ones of the next
// are requested, so that its descriptor, its rows' addresses and its first operands arrive under the products, and the results of one tile
// leave under the products of the next.  What a tile costs beside its products (10 to 15 us for a 256 x 256 tile, of 30 at a
// reduction of 768) is hidden, in short reductions it was most of the time; two workgroups per CU cover for each other's barriers and epilogues.
//   Who takes what: the 64 workgroups of an XCD (blockIdx modulo 8) share an eighth of the tiles of every problem, so that rows are found in the
// XCD's L2, the problems with the longest reductions first.  Every wavefront works the sharing out for itself (RunPlan).
//   Waits: a step needs the slab after it.  Loads and stores count together and in order, and a tile stores the same number of times in
// every wavefront (conv_epilogue_as), so the one wait in which the results are newer than the slab leaves them out.
// us, conv_gemm_kernel / here: see conv_many_tile.
constexpr int RUN_PER_XCD = 64;
constexpr int RUN_SLOT_BITS = 26;  // a tile of an XCD: problem << RUN_SLOT_BITS | number in the XCD's share of it

__device__ __forceinline__ int wave_scan(int v) {  // inclusive sum over the lanes
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast 15, 31
  return v + __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
}
__device__ __forceinline__ int wave_max(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(v, 63);
}

// The tiles a workgroup of conv_gemm_run_kernel takes, in order.  Lane w stands for workgroup w of the XCD and knows how much it has been
// given; problem by problem the workgroups that have less catch up first, the rest is dealt in rounds, what is left over to those that are
// behind.  A tile is worth its reduction and a fixed part.  (Dealt in rounds throughout, whoever has a long tile more gets as many short ones: a
// step of the ResNet-50 shape 22.0 -> 24.7 ms.  Drawn from a counter per XCD, the draws waited in line with the slabs: four of
// 6272 x 768 x 3072 with a residual 134 -> 167 us.)
struct RunPlan {
  int first, caught, base, rounds, extra;  // lane i, problem i: own tiles caught up with (first, how many), start of the rounds, rounds, one of the rest or -1
  int whole, rest;                         // blocks of 64 tiles of the problem, and what is left: a block is eight runs of eight neighbours, one per XCD
  int n, xcd, own, at, pos;                // place in the order

  __device__ __forceinline__ void start(const GemmBatch& batch, int lane) {
    n = batch.n;
    xcd = (int)blockIdx.x & 7;
    own = (int)blockIdx.x >> 3;
    at = pos = 0;
    first = caught = base = rounds = extra = whole = rest = 0;
    int size = 0, cost = 1;
    if (lane < n) {
      const int tiles = (lane + 1 < n ? batch.starts.at[lane + 1] : batch.total_tiles) - batch.starts.at[lane];
      whole = tiles >> 6;
      rest = tiles & 63;
      size = whole * 8 + (rest * (xcd + 1) >> 3) - (rest * xcd >> 3);
      if (n > 1) cost = (min(batch.p[lane].K, 1 << 14) >> 6) + 4;
    }
    if (n == 1) {  // in rounds (100352 x 256 x 64 21.9 -> 20.9 us without the rest)
      rounds = size >> 6;
      extra = own < (size & 63) ? 64 * rounds + own : -1;
      return;
    }
    int given = 0;
    for (int i = 0; i < n; ++i) {
      int m = __builtin_amdgcn_readlane(size, i);
      const int c = __builtin_amdgcn_readlane(cost, i);
      const int most = wave_max(given);
      int take = (int)((float)(most - given) * __builtin_amdgcn_rcpf((float)c));
      const int upto = wave_scan(take), from = upto - take;
      take = max(0, min(take, m - from));
      const int spent = min(m, __builtin_amdgcn_readlane(upto, 63));
      given += take * c;
      m -= spent;
      const int q = m >> 6, r = m & 63;
      const unsigned long long behind = __builtin_amdgcn_ballot_w64(2 * (most - given) >= c);
      auto below = [&](unsigned long long set) { return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(set >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)set, 0u)); };
      const int rank = (behind >> lane) & 1 ? below(behind) : __builtin_popcountll(behind) + below(~behind);
      given += (q + (rank < r)) * c;
      const int f = __builtin_amdgcn_readlane(from, own), t = __builtin_amdgcn_readlane(take, own), k = __builtin_amdgcn_readlane(rank, own);
      if (lane == i) {
        first = f;
        caught = t;
        base = spent;
        rounds = q;
        extra = k < r ? spent + 64 * q + k : -1;
      }
    }
  }
  __device__ __forceinline__ int next() {  // or -1
    for (; at < n; ++at, pos = 0) {
      const int t = __builtin_amdgcn_readlane(caught, at), q = __builtin_amdgcn_readlane(rounds, at), e = __builtin_amdgcn_readlane(extra, at);
      int slot = -1;
      if (pos < t) slot = __builtin_amdgcn_readlane(first, at) + pos;
      else if (pos < t + q) slot = __builtin_amdgcn_readlane(base, at) + (pos - t) * RUN_PER_XCD + own;
      else if (pos == t + q) slot = e;
      if (slot < 0) continue;
      ++pos;
      return at << RUN_SLOT_BITS | slot;
    }
    return -1;
  }
  // Tile of the problem, in the order of its share.
  __device__ __forceinline__ int tile(int pi, int slot) const {
    const int w = __builtin_amdgcn_readlane(whole, pi);
    return slot < 8 * w ? (slot >> 3) * 64 + xcd * 8 + (slot & 7) : w * 56 + slot + (__builtin_amdgcn_readlane(rest, pi) * xcd >> 3);
  }
};

__global__ __launch_bounds__(256, 2) void conv_gemm_run_kernel(const GemmBatch batch) {
  constexpr int BM = 128, BN = 128, WAVES_N = 2, BK = 64, MI = 2, NI = 2, WT = 64;
  using Loads = SlabLoads<BM, BN, 4, BK>;
  constexpr int ROW = Loads::ROW, STAGE_BYTES = (BM + BN) * ROW, KK = BK / 16, LP = Loads::N, STORES = MI * NI * 2;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE_BYTES];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const unsigned lds = (unsigned)(uintptr_t)(lds_ptr)smem;
  RunPlan plan;
  plan.start(batch, lane);
  // Tiles of a problem in panels of about eight columns, row by row inside a panel: the 64 tiles of an XCD in one round then share
  // few rows of either operand (8192^3 1209 -> 1041 us).
  auto place = [&](const GemmProb& P, int j, int& row0, int& col0) {
    const int local = plan.tile(j >> RUN_SLOT_BITS, j & ((1 << RUN_SLOT_BITS) - 1));
    const int tiles_m = (P.M + BM - 1) / BM, panels = (P.tiles_n + 7) >> 3, w = (P.tiles_n + panels - 1) / panels;
    const int panel = local / (tiles_m * w), in = local - panel * tiles_m * w, pw = min(w, P.tiles_n - panel * w), tm = in / pw;
    row0 = tm * BM;
    col0 = (panel * w + in - tm * pw) * BN;
  };
  Loads loads;
  bool more = true;
  int cur = plan.next(), ahead[3] = {-1, -1, -1}, known = 0;  // the tile contracted, those after it whose loads have begun
  if (cur < 0) return;
  auto start = [&](int j) {
    const GemmProb& P = batch.p[j >> RUN_SLOT_BITS];
    int row0, col0;
    place(P, j, row0, col0);
    loads.start(P, row0, col0, wave, lane);
  };
  auto advance = [&]() {
    if (loads.left != 1 || !more) return loads.advance();
    const int j = plan.next();
    if (j < 0) {
      more = false;
      return loads.advance();
    }
    if (known == 0) ahead[0] = j;
    else if (known == 1) ahead[1] = j;
    else ahead[2] = j;
    ++known;
    start(j);
  };
  start(cur);
#pragma unroll
  for (int e = 0; e < LP; ++e) loads.issue(lds, wave, e);
  advance();
#pragma unroll
  for (int e = 0; e < LP; ++e) loads.issue(lds + STAGE_BYTES, wave, e);
  // Addresses of the two stages and of the fragments in them; exchanged behind a tile of an odd number of slabs, so that the loop has
  // constant indices.
  const int l31 = lane & 31, hi = lane >> 5, swa = Loads::swz(l31);
  unsigned at[2], xa[2][KK], xb[2][KK];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    at[q] = lds + q * STAGE_BYTES;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const unsigned x = q * STAGE_BYTES + l31 * ROW + (((kk * 2 + hi) ^ swa) << 4);
      xa[q][kk] = x + wm * WT * ROW;
      xb[q][kk] = x + BM * ROW + wn * WT * ROW;
    }
  }
  uint4 fa[2][MI], fb[2][NI];
  auto frag = [&](int q, int kk, int buf, int e) {
    if (e < MI) fa[buf][e] = *reinterpret_cast<const uint4*>(smem + xa[q][kk] + e * 32 * ROW);
    else fb[buf][e - MI] = *reinterpret_cast<const uint4*>(smem + xb[q][kk] + (e - MI) * 32 * ROW);
  };
  wait_newest<LP>();
  slab_barrier();
  advance();
#pragma unroll
  for (int e = 0; e < MI + NI; ++e) frag(0, 0, 0, e);
  v16f_t acc[MI][NI];
  bool stored = false;  // the results of the tile before are newer than the slab the next wait is for
  auto step = [&](auto qc) {
    constexpr int q = decltype(qc)::value;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const bool last = kk == KK - 1;
      if (last) {
        if (stored) wait_newest<STORES>();
        else wait_newest<0>();
        stored = false;
        slab_barrier();
      }
#pragma unroll
      for (int e = 0; e < MI * NI; ++e) {
        acc[e / NI][e % NI] = mfma_bf16(fb[kk & 1][e % NI], fa[kk & 1][e / NI], acc[e / NI][e % NI]);  // transposed: see the epilogue
        frag(last ? 1 - q : q, last ? 0 : kk + 1, (kk + 1) & 1, e);
        if (last) {
#pragma unroll
          for (int r = 0; r < LP / (MI * NI); ++r) loads.issue(at[q], wave, e * (LP / (MI * NI)) + r);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    advance();
  };
  static_assert(MI + NI == MI * NI && LP % (MI * NI) == 0, "one fragment and the same number of loads beside each product");
  for (;;) {
    const GemmProb& P = batch.p[cur >> RUN_SLOT_BITS];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    bool odd = false;
    for (int t = P.K / BK;;) {
      step(std::integral_constant<int, 0>{});
      if (--t == 0) { odd = true; break; }
      step(std::integral_constant<int, 1>{});
      if (--t == 0) break;
    }
    if (odd) {
      auto exchange = [](unsigned& x, unsigned& y) { const unsigned z = x; x = y; y = z; };
      exchange(at[0], at[1]);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        exchange(xa[0][kk], xa[1][kk]);
        exchange(xb[0][kk], xb[1][kk]);
      }
    }
    int row0, col0;
    place(P, cur, row0, col0);
    conv_epilogue_as<MI, NI, true, 0, false, false>(P, acc, row0 + wm * WT, col0 + wn * WT, lane);
    stored = true;
    if (known == 0) break;
    cur = ahead[0];
    ahead[0] = ahead[1];
    ahead[1] = ahead[2];
    --known;
  }
  wait_newest<0>();  // no load is left that writes LDS when this workgroup gives it back
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, int WPS>
static void launch_dl(const GemmBatch& b, dim3 grid, hipStream_t stream) {
  if (conv_has_gelu(b)) hipLaunchKernelGGL((conv_gelu_dl_kernel<BM, BN, WAVES_M, WAVES_N, BK, STAGES, WPS>), grid, dim3(WAVES_M * WAVES_N * 64), 0, stream, b);
  else hipLaunchKernelGGL((conv_gemm_dl_kernel<BM, BN, WAVES_M, WAVES_N, BK, STAGES, WPS>), grid, dim3(WAVES_M * WAVES_N * 64), 0, stream, b);
}

// Elements between the first tap of the lowest and of the highest row that the gathered operand has.
static int64_t conv_row_span(const GemmProb& p) {
  const ConvGeom& g = p.g;
  if (p.a_mode == OP_PLAIN_K) return (int64_t)(p.M - 1) * p.lda;
  const int64_t images = p.M / (g.OH * g.OW) - 1;
  auto reach = [&](int last) { return p.a_mode == OP_CONV_FWD ? (int64_t)last * g.stride : (int64_t)((last + g.pad) / g.stride - g.pad / g.stride); };
  return ((images * g.H + reach(g.OH - 1)) * g.W + reach(g.OW - 1)) * g.C;
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
  // 32-bit byte offsets: of the weights' rows, of the gathered rows from the lowest one (SlabLoads; they end a slab and a load below 2^32), and
  // inside 32 rows of the result
  const int64_t a_elems = p.a_mode == OP_PLAIN_K ? (int64_t)p.M * p.lda : (int64_t)(p.M / (p.g.OH * p.g.OW) + 1) * p.g.H * p.g.W * p.g.C;
  return a_elems < (1ll << 31) && (int64_t)p.N * p.ldb < (1ll << 31) && conv_row_span(p) < (1ll << 31) - 64 && p.ldo < (1 << 26);
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

// Launches of 512 tiles of 128 x 128 and more: conv_gemm_run_kernel, 256 x 256, or `named`, the tile conv_dl_tile names, by the time each takes:
// full rounds (of 512 tiles for the first, of 768 for conv_gemm_kernel, of 256 for the others) times what a tile costs, fixed and per 1000 of the
// reduction, and the same for the tiles themselves, whose last round has the memory to itself.  Coefficients (us) fitted to 176 products of 512 to
// 5720 tiles, N 72 to 3200, K 64 to 3008, one to eight problems, rms 7 to 10 %.  Over 193 other products of the same ranges what it takes is 2.7 %
// faster than the tiles of conv_dl_tile on average and 1.5 % slower than the best of the five (1.35 for six problems of 64 to 1088 in one launch,
// whose mean says little), conv_gemm_run_kernel alone 5.8 % slower.
// us, conv_gemm_kernel / 256 x 256 / 256 x 128 / 192 x 128 / walked:
//   6272 x 3072 x 768     45.7 / 46.9 / 47.3 / 51.1 / 40.2       32203 x 784 x 384    32.0 / 34.5 / 35.9 / 35.5 / 30.2
//   36029 x 1672 x 2304   346 / 250 / 294 / 304 / 305            7163 x 2384 x 2560   113 / 115 / 108 / 88 / 100
//   113066 x 496 x 1600   222 / 189 / 207 / 229 / 236            66517 x 824 x 1024   151 / 151 / 142 / 137 / 132
// Below 640 walked, where 256 x 256 gains little and loses up to 15 %, but for one round of those (25088 x 512 x 128 12.9 / 12.0 / 14.9 / 16.8 / 14.9); below
// 350 not walked: a slab or five are little to walk with, and conv_gemm_kernel has three workgroups per CU (walked against it, means over the products
// of one problem: K 64 1.23, 128 1.13, 192 1.10, 256 1.02, 320 1.03, 384 0.98, 448 to 512 0.97).
//   100352 x 256 x 64     15.7 / 19.4 / 24.0 / 24.6 / 18.5       14028 x 1656 x 128   16.8 / 21.3 / 22.8 / 23.7 / 20.5
//   17073 x 1304 x 192    19.4 / 23.9 / 25.1 / 25.5 / 22.3       55962 x 296 x 320    24.2 / 27.9 / 26.5 / 26.3 / 25.0
// Residuals, masks, addends and GELUs leave a launch where it was: their reads wait in line with the slabs requested ahead, and conv_gemm_kernel's
// three workgroups per CU read whole rows.  Steps of ResNet-50 and ViT-B/16 shapes, ms per four, with all such launches walked / those of a mean
// reduction of 512 and more / none / no launch walked at all: - / 78.2 / 77.4 / 77.5 and 206.2 / 206.2 / 204.9 / 208.6.
static bool conv_reads_beside(const GemmProb& p) {  // its epilogue reads a tensor, or is a GELU
  return p.aux1 || (p.flags & GF_GELU) || (p.epi == EPI_DGRAD && (p.aux0 || (p.flags & GF_ACCUM)));
}
static int conv_many_tile(const GemmProb* p, int n, int named) {
  double t128 = 0, t256 = 0, wide = 0, t192 = 0, deep = 0;
  for (int i = 0; i < n; ++i) {
    auto count = [&](int bm, int bn) { return (double)((p[i].M + bm - 1) / bm) * ((p[i].N + bn - 1) / bn); };
    if (conv_reads_beside(p[i])) return named;
    t128 += count(128, 128);
    wide += count(256, 256);
    t256 += count(256, 128);
    t192 += count(192, 128);
    deep += count(128, 128) * p[i].K;
  }
  const double k = 1e-3 * deep / t128;
  auto us = [&](double tiles, int slots, double a, double b, double c, double d, double e) {
    return a + std::ceil(tiles / slots) * (b + c * k) + tiles / slots * (d + e * k);
  };
  if (k < 0.64 && wide > 256) return k < 0.35 ? named : DL_RUN;
  const double walked = us(t128, 512, 6.7, -1.3, 4.4, 3.8, 10.8), square = us(wide, 256, 3.7, 2.8, 10.3, 3.1, 13.7);
  const double other = named == DL_256x128   ? us(t256, 256, 4.3, 2.4, 7.0, 1.5, 7.0)
                       : named == DL_192x128 ? us(t192, 256, 3.7, 3.9, 2.3, -0.7, 8.5)
                       : k < 0.35            ? us(t128, 768, 5.3, 0.5, 3.9, 2.0, 23.4)
                                             : 1e30;
  return other < std::min(walked, square) ? named : square < walked ? DL_256x256 : DL_RUN;
}
int conv_launch_tile(const GemmProb* p, int n, int dtype, bool shared) {
  const int named = conv_dl_tile(p, n, dtype, shared);
  int64_t t128 = 0;
  bool wide = false;
  for (int i = 0; i < n; ++i) {
    if (!conv_dl_eligible(p[i], dtype, 64)) return named;
    t128 += (int64_t)((p[i].M + 127) / 128) * ((p[i].N + 127) / 128);
    wide = wide || p[i].N > 64;
  }
  return wide && t128 >= 512 && t128 < (1 << 28) ? conv_many_tile(p, n, named) : named;
}

hipError_t launch_conv_dl(GemmBatch& b, int dtype, int tile, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > GEMM_MAX_PROBS || !conv_gelu_valid(b, dtype)) return hipErrorInvalidValue;
  int bm, bn;
  switch (tile) {
    case DL_256x256: bm = 256; bn = 256; break;
    case DL_256x128: bm = 256; bn = 128; break;
    case DL_192x128: bm = 192; bn = 128; break;
    case DL_128x128: case DL_RUN: bm = 128; bn = 128; break;
    case DL_64x64: case DL_64x64_SHORT: bm = 64; bn = 64; break;
    default: return hipErrorInvalidValue;
  }
  // tiles that take the same time are walked in the same rounds, the longest first
  if (tile == DL_RUN) std::stable_sort(b.p, b.p + b.n, [](const GemmProb& x, const GemmProb& y) { return x.K > y.K; });
  int64_t total = 0;
  for (int i = 0; i < b.n; ++i) {
    GemmProb& p = b.p[i];
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || !conv_dl_eligible(p, dtype, tile == DL_64x64_SHORT ? 32 : 64)) return hipErrorInvalidValue;
    if (tile == DL_RUN && conv_reads_beside(p)) return hipErrorInvalidValue;
    p.splits = 1;
    p.tiles_n = (p.N + bn - 1) / bn;
    p.tile_begin = (int)total;
    total += (int64_t)((p.M + bm - 1) / bm) * p.tiles_n;
    if (total >= (tile == DL_RUN ? 1ll << 28 : 1ll << 31)) return hipErrorInvalidValue;
  }
  b.total_tiles = (int)total;
  tile_starts_set(b.starts, b.p, b.n);
  const dim3 grid((unsigned)total);
  switch (tile) {
    case DL_RUN:
      hipLaunchKernelGGL(conv_gemm_run_kernel, dim3(8 * RUN_PER_XCD), dim3(256), 0, stream, b);
      break;
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
