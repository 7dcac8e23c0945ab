// Convolution / token-wise weight gradients of launches short of workgroups on gfx950.  The tiles of conv_wgrad_kernel, one slab
// ahead and three or four of them to a CU, cover for each other; where a CU has one of them, every slab is a chain of memory
// round trip, LDS write, barrier, read and product.  Here: smaller tiles, and more requests on their way per workgroup.
// Same reduction ranges, same partial sums (kernels.h).  us with the fold, conv_wgrad_kernel / here, at the number of ranges in brackets:
//   bf16  128 x 1152 over 25088 positions [28]  35.3 / 30.7      64 x 576 over 100352 [98]  34.7 / 30.9     256 x 2304 over 6272 [7]  33.4 / 28.5
//         128 x 1152 over 1568 [7]              16.9 / 13.1      512 x 256 over 784 [5]     14.1 / 10.9     24 x 144 over 6272 [14]   16.7 / 14.0
//   fp32  128 x 576 over 800 [5]                24.9 / 11.8      128 x 1152 over 1568 [7]   32.5 / 20.2     64 x 576 over 12544 [28]  36.0 / 27.9
//         24 x 144 over 6272 [16]               33.9 / 13.9      512 x 256 over 784 [5]     25.1 / 13.9     32 x 288 over 3136 [10]   27.6 / 12.2
// Errors against 64 bits: bf16 the same, fp32 half (four partial sums per range).
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "kernels.h"
#include "mfma_frag.h"

namespace cdp {

namespace {

__device__ uint4 g_wgrad_zero[4];  // zero-initialised; source of structural zeros

typedef __attribute__((address_space(3))) void* lds_void;
typedef __attribute__((address_space(3))) frag_v4s* lds_v4s;

}  // namespace

// bf16: tiles of 64 x 128 of the weight matrix, operands straight into LDS (rows of a slab as they lie in memory, read back transposed), three
// slabs of 64 positions, two of them in flight.  One instruction fills 1 KB of LDS lane by lane, so rows are unpadded
// and the loading lane picks the 16-byte piece that belongs in its slot: the four rows that a transposing read takes together
// are four pieces apart.  The stages are separate arrays, the waits builtins and the last slabs straight-line code because the
// compiler otherwise waits for every request at the first fragment read.
__global__ __launch_bounds__(256, 2) void conv_wgrad_dl_kernel(const GemmBatch batch) {
  constexpr int TO = 64, TC = 128, WAVES_O = 2, WAVES_C = 2, BK = 64, STAGES = 3, NW = WAVES_O * WAVES_C;
  constexpr int WTO = TO / WAVES_O, WTC = TC / WAVES_C, MI = WTO / 32, NI = WTC / 32;
  constexpr int PD = TO * 2, PX = TC * 2;             // bytes of a staged row
  constexpr int CPD = PD / 16, CPX = PX / 16;         // chunks of a staged row
  constexpr int RBD = 64 / CPD, RBX = 64 / CPX;       // rows of a 1 KB block
  constexpr int LPD = BK / RBD / NW, LPX = BK / RBX / NW;  // blocks a wave loads per slab
  static_assert(LPD * RBD * NW == BK && LPX * RBX * NW == BK, "rows of a slab are dealt to the waves in 1 KB blocks");
  constexpr int XROWS = LPX * RBX;                    // x rows a wave loads per slab
  constexpr int XG = 64 / XROWS;                      // slabs whose x rows the 64 lanes decode at once
  constexpr int XOFF = BK * PD;                       // x behind dy in a stage
  constexpr int SB = BK * (TO + TC) * 2;
  __shared__ __attribute__((aligned(1024))) unsigned char st0[SB];
  __shared__ __attribute__((aligned(1024))) unsigned char st1[SB];
  __shared__ __attribute__((aligned(1024))) unsigned char st2[SB];

  const int tile = xcd_block_cyclic((int)blockIdx.x, batch.total_tiles, batch.xcd_run);
  const GemmProb& P = batch.p[find_problem(batch, tile)];
  const int row_tiles = (P.M + TO - 1) / TO, local = tile - P.tile_begin;
  const int tc = local % P.tiles_n, to = local / P.tiles_n % row_tiles, split = local / P.tiles_n / row_tiles;
  const int o0 = to * TO, col0 = tc * TC;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wo = wave / WAVES_C, wc = wave % WAVES_C;
  const int Cout = P.M, Ncol = P.N, Mpos = P.K;
  const ConvGeom g = P.g;
  const bool gather = P.b_mode == OP_CONV_WGRAD;

  // the range: whole slabs of 64 positions, as the register-staged kernel cuts it
  constexpr int RS = 64;
  const int nslab_total = (Mpos + RS - 1) / RS, per = (nslab_total + P.splits - 1) / P.splits;
  const int m_begin = min(split * per * RS, Mpos), m_end = min(m_begin + per * RS, Mpos);
  const int nslab = (m_end - m_begin + BK - 1) / BK;

  const uint16_t* const zero = reinterpret_cast<const uint16_t*>(g_wgrad_zero);
  // dy: row wave * LPD * RBD + i * RBD + drow of the slab, slot lane % CPD of it
  auto swz = [](int r, int cpr) { return cpr >= 16 ? (r & 3) << 2 : ((r >> 1) & 1) << 2; };
  const int drow = wave * LPD * RBD + lane / CPD;
  const int dcol = o0 + ((lane % CPD) ^ swz(drow, CPD)) * 8;
  const bool dok = dcol < Cout;
  const uint16_t* dptr = static_cast<const uint16_t*>(P.A) + (int64_t)(m_begin + drow) * P.lda + dcol;
  int dq = m_begin + drow;
  // x: the lane's column (tap, channel) never changes; row wave * XROWS + i * RBX + lane / CPX
  const int xrow = wave * XROWS + lane / CPX;
  const int xcol = col0 + ((lane % CPX) ^ swz(xrow, CPX)) * 8;
  const bool xok = xcol < Ncol;
  int x_kh = 0, x_kw = 0, x_delta = xcol;
  if (gather && xok) {
    const int tap = xcol / g.C, c = xcol - tap * g.C;
    x_kh = tap / g.KW;
    x_kw = tap - x_kh * g.KW;
    x_delta = (x_kh * g.W + x_kw) * g.C + c;
  }
  const uint16_t* const Xp = static_cast<const uint16_t*>(P.B) + x_delta;
  int xq = m_begin + xrow;
  int dec_base = 0, dec_hw = 0;  // lane l: row l % XROWS of the wave's x rows, slab l / XROWS of the current group
  auto decode = [&](int s) {     // s: first slab of a group
    const int m = m_begin + (s + lane / XROWS) * BK + wave * XROWS + lane % XROWS;
    const int b = m / (g.OH * g.OW), rem = m - b * (g.OH * g.OW);
    const int oh = rem / g.OW, ow = rem - oh * g.OW;
    const int ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
    dec_base = ((b * g.H + ih0) * g.W + iw0) * g.C;
    dec_hw = m < m_end ? (int)(((unsigned)(ih0 & 0xffff) << 16) | (unsigned)(iw0 & 0xffff)) : (int)0x80008000u;
  };
  int sg = 0, snext = 0;  // slab inside the decoded group; next slab to request
  auto issue = [&](unsigned char* stage) {
#pragma unroll
    for (int i = 0; i < LPD; ++i) {
      const uint16_t* p = dok && dq + i * RBD < m_end ? dptr + (int64_t)(i * RBD) * P.lda : zero;
      __builtin_amdgcn_global_load_lds(p, (lds_void)(stage + (wave * LPD + i) * 1024), 16, 0, 0);
    }
    dptr += (int64_t)BK * P.lda;
    dq += BK;
    if (gather) {
      if (sg == 0) decode(snext);
#pragma unroll
      for (int i = 0; i < LPX; ++i) {
        const int src = (sg * XROWS + i * RBX + lane / CPX) * 4;
        const int base = __builtin_amdgcn_ds_bpermute(src, dec_base), hw = __builtin_amdgcn_ds_bpermute(src, dec_hw);
        const int ih = (hw >> 16) + x_kh, iw = (int)(short)(hw & 0xffff) + x_kw;
        const bool ok = xok && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
        const uint16_t* p = ok ? Xp + base : zero;
        __builtin_amdgcn_global_load_lds(p, (lds_void)(stage + XOFF + (wave * LPX + i) * 1024), 16, 0, 0);
      }
      sg = sg + 1 == XG ? 0 : sg + 1;
      ++snext;
    } else {
#pragma unroll
      for (int i = 0; i < LPX; ++i) {
        const int m = xq + i * RBX;
        const uint16_t* p = xok && m < m_end ? Xp + (int64_t)m * P.ldb : zero;
        __builtin_amdgcn_global_load_lds(p, (lds_void)(stage + XOFF + (wave * LPX + i) * 1024), 16, 0, 0);
      }
      xq += BK;
    }
  };

  v16f_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  float bsum[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) bsum[i] = 0.f;

  // fragments (frag_tr_bf16 on swizzled rows): row 8 * (lane / 32) + rho / 4, columns r0 + 16 * ((lane / 16) & 1) + 4 * (rho & 3)
  const int rho = lane & 15, frow = 8 * (lane >> 5) + (rho >> 2);
  const int flow = 2 * ((lane >> 4) & 1) + ((rho & 3) >> 1), fbyte = (rho & 1) * 8;
  int offd[MI], offx[NI];
#pragma unroll
  for (int i = 0; i < MI; ++i) offd[i] = frow * PD + ((((wo * WTO + i * 32) / 8 + flow) ^ swz(frow, CPD)) << 4) + fbyte;
#pragma unroll
  for (int j = 0; j < NI; ++j) offx[j] = XOFF + frow * PX + ((((wc * WTC + j * 32) / 8 + flow) ^ swz(frow, CPX)) << 4) + fbyte;
  auto frag = [&](const unsigned char* p, int pitch) {
    union { frag_v4s v[2]; uint4 u; } r;
    r.v[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p));
    r.v[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + 4 * pitch));
    return r.u;
  };
  const bool do_beta = tc == 0 && P.aux3 != nullptr && wc == 0;
  auto colsum = [&](uint4 a) {  // the eight positions that a lane holds of its column
    auto pair = [&](uint32_t w) { return __uint_as_float(w << 16) + __uint_as_float(w & 0xffff0000u); };
    return (pair(a.x) + pair(a.y)) + (pair(a.z) + pair(a.w));
  };
  auto contract = [&](const unsigned char* stage) {
    constexpr int KK = BK / 16;
    uint4 a[2][MI], b[2][NI];
    auto frags = [&](int kk, int buf) {
#pragma unroll
      for (int i = 0; i < MI; ++i) a[buf][i] = frag(stage + offd[i] + kk * 16 * PD, PD);
#pragma unroll
      for (int j = 0; j < NI; ++j) b[buf][j] = frag(stage + offx[j] + kk * 16 * PX, PX);
    };
    frags(0, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk + 1 < KK) frags(kk + 1, (kk + 1) & 1);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = mfma_bf16(a[kk & 1][i], b[kk & 1][j], acc[i][j]);
      if (do_beta) {
#pragma unroll
        for (int i = 0; i < MI; ++i) bsum[i] += colsum(a[kk & 1][i]);
      }
    }
  };

  unsigned char* const st[3] = {st0, st1, st2};
  auto wait_slabs = [&](auto n) {  // all but the newest n slabs
    constexpr int N = decltype(n)::value * (LPD + LPX);
    static_assert(N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));  // vmcnt(N) lgkmcnt(0)
  };
  auto barrier = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
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
  if (nslab >= STAGES - 1) {
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
    static_for<STAGES>([&](auto k) {
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

  // acc rows = o, cols = (tap, c); plain stores into this range's partial buffer (an empty range writes zeros)
  float* __restrict__ part = static_cast<float*>(P.out) + (int64_t)split * Cout * Ncol;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = o0 + wo * WTO + i * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
      if (r >= Cout) continue;
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int c = col0 + wc * WTC + j * 32 + (lane & 31);
        if (c < Ncol) part[(int64_t)r * Ncol + c] = acc[i][j][v];
      }
    }
  if (do_beta) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const float s = bsum[i] + __shfl_xor(bsum[i], 32, 64);
      const int r = o0 + wo * WTO + i * 32 + (lane & 31);
      if (lane < 32 && r < Cout) static_cast<float*>(P.aux3)[(int64_t)split * Cout + r] = s;
    }
  }
}

// fp32, launches short of workgroups: 32 x 32 tiles of the weight matrix whose four wavefronts take every fourth group of 32 positions of
// the range with both operands straight from memory (a load is 32 neighbouring channels of two positions, 16 products of loads
// are on their way ahead of the products that use them), and add their tiles through LDS in wavefront order.
__global__ __launch_bounds__(256, 2) void conv_wgrad_few_kernel(const GemmBatch batch) {
  constexpr int MB = 32;  // positions per group; ranges are whole groups, as conv_wgrad_kernel cuts them
  __shared__ float red[4 * 16 * 64];
  __shared__ float bred[4 * 32];
  const int tile = xcd_block_cyclic((int)blockIdx.x, batch.total_tiles, batch.xcd_run);
  const GemmProb& P = batch.p[find_problem(batch, tile)];
  const int row_tiles = (P.M + 31) / 32, local = tile - P.tile_begin;
  const int tc = local % P.tiles_n, to = local / P.tiles_n % row_tiles, split = local / P.tiles_n / row_tiles;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l31 = lane & 31, hi = lane >> 5;
  const int o0 = to * 32, col0 = tc * 32, Cout = P.M, Ncol = P.N;
  const ConvGeom g = P.g;
  const bool gather = P.b_mode == OP_CONV_WGRAD;
  const int nslab_total = (P.K + MB - 1) / MB, per = (nslab_total + P.splits - 1) / P.splits;
  const int m_begin = min(split * per * MB, P.K), m_end = min(m_begin + per * MB, P.K);
  // rows and columns past the end repeat the last one: they only reach outputs that are not stored
  const float* const Dp = static_cast<const float*>(P.A) + min(o0 + l31, Cout - 1);
  const int xcol = min(col0 + l31, Ncol - 1);
  int x_kh = 0, x_kw = 0, x_delta = xcol;
  if (gather) {
    const int tap = xcol / g.C, c = xcol - tap * g.C;
    x_kh = tap / g.KW;
    x_kw = tap - x_kh * g.KW;
    x_delta = (x_kh * g.W + x_kw) * g.C + c;
  }
  const float* const Xp = static_cast<const float*>(P.B);
  // products of group `mc`: element i is position mc + 2 i + hi; what is outside the range or the image is zero
  auto load = [&](int mc, float (&a)[16], float (&b)[16]) {
    const int md = min(mc + l31, P.K - 1);  // decoded by lane
    int base = 0, hw = 0;
    if (gather) {
      const int s = md / (g.OH * g.OW), rem = md - s * (g.OH * g.OW);
      const int oh = rem / g.OW, ow = rem - oh * g.OW;
      const int ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
      base = ((s * g.H + ih0) * g.W + iw0) * g.C;
      hw = (int)(((unsigned)(ih0 & 0xffff) << 16) | (unsigned)(iw0 & 0xffff));
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = Dp[(int64_t)min(mc + 2 * i + hi, P.K - 1) * P.lda];
    if (gather) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int bj = __shfl(base, 2 * i + hi, 64), hj = __shfl(hw, 2 * i + hi, 64);
        const int ih = (hj >> 16) + x_kh, iw = (int)(short)(hj & 0xffff) + x_kw;
        const bool ok = (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
        const float x = Xp[ok ? bj + x_delta : 0];
        b[i] = ok ? x : 0.f;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) b[i] = Xp[(int64_t)min(mc + 2 * i + hi, P.K - 1) * P.ldb + xcol];
    }
    if (mc + MB > m_end) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (mc + 2 * i + hi >= m_end) a[i] = b[i] = 0.f;
    }
  };
  v16f_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  float bsum = 0.f;
  auto product = [&](const float (&a)[16], const float (&b)[16]) {
#pragma unroll
    for (int i = 0; i < 16; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; ++i) bsum += a[i];
  };
  float a0[16], b0[16], a1[16], b1[16];
  int m = m_begin + wave * MB;
  if (m < m_end) load(m, a0, b0);
  for (; m < m_end; m += 8 * MB) {
    if (m + 4 * MB < m_end) load(m + 4 * MB, a1, b1);
    product(a0, b0);
    if (m + 4 * MB >= m_end) break;
    if (m + 8 * MB < m_end) load(m + 8 * MB, a0, b0);
    product(a1, b1);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = acc[v];
  bsum += __shfl_xor(bsum, 32, 64);
  if (hi == 0) bred[wave * 32 + l31] = bsum;
  __syncthreads();
  float* __restrict__ part = static_cast<float*>(P.out) + (int64_t)split * Cout * Ncol;
  const int c = col0 + l31;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int v = wave * 4 + q, r = o0 + wave * 8 + hi * 4 + q;
    const float s = (red[v * 64 + lane] + red[(16 + v) * 64 + lane]) + (red[(32 + v) * 64 + lane] + red[(48 + v) * 64 + lane]);
    if (r < Cout && c < Ncol) part[(int64_t)r * Ncol + c] = s;
  }
  if (tc == 0 && P.aux3 != nullptr && threadIdx.x < 32 && o0 + l31 < Cout)
    static_cast<float*>(P.aux3)[(int64_t)split * Cout + o0 + l31] = (bred[l31] + bred[32 + l31]) + (bred[64 + l31] + bred[96 + l31]);
}

// As many workgroups as are resident at once (bf16: 72 KB of LDS, two per CU; fp32 three), and in fp32 a third more, but where the
// other kernel has tiles of 64 rows and ranges are one or two groups of positions, so that two or three of the four wavefronts here have nothing to
// do.  us past the line, conv_wgrad_kernel / here: bf16 1008 workgroups (256 x 2304 over 6272 [14]) 30.2 / 32.3, 980 (64 x 576 over 100352 [196])
// 31.9 / 34.0; fp32 2304 (512 x 4608 over 98 [1]) 26.6 / 27.6, 2048 (1024 x 512 over 200 [4]) 17.3 / 17.8, 7632 (128 x 1152 over 25088 [53]) 90 / 147.
// Short ranges: 884 (104 x 7056 over 25 [1]) 10.6 / 13.7, 832 (40 x 3312 over 98 [4]) 10.0 / 12.2, 640 (64 x 5112 over 49 [2]) 10.4 / 10.2, of 128 rows 952
// (216 x 1080 over 200 [4]) 16.9 / 13.3; longer ones 832 (64 x 1656 over 2450 [8]) 28.5 / 21.8.
bool conv_wgrad_small_wanted(const GemmBatch& b, int dtype) {
  const bool bf16 = dtype == DT_BF16;
  const int to = bf16 ? 64 : 32, tc = bf16 ? 128 : 32;
  int64_t total = 0;
  bool idle = !bf16;  // every problem leaves wavefronts idle
  for (int i = 0; i < b.n; ++i) {
    const GemmProb& p = b.p[i];
    if (bf16 && ((reinterpret_cast<uintptr_t>(p.A) | reinterpret_cast<uintptr_t>(p.B)) & 15)) return false;  // 16 bytes per request
    total += (int64_t)((p.M + to - 1) / to) * ((p.N + tc - 1) / tc) * p.splits;
    idle = idle && p.M < 128 && ((int64_t)p.K + 31) / 32 <= 2 * (int64_t)p.splits;
  }
  return total <= (bf16 ? 512 : idle ? 768 : 1024);
}

hipError_t launch_conv_wgrad_small(GemmBatch& b, int dtype, hipStream_t stream) {
  const bool bf16 = dtype == DT_BF16;
  const int to = bf16 ? 64 : 32, tc = bf16 ? 128 : 32;
  int total = 0;
  for (int i = 0; i < b.n; ++i) {
    GemmProb& p = b.p[i];
    p.tiles_n = (p.N + tc - 1) / tc;
    p.tile_begin = total;
    total += ((p.M + to - 1) / to) * p.tiles_n * p.splits;
  }
  b.total_tiles = total;
  tile_starts_set(b.starts, b.p, b.n);
  b.xcd_run = b.n == 1 ? 32 : 16;  // (below 256 or 128 workgroups the order is as listed)
  if (bf16) hipLaunchKernelGGL(conv_wgrad_dl_kernel, dim3(total), dim3(256), 0, stream, b);
  else hipLaunchKernelGGL(conv_wgrad_few_kernel, dim3(total), dim3(256), 0, stream, b);
  return hipGetLastError();
}

}  // namespace cdp
