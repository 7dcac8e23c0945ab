// HBM-bound and latency-bound kernels of the CDP hot path: micro-batch staging, the
// softmax cross-entropy head (one wavefront per row), bias-gradient column sums, the
// SGD update with re-layout of the new weight version (Eq. (CDP): theta_{t+1} =
// theta_t - gamma/N * sum_i grad f_i), pooling.
#include "elem.h"
#include "kernels.h"
#include "sgd_step.h"

namespace cdp {

#define CDP_DISPATCH(dtype, CALL)                 \
  do {                                            \
    if ((dtype) == DT_BF16) { using T = uint16_t; CALL; } \
    else { using T = float; CALL; }               \
  } while (0)

static inline int blocks_for(int64_t n, int per_block, int cap = 1 << 20) {
  int64_t b = (n + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

// ---------------------------------------------------------------------------------
template <typename T>
__global__ void stage_input_kernel(const float* __restrict__ x, const int32_t* __restrict__ y, T* __restrict__ xo,
                                   int32_t* __restrict__ yo, float* __restrict__ loss_slot, int n_slots, int rows, int64_t n) {
  if (blockIdx.x == 0 && (int)threadIdx.x < n_slots) loss_slot[threadIdx.x] = 0.f;  // the head adds row losses into them
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    st_f32<T>(xo, i, x[i]);
    if (i < rows) yo[i] = y[i];
  }
}

hipError_t launch_stage_input(const float* x, const int32_t* y, void* x_out, int32_t* y_out, float* loss_slot, int n_slots,
                              int rows, int64_t per_row, int dtype, hipStream_t stream) {
  int64_t n = (int64_t)rows * per_row;
  if (n < rows || n_slots < 1 || n_slots > 256) return hipErrorInvalidValue;
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((stage_input_kernel<T>), dim3(blocks_for(n, 256 * 4, 4096)), dim3(256), 0, stream,
                                         x, y, static_cast<T*>(x_out), y_out, loss_slot, n_slots, rows, n));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// One wavefront per row: max, sum of exponentials, loss and gradient; four rows per
// workgroup.  Row losses are added (fp32 atomic) into *loss_out, which the staging kernel
// of the same micro-batch has set to zero.
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

constexpr int CE_ROW_REGS = 16;  // rows of up to 1024 classes are held in registers
template <typename T>
__global__ __launch_bounds__(256) void ce_head_kernel(const float* __restrict__ logits, const int32_t* __restrict__ labels,
                                                      T* __restrict__ dlogits, float* __restrict__ loss_out, int B, int C,
                                                      int rows_per_slot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x * 4 + wave;
  if (row >= B) return;
  const float invB = 1.0f / (float)B;
  const float* z = logits + (int64_t)row * C;
  const int y = labels[row];
  if (C <= 64 * CE_ROW_REGS) {
    // The row lives in registers: all of a lane's reads are in flight together and every exponential is taken
    // once.  Same operations in the same order as the loops below, so the results are the same bits.
    float zc[CE_ROW_REGS];
#pragma unroll
    for (int k = 0; k < CE_ROW_REGS; ++k) {
      const int c = lane + 64 * k;
      zc[k] = c < C ? z[c] : -INFINITY;
    }
    const float zy = lane == 0 ? z[y] : 0.f;
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < CE_ROW_REGS; ++k) m = fmaxf(m, zc[k]);
    m = wave_max(m);
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < CE_ROW_REGS; ++k) {
      zc[k] = expf(zc[k] - m);
      if (lane + 64 * k < C) s += zc[k];
    }
    s = wave_sum(s);
    const float inv = 1.0f / s;
#pragma unroll
    for (int k = 0; k < CE_ROW_REGS; ++k) {
      const int c = lane + 64 * k;
      if (c < C) st_f32<T>(dlogits, (int64_t)row * C + c, (zc[k] * inv - (c == y ? 1.f : 0.f)) * invB);
    }
    if (lane == 0)
      atomicAdd(reinterpret_cast<int*>(loss_out) + row / rows_per_slot, __float2int_rn(((m + logf(s)) - zy) / (float)rows_per_slot * LOSS_SCALE));
    return;
  }
  float m = -INFINITY;
  for (int c = lane; c < C; c += 64) m = fmaxf(m, z[c]);
  m = wave_max(m);
  float s = 0.f;
  for (int c = lane; c < C; c += 64) s += expf(z[c] - m);
  s = wave_sum(s);
  const float inv = 1.0f / s;
  for (int c = lane; c < C; c += 64) {
    float p = expf(z[c] - m) * inv;
    st_f32<T>(dlogits, (int64_t)row * C + c, (p - (c == y ? 1.f : 0.f)) * invB);
  }
  if (lane == 0)
    atomicAdd(reinterpret_cast<int*>(loss_out) + row / rows_per_slot, __float2int_rn(((m + logf(s)) - z[y]) / (float)rows_per_slot * LOSS_SCALE));
}

hipError_t launch_ce_head(const float* logits, const int32_t* labels, void* dlogits, float* loss_out, int B, int C,
                          int rows_per_slot, int dtype, hipStream_t stream) {
  if (rows_per_slot <= 0 || B % rows_per_slot != 0) return hipErrorInvalidValue;
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((ce_head_kernel<T>), dim3((B + 3) / 4), dim3(256), 0, stream, logits, labels,
                                         static_cast<T*>(dlogits), loss_out, B, C, rows_per_slot));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Column sums: block = 64 columns x 4 row lanes; grid.y splits the rows; fp32 atomics.
constexpr int COLSUM_ROWS_PER_BLOCK = 512;
template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(const ColsumBatch b) {
  __shared__ float red[4][64];
  const ColsumProb& P = b.p[blockIdx.z];
  const int col = blockIdx.x * 64 + (threadIdx.x & 63);
  const int rl = threadIdx.x >> 6;
  const int r0 = blockIdx.y * COLSUM_ROWS_PER_BLOCK;
  if (blockIdx.x * 64 >= P.cols || r0 >= P.rows) return;
  const int r1 = min(P.rows, r0 + COLSUM_ROWS_PER_BLOCK);
  float s = 0.f;
  if (col < P.cols)
    for (int r = r0 + rl; r < r1; r += 4) s += ld_f32<T>(static_cast<const T*>(P.src), (int64_t)r * P.ld + col);
  red[rl][threadIdx.x & 63] = s;
  __syncthreads();
  if (rl == 0 && col < P.cols) atomicAdd(P.out + col, red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x]);
}

hipError_t launch_colsum_batch(const ColsumBatch& b, int dtype, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > COLSUM_MAX_PROBS) return hipErrorInvalidValue;
  int gx = 1, gy = 1;
  for (int i = 0; i < b.n; ++i) {
    gx = max(gx, (b.p[i].cols + 63) / 64);
    gy = max(gy, (b.p[i].rows + COLSUM_ROWS_PER_BLOCK - 1) / COLSUM_ROWS_PER_BLOCK);
  }
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((colsum_kernel<T>), dim3(gx, gy, b.n), dim3(256), 0, stream, b));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Vector parameters of a stage (bias, gamma, beta of all its layers) in one launch: block y
// picks the vector, blocks x stride over its elements.
__global__ void update_vec_kernel(const VecUpdateBatch b, SgdParams sgd) {
  const VecUpdate& u = b.v[blockIdx.y];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < u.n; i += (int64_t)gridDim.x * blockDim.x) {
    float w = u.master[i];
    if (sgd.apply) {
      w = sgd_step(w, u.G[i], u.V ? u.V + i : nullptr, sgd);
      u.master[i] = w;
    }
    u.G[i] = 0.f;
    u.copy[i] = w;
  }
}
hipError_t launch_update_vec_batch(const VecUpdateBatch& b, SgdParams sgd, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > VEC_UPDATE_MAX) return hipErrorInvalidValue;
  int64_t longest = 1;
  for (int i = 0; i < b.n; ++i) {
    if (b.v[i].n <= 0 || !b.v[i].master || !b.v[i].G || !b.v[i].copy) return hipErrorInvalidValue;
    longest = b.v[i].n > longest ? b.v[i].n : longest;
  }
  hipLaunchKernelGGL(update_vec_kernel, dim3(blocks_for(longest, 256, 1024), b.n), dim3(256), 0, stream, b, sgd);
  return hipGetLastError();
}

// W[O][T][C]: tile 64(o) x 64(c) for one tap t.  Reads G and master coalesced along c,
// writes master / wf / wp coalesced along c and wt coalesced along o via an LDS transpose.
// The tiles of all matrices of a stage form one flat list.
template <typename T>
__global__ __launch_bounds__(256) void repack_kernel(const RepackBatch batch) {
  __shared__ float tile[64][65];
  const RepackArgs& a = batch.a[tile_starts_find(batch.starts, batch.n, (int)blockIdx.x)];
  int local = (int)blockIdx.x - a.tile_begin;
  const int tiles_c = (a.C + 63) / 64, tiles_o = (a.O + 63) / 64;
  const int c0 = (local % tiles_c) * 64;
  local /= tiles_c;
  const int o0 = (local % tiles_o) * 64, t = local / tiles_o;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  T* wf = static_cast<T*>(a.wf);
  T* wt = static_cast<T*>(a.wt);
  T* wp = static_cast<T*>(a.wp);
  // all loads of the tile first (the stores below may alias them for all the compiler knows: interleaved, the 16
  // rows of a thread would be 16 memory round trips one after the other)
  float wv[16], gv[16], vv[16], gam[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int o = o0 + ty + i * 4, c = c0 + tx;
    wv[i] = gv[i] = vv[i] = 0.f;
    gam[i] = 1.f;
    if (o < a.O && c < a.C) {
      const int64_t idx = ((int64_t)o * a.T + t) * a.C + c;
      wv[i] = a.master[idx];
      if (a.sgd.apply) {
        gv[i] = a.G[idx];
        if (a.V) vv[i] = a.V[idx];
      }
      if (a.gamma) gam[i] = a.gamma[o];
    }
  }
  // vmcnt(0), here and for all of them: waited for under the condition of its own stores, every row would wait again, and for
  // the stores of the rows before it (17 tiles 14.2 us so / 11.2 us, 1472 tiles 33.0 / 26.6)
  __builtin_amdgcn_s_waitcnt(0x0f70);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int o = o0 + ty + i * 4, c = c0 + tx;
    float v = 0.f;
    if (o < a.O && c < a.C) {
      const int64_t idx = ((int64_t)o * a.T + t) * a.C + c;
      float w = wv[i];
      if (a.sgd.apply) {
        w = sgd_step(w, gv[i], a.V ? &vv[i] : nullptr, a.sgd);
        a.master[idx] = w;
        if (a.V) a.V[idx] = vv[i];
      }
      if (a.zero_g) a.G[idx] = 0.f;
      if (wp) st_f32<T>(wp, idx, w);
      v = a.gamma ? gam[i] * w : w;
      st_f32<T>(wf, (int64_t)o * a.ldf + (int64_t)t * a.C + c, v);
    }
    tile[ty + i * 4][tx] = v;
  }
  __syncthreads();
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int c = c0 + ty + i * 4, o = o0 + tx;
    if (o < a.O && c < a.C) st_f32<T>(wt, ((int64_t)c * a.T + t) * a.O + o, tile[tx][ty + i * 4]);
  }
}

hipError_t launch_repack_batch(RepackBatch& b, int dtype, hipStream_t stream) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > REPACK_MAX) return hipErrorInvalidValue;
  int64_t total = 0;
  for (int i = 0; i < b.n; ++i) {
    RepackArgs& a = b.a[i];
    if (a.O <= 0 || a.C <= 0 || a.T <= 0) return hipErrorInvalidValue;
    a.tile_begin = (int)total;
    total += (int64_t)((a.C + 63) / 64) * ((a.O + 63) / 64) * a.T;
    if (total >= (1ll << 31)) return hipErrorInvalidValue;
  }
  tile_starts_set(b.starts, b.a, b.n);
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((repack_kernel<T>), dim3((unsigned)total), dim3(256), 0, stream, b));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// One 16-byte chunk of a column row per thread.  Inside a filter row kh the index k = (kw, c)
// runs over KW*C elements that are contiguous in x, so (kh, offset in the filter row) is
// stepped along the chunk and each filter row needs one bounds test on its offset range.
template <typename T>
__global__ void im2col_kernel(const T* __restrict__ x, T* __restrict__ col, int64_t n_chunks, ConvGeom g, int kpad) {
  constexpr int VEC = 16 / sizeof(T);
  const int cpr = kpad / VEC, RW = g.KW * g.C, K = g.KH * RW;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_chunks; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = i / cpr;
    const int k0 = (int)(i - m * cpr) * VEC;
    const int b = (int)(m / (g.OH * g.OW));
    const int rem = (int)(m - (int64_t)b * (g.OH * g.OW));
    const int oh = rem / g.OW, ow = rem - oh * g.OW;
    const int ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
    // offsets r in [r_lo, r_hi) of a filter row fall inside the image
    const int r_lo = max(0, -iw0) * g.C, r_hi = min(g.KW, g.W - iw0) * g.C;
    int kh = k0 / RW, r = k0 - kh * RW;
    const T* row = x + (((int64_t)b * g.H + ih0 + kh) * g.W + iw0) * g.C;  // x[b][ih0+kh][iw0][0]
    union { uint4 v; T e[VEC]; } out;
    out.v = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      if (k0 + e < K) {
        const int ih = ih0 + kh;
        if (ih >= 0 && ih < g.H && r >= r_lo && r < r_hi) out.e[e] = row[r];
        if (++r == RW) { r = 0; ++kh; row += (int64_t)g.W * g.C; }
      }
    }
    *reinterpret_cast<uint4*>(col + i * VEC) = out.v;
  }
}
// The same matrix, one workgroup per output row (b, oh): the KH image rows the row's windows touch are copied
// into LDS in 16-byte pieces, with zeros to the left and right of each row and in place of rows outside the
// image, so that every element of a column row is one LDS read at kh * LROW + LOFF + ow * stride * C + r with
// no bounds test; the chunks leave as 16-byte stores.  (Read straight from memory, a chunk is eight 2-byte
// loads and a handful of integer divisions per thread: 72 us for the 7 x 7 stem of a 32 x 224 x 224 micro-batch,
// a third of the rate at which its 128 MB can be written.)
// For image rows that are whole 16-byte pieces (W * C a multiple of the vector width, aligned base).
template <typename T>
__global__ __launch_bounds__(256) void im2col_rows_kernel(const T* __restrict__ x, T* __restrict__ col, ConvGeom g, int kpad, int LROW, int LOFF) {
  constexpr int VEC = 16 / sizeof(T);
  extern __shared__ __attribute__((aligned(16))) unsigned char im2col_smem[];
  T* rows = reinterpret_cast<T*>(im2col_smem);  // [KH][LROW]; image element (iw, c) of row kh at kh * LROW + LPADV + iw * C + c
  const int b = blockIdx.x / g.OH, oh = blockIdx.x - b * g.OH;
  const int ih0 = oh * g.stride - g.pad;
  const int WC = g.W * g.C, RW = g.KW * g.C, K = g.KH * RW;
  const int LPADV = LOFF + g.pad * g.C;  // a multiple of VEC
  const int cprow = LROW / VEC;          // 16-byte pieces per LDS row
  for (int id = threadIdx.x; id < g.KH * cprow; id += 256) {
    const int kh = id / cprow, pc = (id - kh * cprow) * VEC;
    const int ih = ih0 + kh, src = pc - LPADV;  // element offset in the image row
    uint4 v = make_uint4(0, 0, 0, 0);
    if (ih >= 0 && ih < g.H && src >= 0 && src < WC) v = *reinterpret_cast<const uint4*>(x + ((int64_t)b * g.H + ih) * WC + src);
    *reinterpret_cast<uint4*>(rows + kh * LROW + pc) = v;
  }
  __syncthreads();
  const int cpr = kpad / VEC;
  T* out = col + (int64_t)blockIdx.x * g.OW * kpad;
  for (int q = threadIdx.x; q < g.OW * cpr; q += 256) {
    const int ow = q / cpr, k0 = (q - ow * cpr) * VEC;
    int kh = k0 / RW, r = k0 - kh * RW;
    const T* src = rows + kh * LROW + LOFF + ow * g.stride * g.C;
    union { uint4 v; T e[VEC]; } o;
    o.v = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      if (k0 + e < K) {
        o.e[e] = src[r];
        if (++r == RW) { r = 0; src += LROW; }
      }
    }
    *reinterpret_cast<uint4*>(out + (int64_t)q * VEC) = o.v;
  }
}

hipError_t launch_im2col(const void* x, void* col, int B, const ConvGeom& g, int kpad, int dtype, hipStream_t stream) {
  const int vec = dtype == DT_BF16 ? 8 : 4;
  if (kpad % vec || kpad < g.KH * g.KW * g.C) return hipErrorInvalidValue;
  const int64_t n = (int64_t)B * g.OH * g.OW * (kpad / vec);
  {
    // LDS row: [zeros up to LPADV = pad * C rounded up to the vector width][W * C image elements][zeros], long
    // enough for the last window: offset LOFF + (OW - 1) * stride * C + KW * C - 1
    const int WC = g.W * g.C, es = dtype == DT_BF16 ? 2 : 4;
    const int lpadv = (g.pad * g.C + vec - 1) / vec * vec, loff = lpadv - g.pad * g.C;
    const int need = std::max(lpadv + WC, loff + (g.OW - 1) * g.stride * g.C + g.KW * g.C);
    const int lrow = (need + vec - 1) / vec * vec;
    const size_t lds = (size_t)g.KH * lrow * es;
    if (WC % vec == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(col) % 16 == 0 && lds <= 48 * 1024 &&
        (int64_t)B * g.OH < (1ll << 31)) {
      CDP_DISPATCH(dtype, hipLaunchKernelGGL((im2col_rows_kernel<T>), dim3((unsigned)(B * g.OH)), dim3(256), lds, stream,
                                             static_cast<const T*>(x), static_cast<T*>(col), g, kpad, lrow, loff));
      return hipGetLastError();
    }
  }
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((im2col_kernel<T>), dim3(blocks_for(n, 256, 1 << 20)), dim3(256), 0, stream,
                                         static_cast<const T*>(x), static_cast<T*>(col), n, g, kpad));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
template <typename T>
__global__ void maxpool_fwd_kernel(const T* __restrict__ x, T* __restrict__ y, int B, int H, int W, int C, int OH, int OW,
                                   int k, int s, int p) {
  const int64_t n = (int64_t)B * OH * OW * C;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int c = (int)(i % C);
    int64_t q = i / C;
    int ow = (int)(q % OW); q /= OW;
    int oh = (int)(q % OH);
    int b = (int)(q / OH);
    float best = -INFINITY;
    for (int kh = 0; kh < k; ++kh)
      for (int kw = 0; kw < k; ++kw) {
        int ih = oh * s - p + kh, iw = ow * s - p + kw;
        if (ih < 0 || iw < 0 || ih >= H || iw >= W) continue;
        best = fmaxf(best, ld_f32<T>(x, (((int64_t)b * H + ih) * W + iw) * C + c));
      }
    st_f32<T>(y, i, best);
  }
}

// dx[b][ih][iw][c] = sum over windows whose first maximum sits at (ih, iw) of dy.
template <typename T>
__global__ void maxpool_bwd_kernel(const T* __restrict__ x, const T* __restrict__ dy, T* __restrict__ dx, int B, int H, int W,
                                   int C, int OH, int OW, int k, int s, int p, int mask_relu) {
  const int64_t n = (int64_t)B * H * W * C;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int c = (int)(i % C);
    int64_t q = i / C;
    int iw = (int)(q % W); q /= W;
    int ih = (int)(q % H);
    int b = (int)(q / H);
    const float xv = ld_f32<T>(x, i);
    float g = 0.f;
    if (!(mask_relu && !(xv > 0.f))) {
      // windows (oh, ow) that contain (ih, iw): oh*s - p <= ih <= oh*s - p + k - 1
      int oh_lo = max(0, (ih + p - k + s) / s), oh_hi = min(OH - 1, (ih + p) / s);
      int ow_lo = max(0, (iw + p - k + s) / s), ow_hi = min(OW - 1, (iw + p) / s);
      for (int oh = oh_lo; oh <= oh_hi; ++oh)
        for (int ow = ow_lo; ow <= ow_hi; ++ow) {
          // is (ih, iw) the first maximum of this window in (kh, kw) scan order?
          bool first = true;
          for (int kh = 0; kh < k && first; ++kh)
            for (int kw = 0; kw < k; ++kw) {
              int jh = oh * s - p + kh, jw = ow * s - p + kw;
              if (jh < 0 || jw < 0 || jh >= H || jw >= W) continue;
              if (jh == ih && jw == iw) continue;
              float o = ld_f32<T>(x, (((int64_t)b * H + jh) * W + jw) * C + c);
              bool before = (jh < ih) || (jh == ih && jw < iw);
              if (o > xv || (before && o == xv)) { first = false; break; }
            }
          if (first) g += ld_f32<T>(dy, (((int64_t)b * OH + oh) * OW + ow) * C + c);
        }
    }
    st_f32<T>(dx, i, g);
  }
}

// Same rule, 16 bytes of channels per thread (C a multiple of the chunk).
template <typename T>
__global__ void maxpool_bwd_vec_kernel(const T* __restrict__ x, const T* __restrict__ dy, T* __restrict__ dx, int B, int H, int W,
                                       int C, int OH, int OW, int k, int s, int p, int mask_relu) {
  constexpr int VEC = 16 / sizeof(T);
  union Ch { uint4 v; T e[VEC]; };
  const int cpp = C / VEC;
  const int64_t n = (int64_t)B * H * W * cpp;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % cpp) * VEC;
    int64_t q = i / cpp;
    const int iw = (int)(q % W); q /= W;
    const int ih = (int)(q % H);
    const int b = (int)(q / H);
    Ch xc;
    xc.v = *reinterpret_cast<const uint4*>(x + (((int64_t)b * H + ih) * W + iw) * C + c);
    float xv[VEC], g[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) { xv[e] = ld_f32<T>(xc.e, e); g[e] = 0.f; }
    const int oh_lo = max(0, (ih + p - k + s) / s), oh_hi = min(OH - 1, (ih + p) / s);
    const int ow_lo = max(0, (iw + p - k + s) / s), ow_hi = min(OW - 1, (iw + p) / s);
    for (int oh = oh_lo; oh <= oh_hi; ++oh)
      for (int ow = ow_lo; ow <= ow_hi; ++ow) {
        bool first[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) first[e] = true;
        for (int kh = 0; kh < k; ++kh)
          for (int kw = 0; kw < k; ++kw) {
            const int jh = oh * s - p + kh, jw = ow * s - p + kw;
            if (jh < 0 || jw < 0 || jh >= H || jw >= W || (jh == ih && jw == iw)) continue;
            Ch oc;
            oc.v = *reinterpret_cast<const uint4*>(x + (((int64_t)b * H + jh) * W + jw) * C + c);
            const bool before = (jh < ih) || (jh == ih && jw < iw);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
              const float o = ld_f32<T>(oc.e, e);
              if (o > xv[e] || (before && o == xv[e])) first[e] = false;
            }
          }
        Ch dc;
        dc.v = *reinterpret_cast<const uint4*>(dy + (((int64_t)b * OH + oh) * OW + ow) * C + c);
#pragma unroll
        for (int e = 0; e < VEC; ++e)
          if (first[e]) g[e] += ld_f32<T>(dc.e, e);
      }
    Ch out;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float v = (mask_relu && !(xv[e] > 0.f)) ? 0.f : g[e];
      st_f32<T>(out.e, e, v);
    }
    *reinterpret_cast<uint4*>(dx + (((int64_t)b * H + ih) * W + iw) * C + c) = out.v;
  }
}

// 16 bytes of channels per thread (C a multiple of the chunk).
template <typename T>
__global__ void maxpool_fwd_vec_kernel(const T* __restrict__ x, T* __restrict__ y, int B, int H, int W, int C, int OH, int OW,
                                       int k, int s, int p) {
  constexpr int VEC = 16 / sizeof(T);
  union Ch { uint4 v; T e[VEC]; };
  const int cpp = C / VEC;
  const int64_t n = (int64_t)B * OH * OW * cpp;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % cpp) * VEC;
    int64_t q = i / cpp;
    const int ow = (int)(q % OW); q /= OW;
    const int oh = (int)(q % OH);
    const int b = (int)(q / OH);
    float best[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) best[e] = -INFINITY;
    for (int kh = 0; kh < k; ++kh)
      for (int kw = 0; kw < k; ++kw) {
        const int ih = oh * s - p + kh, iw = ow * s - p + kw;
        if (ih < 0 || iw < 0 || ih >= H || iw >= W) continue;
        Ch xc;
        xc.v = *reinterpret_cast<const uint4*>(x + (((int64_t)b * H + ih) * W + iw) * C + c);
#pragma unroll
        for (int e = 0; e < VEC; ++e) best[e] = fmaxf(best[e], ld_f32<T>(xc.e, e));
      }
    Ch out;
#pragma unroll
    for (int e = 0; e < VEC; ++e) st_f32<T>(out.e, e, best[e]);
    *reinterpret_cast<uint4*>(y + i * VEC) = out.v;
  }
}

hipError_t launch_maxpool_fwd(const void* x, void* y, int B, int H, int W, int C, int k, int s, int p, int dtype,
                              hipStream_t stream) {
  int OH = (H + 2 * p - k) / s + 1, OW = (W + 2 * p - k) / s + 1;
  int64_t n = (int64_t)B * OH * OW * C;
  const int vec = dtype == DT_BF16 ? 8 : 4;
  if (C % vec == 0) {
    CDP_DISPATCH(dtype, hipLaunchKernelGGL((maxpool_fwd_vec_kernel<T>), dim3(blocks_for(n / vec, 256, 1 << 20)), dim3(256), 0, stream,
                                           static_cast<const T*>(x), static_cast<T*>(y), B, H, W, C, OH, OW, k, s, p));
    return hipGetLastError();
  }
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((maxpool_fwd_kernel<T>), dim3(blocks_for(n, 256, 65536)), dim3(256), 0, stream,
                                         static_cast<const T*>(x), static_cast<T*>(y), B, H, W, C, OH, OW, k, s, p));
  return hipGetLastError();
}
// Backward in two steps when a workspace is given: every window's first maximum (tap index
// in (kh, kw) scan order, one byte per output element), then a gather in which an input
// position compares its tap index in each window that covers it.  Each window is scanned
// once instead of once per covered position.
template <typename T>
__global__ void maxpool_argmax_kernel(const T* __restrict__ x, uint8_t* __restrict__ idx, int B, int H, int W, int C, int OH,
                                      int OW, int k, int s, int p) {
  constexpr int VEC = 16 / sizeof(T);
  union Ch { uint4 v; T e[VEC]; };
  union Ix { uint2 v; uint8_t e[8]; };
  const int cpp = C / VEC;
  const int64_t n = (int64_t)B * OH * OW * cpp;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % cpp) * VEC;
    int64_t q = i / cpp;
    const int ow = (int)(q % OW); q /= OW;
    const int oh = (int)(q % OH);
    const int b = (int)(q / OH);
    float best[VEC];
    Ix arg;
    arg.v = make_uint2(0xffffffffu, 0xffffffffu);  // 255: no tap inside the image
#pragma unroll
    for (int e = 0; e < VEC; ++e) best[e] = -INFINITY;
    for (int kh = 0; kh < k; ++kh)
      for (int kw = 0; kw < k; ++kw) {
        const int jh = oh * s - p + kh, jw = ow * s - p + kw;
        if (jh < 0 || jw < 0 || jh >= H || jw >= W) continue;
        Ch xc;
        xc.v = *reinterpret_cast<const uint4*>(x + (((int64_t)b * H + jh) * W + jw) * C + c);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float v = ld_f32<T>(xc.e, e);
          if (v > best[e] || arg.e[e] == 255) { best[e] = v; arg.e[e] = (uint8_t)(kh * k + kw); }
        }
      }
    uint8_t* dst = idx + i * VEC;
    if (VEC == 8) *reinterpret_cast<uint2*>(dst) = arg.v;
    else *reinterpret_cast<uint32_t*>(dst) = arg.v.x;
  }
}

template <typename T>
__global__ void maxpool_bwd_idx_kernel(const T* __restrict__ x, const T* __restrict__ dy, const uint8_t* __restrict__ idx,
                                       T* __restrict__ dx, int B, int H, int W, int C, int OH, int OW, int k, int s, int p,
                                       int mask_relu) {
  constexpr int VEC = 16 / sizeof(T);
  union Ch { uint4 v; T e[VEC]; };
  union Ix { uint2 v; uint8_t e[8]; };
  const int cpp = C / VEC;
  const int64_t n = (int64_t)B * H * W * cpp;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % cpp) * VEC;
    int64_t q = i / cpp;
    const int iw = (int)(q % W); q /= W;
    const int ih = (int)(q % H);
    const int b = (int)(q / H);
    float g[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) g[e] = 0.f;
    const int oh_lo = max(0, (ih + p - k + s) / s), oh_hi = min(OH - 1, (ih + p) / s);
    const int ow_lo = max(0, (iw + p - k + s) / s), ow_hi = min(OW - 1, (iw + p) / s);
    for (int oh = oh_lo; oh <= oh_hi; ++oh)
      for (int ow = ow_lo; ow <= ow_hi; ++ow) {
        const int tap = (ih - (oh * s - p)) * k + (iw - (ow * s - p));
        const int64_t o = (((int64_t)b * OH + oh) * OW + ow) * C + c;
        Ix a;
        if (VEC == 8) a.v = *reinterpret_cast<const uint2*>(idx + o);
        else a.v = make_uint2(*reinterpret_cast<const uint32_t*>(idx + o), 0u);
        Ch dc;
        dc.v = *reinterpret_cast<const uint4*>(dy + o);
#pragma unroll
        for (int e = 0; e < VEC; ++e)
          if (a.e[e] == tap) g[e] += ld_f32<T>(dc.e, e);
      }
    Ch out;
    if (mask_relu) {
      Ch xc;
      xc.v = *reinterpret_cast<const uint4*>(x + (((int64_t)b * H + ih) * W + iw) * C + c);
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if (!(ld_f32<T>(xc.e, e) > 0.f)) g[e] = 0.f;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) st_f32<T>(out.e, e, g[e]);
    *reinterpret_cast<uint4*>(dx + (((int64_t)b * H + ih) * W + iw) * C + c) = out.v;
  }
}

hipError_t launch_maxpool_bwd(const void* x, const void* dy, void* dx, int B, int H, int W, int C, int k, int s, int p,
                              int mask_relu, void* workspace, int64_t workspace_bytes, int dtype, hipStream_t stream) {
  int OH = (H + 2 * p - k) / s + 1, OW = (W + 2 * p - k) / s + 1;
  int64_t n = (int64_t)B * H * W * C;
  const int vec = dtype == DT_BF16 ? 8 : 4;
  const int64_t n_out = (int64_t)B * OH * OW * C;
  if (C % vec == 0 && workspace != nullptr && workspace_bytes >= n_out && k * k < 255) {
    uint8_t* idx = static_cast<uint8_t*>(workspace);
    CDP_DISPATCH(dtype, hipLaunchKernelGGL((maxpool_argmax_kernel<T>), dim3(blocks_for(n_out / vec, 256, 1 << 20)), dim3(256), 0,
                                           stream, static_cast<const T*>(x), idx, B, H, W, C, OH, OW, k, s, p));
    CDP_DISPATCH(dtype, hipLaunchKernelGGL((maxpool_bwd_idx_kernel<T>), dim3(blocks_for(n / vec, 256, 1 << 20)), dim3(256), 0,
                                           stream, static_cast<const T*>(x), static_cast<const T*>(dy), idx, static_cast<T*>(dx),
                                           B, H, W, C, OH, OW, k, s, p, mask_relu));
    return hipGetLastError();
  }
  if (C % vec == 0) {
    CDP_DISPATCH(dtype, hipLaunchKernelGGL((maxpool_bwd_vec_kernel<T>), dim3(blocks_for(n / vec, 256, 1 << 20)), dim3(256), 0, stream,
                                           static_cast<const T*>(x), static_cast<const T*>(dy), static_cast<T*>(dx), B, H, W, C,
                                           OH, OW, k, s, p, mask_relu));
    return hipGetLastError();
  }
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((maxpool_bwd_kernel<T>), dim3(blocks_for(n, 256, 65536)), dim3(256), 0, stream,
                                         static_cast<const T*>(x), static_cast<const T*>(dy), static_cast<T*>(dx), B, H, W, C,
                                         OH, OW, k, s, p, mask_relu));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
template <typename T>
__global__ void gap_fwd_kernel(const T* __restrict__ x, T* __restrict__ y, int B, int HW, int C) {
  const int64_t n = (int64_t)B * C;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int c = (int)(i % C);
    int b = (int)(i / C);
    // eight reads in flight at a time, added in position order (the sum is that of the plain loop)
    const int64_t base = (int64_t)b * HW * C + c;
    float s = 0.f;
    int q = 0;
    for (; q + 8 <= HW; q += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = ld_f32<T>(x, base + (int64_t)(q + u) * C);
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; q < HW; ++q) s += ld_f32<T>(x, base + (int64_t)q * C);
    st_f32<T>(y, i, s / (float)HW);
  }
}
template <typename T>
__global__ void gap_bwd_kernel(const T* __restrict__ x, const T* __restrict__ dy, T* __restrict__ dx, int B, int HW, int C,
                               int mask_relu) {
  const int64_t n = (int64_t)B * HW * C;
  const float inv = 1.0f / (float)HW;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int c = (int)(i % C);
    int b = (int)(i / ((int64_t)HW * C));
    float g = ld_f32<T>(dy, (int64_t)b * C + c) * inv;
    if (mask_relu && !(ld_f32<T>(x, i) > 0.f)) g = 0.f;
    st_f32<T>(dx, i, g);
  }
}
hipError_t launch_gap_fwd(const void* x, void* y, int B, int HW, int C, int dtype, hipStream_t stream) {
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((gap_fwd_kernel<T>), dim3(blocks_for((int64_t)B * C, 256, 4096)), dim3(256), 0, stream,
                                         static_cast<const T*>(x), static_cast<T*>(y), B, HW, C));
  return hipGetLastError();
}
hipError_t launch_gap_bwd(const void* x, const void* dy, void* dx, int B, int HW, int C, int mask_relu, int dtype,
                          hipStream_t stream) {
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((gap_bwd_kernel<T>), dim3(blocks_for((int64_t)B * HW * C, 256, 65536)), dim3(256), 0,
                                         stream, static_cast<const T*>(x), static_cast<const T*>(dy), static_cast<T*>(dx), B, HW,
                                         C, mask_relu));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
template <typename T>
__global__ void to_f32_kernel(const T* __restrict__ src, float* __restrict__ dst, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = ld_f32<T>(src, i);
}
hipError_t launch_to_f32(const void* src, float* dst, int64_t n, int dtype, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  CDP_DISPATCH(dtype, hipLaunchKernelGGL((to_f32_kernel<T>), dim3(blocks_for(n, 256, 4096)), dim3(256), 0, stream,
                                         static_cast<const T*>(src), dst, n));
  return hipGetLastError();
}

}  // namespace cdp
