// The self-attention core: one kernel forward, two backward, nothing but the probabilities (fp32: and the gradient of
// the scores) travelling through memory between the products.  First bf16, then fp32.
//
// What bounds them: 32 samples x 12 heads x 196 tokens of width 64 are 68 MB forward and 97 MB backward (q, k, v, d out,
// the probabilities, the results) against 3.8 and 7.6 GFLOP, so memory; the contractions are short and the softmax
// sits between them, so what costs time is everything that is not one of those bytes.  Every wavefront computes score
// blocks TRANSPOSED (rows = keys, columns = the 32 queries of its lanes): a lane then holds 4 neighbouring keys per
// group of accumulator registers for one query, row sums and maxima are sums inside the lane plus one exchange with
// lane +- 32, and the rounded probabilities are, in the registers they are in, the column operand of the next
// product: lane half `hi` holds keys 16 s + 4 hi + 0..3 and 16 s + 8 + 4 hi + 0..3 of a 16-key step, and the row operand
// is read from LDS (transposing reads) in that same order of keys, which a contraction is free to choose.
// A workgroup is four wavefronts of 32 queries (or keys) each; k and v (or q and d out) of the head are staged in LDS
// once, without padding for heads of width 64 (16-byte chunks swizzled by the row instead) so that three workgroups
// fit a CU: 768 workgroups for the shape above, three per CU.
// The limit in tokens is LDS (64-wide heads: 624); past 256 tokens the forward contracts the scores twice instead of
// keeping them (8 x 400 tokens, 8 heads of 64: 43 -> 22 us forward, 84 -> 49 us backward against separate kernels).
// Measured there (us, forward / backward): score rows and products as kernels of their own 50 / 101; these three
// 20 / 48.  What is left above the bytes (13 / 28 at the rate of a large copy, were every tensor
// read once per kernel) is that the resident workgroups move in step: they stage, contract and store together; 192
// workgroups, less than one per CU, take 10 us already.  Requested is more: every workgroup of 128 tokens stages k and v (or q and
// d out) of its head again, twice at 196 tokens, and dq walks the probabilities twice, for the row sums and for the products; the
// bound above takes those second reads for hits of the XCD's L2, to which the workgroups of a head are dealt together.
#include "elem.h"
#include "kernels.h"

#include <algorithm>

namespace cdp {

namespace {

typedef short att_v4s __attribute__((ext_vector_type(4)));

struct AttnArgs {
  const uint16_t* qkv;   // [B][NT][3 D]
  uint16_t* P;           // [B][heads][NT][NT]: written forward, read backward
  const uint16_t* dout;  // backward: [B][NT][D]
  uint16_t* out;         // forward: [B][NT][D]; backward: d qkv [B][NT][3 D]
  float* delta;          // backward: [B][heads][NT], rowsum(dP * P)
  int NT, D, heads;
  int blocks;            // workgroups per (sample, head)
  int vec;               // rows of P are whole, aligned 8-byte groups
  int dvec;              // rows of delta are whole, aligned 16-byte groups
  float scale;
};

// Tile of `rows` token rows of one head in LDS: 16-byte chunk c of row r at chunk (c ^ (r & SWZ)) of the row.
template <int KS> struct AttnTile {
  static constexpr int DH = 16 * KS, CPR = DH / 8;
  static constexpr int SWZ = CPR == 8 ? 7 : 0;
  static constexpr int PITCH = CPR == 8 ? DH : DH + 8;  // elements
  __device__ static __forceinline__ int at(int row, int col) { return row * PITCH + (((col >> 3) ^ (row & SWZ)) << 3) + (col & 7); }
};

// Both tiles of a workgroup (`rows`: the tokens rounded up to 16): rows past the last token are zero.  All chunks of a pass are requested before the first is
// written to LDS.
template <int KS>
__device__ __forceinline__ void stage_two(uint16_t* t0, uint16_t* t1, const uint16_t* s0, const uint16_t* s1, int64_t ld0, int64_t ld1, int NT,
                                          int rows) {
  using Tile = AttnTile<KS>;
  constexpr int CPR = Tile::CPR, U = 4;
  const int total = rows * CPR;
  for (int e0 = threadIdx.x; e0 < total; e0 += 256 * U) {
    uint4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + 256 * u, r = e / CPR, c = (e - r * CPR) * 8;
      const bool in = e < total && r < NT;
      a[u] = in ? *reinterpret_cast<const uint4*>(s0 + (int64_t)r * ld0 + c) : make_uint4(0, 0, 0, 0);
      b[u] = in ? *reinterpret_cast<const uint4*>(s1 + (int64_t)r * ld1 + c) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + 256 * u, r = e / CPR, c = (e - r * CPR) * 8;
      if (e >= total) continue;
      *reinterpret_cast<uint4*>(t0 + Tile::at(r, c)) = a[u];
      *reinterpret_cast<uint4*>(t1 + Tile::at(r, c)) = b[u];
    }
  }
}

// Row operand (rows r0 .. r0 + 31 of the tile, columns 16 ks ..) of a 32x32x16 product that reduces over the head width.
// Where the tile ends after 16 of them the upper 16 rows repeat the lower ones; what comes of them is masked or skipped.
template <int KS>
__device__ __forceinline__ uint4 frag_rows(const uint16_t* tile, int r0, int ks, int lane, int rows) {
  const int r = r0 + (r0 + 32 <= rows ? lane & 31 : lane & 15);
  return *reinterpret_cast<const uint4*>(tile + AttnTile<KS>::at(r, 16 * ks + 8 * (lane >> 5)));
}
// Row operand whose rows are tile columns c0 .. c0 + 31 and whose reduction index is the tile row, taken in the order in
// which an accumulator holds rows: lane half hi gets rows r0 + 4 hi + 0..3, then r0 + 8 + 4 hi + 0..3.
template <int KS>
__device__ __forceinline__ uint4 frag_cols(const uint16_t* tile, int r0, int c0, int lane) {
  const int rho = lane & 15, row = r0 + 4 * (lane >> 5) + (rho >> 2), col = c0 + 16 * ((lane >> 4) & 1) + 4 * (rho & 3);
  typedef __attribute__((address_space(3))) att_v4s* lds_ptr;
  union { att_v4s v[2]; uint4 u; } f;
  f.v[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + AttnTile<KS>::at(row, col)));
  f.v[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + AttnTile<KS>::at(row + 8, col)));
  return f.u;
}
__device__ __forceinline__ uint32_t pack2(float lo, float hi) { return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16); }
__device__ __forceinline__ float lo16(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float hi16(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ v16f_t zero16() {
  v16f_t a;
#pragma unroll
  for (int v = 0; v < 16; ++v) a[v] = 0.f;
  return a;
}

// The 16 probabilities of a lane for keys k0 .. k0 + 15 of its query, w[0] = keys 4 hi + 0..3 and w[1] = 8 + 4 hi + 0..3,
// from / to the query's row in memory (nullptr: zeros / nothing), where a lane half moves 8 neighbouring keys: with
// 8-byte pieces a wavefront's 32 rows cost twice the instructions and the store rate of the CU bounded the kernel.  Rows start at
// any element (NT may be odd): whole pieces move at the alignment of an element all the same, which global memory allows; element by
// element the backward of 64 heads of width 48 and 577 tokens took 415 us, 225 us so.
struct __attribute__((packed, aligned(2))) P8 { uint32_t u[4]; };
__device__ __forceinline__ void swap_halves(uint2 (&w)[2]) {  // (its own inverse)
  auto x = __builtin_amdgcn_permlane32_swap(w[0].x, w[1].x, false, false);
  auto y = __builtin_amdgcn_permlane32_swap(w[0].y, w[1].y, false, false);
  w[0] = make_uint2(x[0], y[0]);
  w[1] = make_uint2(x[1], y[1]);
}
__device__ __forceinline__ void load_p16(const uint16_t* row, int k0, int hi, int NT, int vec, uint2 (&w)[2]) {
  const int k = k0 + 8 * hi;
  w[0] = w[1] = make_uint2(0, 0);
  if (row != nullptr) {
    if (k + 8 <= NT) {
      const P8 p = *reinterpret_cast<const P8*>(row + k);
      w[0] = make_uint2(p.u[0], p.u[1]);
      w[1] = make_uint2(p.u[2], p.u[3]);
    } else if (vec) {
      if (k < NT) w[0] = *reinterpret_cast<const uint2*>(row + k);
    } else {
      uint32_t e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = k + i < NT ? row[k + i] : 0u;
      w[0] = make_uint2(e[0] | (e[1] << 16), e[2] | (e[3] << 16));
      w[1] = make_uint2(e[4] | (e[5] << 16), e[6] | (e[7] << 16));
    }
  }
}
__device__ __forceinline__ void store_p16(uint16_t* row, int k0, int hi, int NT, int vec, uint2 a, uint2 b) {
  uint2 w[2] = {a, b};
  swap_halves(w);
  const int k = k0 + 8 * hi;
  if (row == nullptr) return;
  if (k + 8 <= NT) {
    *reinterpret_cast<P8*>(row + k) = P8{{w[0].x, w[0].y, w[1].x, w[1].y}};
  } else if (vec) {
    if (k < NT) *reinterpret_cast<uint2*>(row + k) = w[0];
  } else {
    const uint32_t e[4] = {w[0].x, w[0].y, w[1].x, w[1].y};
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (k + i < NT) row[k + i] = (uint16_t)(e[i >> 1] >> (16 * (i & 1)));
  }
}
// Transposed 32-column block of a result (rows = head columns 32 ob .., column = the lane's token) -> the token's row.
template <int KS>
__device__ __forceinline__ void store_cols(uint16_t* dst, int ob, int hi, const v16f_t& acc) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int j = 32 * ob + 8 * g + 4 * hi;
    if (j < 16 * KS) *reinterpret_cast<uint2*>(dst + j) = make_uint2(pack2(acc[4 * g], acc[4 * g + 1]), pack2(acc[4 * g + 2], acc[4 * g + 3]));
  }
}

// ---- forward: P = softmax(scale q k^T), out = P v ---------------------------------------------------------------------
// NB > 0: all score blocks of a wavefront's 32 queries stay in registers (at most 32 NB keys).  NB = 0: any number of
// keys, in two passes over the blocks, the first for the row maximum and sum.
template <int KS, int NB>
__global__ __launch_bounds__(256, NB == 8 && KS == 5 ? 2 : 3) void attn_fwd_kernel(const AttnArgs a) {
  using Tile = AttnTile<KS>;
  constexpr int OB = (KS + 1) / 2, DH = Tile::DH;
  extern __shared__ __attribute__((aligned(16))) unsigned char att_smem[];
  const int NT = a.NT, rows = (NT + 15) & ~15, nblk = (NT + 31) >> 5;
  uint16_t* Ks = reinterpret_cast<uint16_t*>(att_smem);
  uint16_t* Vs = Ks + rows * Tile::PITCH;
  const int id = xcd_block_cyclic(blockIdx.x, gridDim.x, a.blocks);  // the workgroups of a head share an XCD's L2
  const int z = id / a.blocks, sample = z / a.heads, head = z % a.heads;
  const int lane = threadIdx.x & 63, l31 = lane & 31, hi = lane >> 5;
  const int q = ((id % a.blocks) * 4 + (threadIdx.x >> 6)) * 32 + l31;
  const int64_t tok = 3ll * a.D;
  const uint16_t* base = a.qkv + sample * NT * tok + head * DH;
  const uint16_t* qrow = base + (int64_t)min(q, NT - 1) * tok;  // rows past the end repeat the last one; nothing of them is stored
  uint4 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const uint4*>(qrow + 16 * ks + 8 * hi);
  stage_two<KS>(Ks, Vs, base + a.D, base + 2 * a.D, tok, tok, NT, rows);
  __syncthreads();
  const float c = a.scale * 1.44269504088896340736f;
  auto scores = [&](int b) {
    v16f_t s = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = mfma_bf16(frag_rows<KS>(Ks, 32 * b, ks, lane, rows), qf[ks], s);
    if (32 * b + 32 > NT) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (32 * b + 8 * (v >> 2) + 4 * hi + (v & 3) >= NT) s[v] = -INFINITY;
    }
    return s;
  };
  auto block_max = [&](const v16f_t& s) {
    float m = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) m = fmaxf(m, s[v]);
    return m;
  };
  v16f_t o[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) o[ob] = zero16();
  uint16_t* prow = q < NT ? a.P + ((int64_t)z * NT + q) * NT : nullptr;
  // a finished block of probabilities: to memory, and as the column operand of out^T = v^T P^T
  auto finish = [&](int b, const v16f_t& p) {
    uint2 w[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) w[g] = make_uint2(pack2(p[4 * g], p[4 * g + 1]), pack2(p[4 * g + 2], p[4 * g + 3]));
#pragma unroll
    for (int s = 0; s < 2; ++s) store_p16(prow, 32 * b + 16 * s, hi, NT, a.vec, w[2 * s], w[2 * s + 1]);
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (32 * b + 16 * s < rows)
#pragma unroll
      for (int ob = 0; ob < OB; ++ob)
        o[ob] = mfma_bf16(frag_cols<KS>(Vs, 32 * b + 16 * s, 32 * ob, lane), make_uint4(w[2 * s].x, w[2 * s].y, w[2 * s + 1].x, w[2 * s + 1].y), o[ob]);
  };
  if constexpr (NB > 0) {
    v16f_t s[NB];
    float m = -INFINITY;
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b < nblk) {
        s[b] = scores(b);
        m = fmaxf(m, block_max(s[b]));
      }
    m = fmaxf(m, __shfl_xor(m, 32, 64)) * c;  // finite: key 0 is always there
    float sum = 0.f;
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b < nblk) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          s[b][v] = __builtin_amdgcn_exp2f(s[b][v] * c - m);
          sum += s[b][v];
        }
      }
    const float inv = __builtin_amdgcn_rcpf(sum + __shfl_xor(sum, 32, 64));
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b < nblk) {
#pragma unroll
        for (int v = 0; v < 16; ++v) s[b][v] *= inv;
        finish(b, s[b]);
      }
  } else {
    float m = -INFINITY, sum = 0.f;
    for (int b = 0; b < nblk; ++b) {
      const v16f_t s = scores(b);
      const float mb = block_max(s);
      const float mn = fmaxf(m, fmaxf(mb, __shfl_xor(mb, 32, 64)) * c);  // the same in both lanes of a query
      sum *= __builtin_amdgcn_exp2f(m - mn);
      m = mn;
#pragma unroll
      for (int v = 0; v < 16; ++v) sum += __builtin_amdgcn_exp2f(s[v] * c - m);
    }
    const float inv = __builtin_amdgcn_rcpf(sum + __shfl_xor(sum, 32, 64));
    for (int b = 0; b < nblk; ++b) {
      v16f_t s = scores(b);
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] = __builtin_amdgcn_exp2f(s[v] * c - m) * inv;
      finish(b, s);
    }
  }
  if (q < NT) {
    uint16_t* dst = a.out + ((int64_t)sample * NT + q) * a.D + head * DH;
#pragma unroll
    for (int ob = 0; ob < OB; ++ob) store_cols<KS>(dst, ob, hi, o[ob]);
  }
}

// ---- backward, queries: delta = rowsum(dP * P) and dq = dS k, with dP = d out v^T, dS = P * (dP - delta) * scale -------
// Two passes over the key blocks, dP contracted in both: keeping all of it for the second costs a workgroup per CU.
template <int KS>
__global__ __launch_bounds__(256, 3) void attn_bwd_dq_kernel(const AttnArgs a) {
  using Tile = AttnTile<KS>;
  constexpr int OB = (KS + 1) / 2, DH = Tile::DH;
  extern __shared__ __attribute__((aligned(16))) unsigned char att_smem[];
  const int NT = a.NT, rows = (NT + 15) & ~15, nblk = (NT + 31) >> 5;
  uint16_t* Vs = reinterpret_cast<uint16_t*>(att_smem);
  uint16_t* Ks = Vs + rows * Tile::PITCH;
  const int id = xcd_block_cyclic(blockIdx.x, gridDim.x, a.blocks);
  const int z = id / a.blocks, sample = z / a.heads, head = z % a.heads;
  const int lane = threadIdx.x & 63, l31 = lane & 31, hi = lane >> 5;
  const int q = ((id % a.blocks) * 4 + (threadIdx.x >> 6)) * 32 + l31;
  const int64_t tok = 3ll * a.D;
  const uint16_t* base = a.qkv + sample * NT * tok + head * DH;
  const uint16_t* drow = a.dout + ((int64_t)sample * NT + min(q, NT - 1)) * a.D + head * DH;
  uint4 df[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) df[ks] = *reinterpret_cast<const uint4*>(drow + 16 * ks + 8 * hi);
  stage_two<KS>(Vs, Ks, base + 2 * a.D, base + a.D, tok, tok, NT, rows);
  __syncthreads();
  // Probabilities as they lie in memory (swap_halves where they are used).  Blocks of 32 whole keys are read without a branch, one block ahead:
  // a read inside one is waited for inside it, and every block then cost a round trip in either pass.  Queries past the last repeat it
  // (their lanes are not stored); the block that the keys end in is read once, ahead of everything.
  const int whole = NT >> 5;
  const uint16_t* prow = a.P + ((int64_t)z * NT + min(q, NT - 1)) * NT;
  auto load_block = [&](int b, uint2 (&w)[2][2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const P8 p = *reinterpret_cast<const P8*>(prow + 32 * b + 16 * t + 8 * hi);
      w[t][0] = make_uint2(p.u[0], p.u[1]);
      w[t][1] = make_uint2(p.u[2], p.u[3]);
    }
  };
  auto dp_block = [&](int b) {
    v16f_t s = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = mfma_bf16(frag_rows<KS>(Vs, 32 * b, ks, lane, rows), df[ks], s);
    return s;
  };
  float delta = 0.f;
  auto sum_block = [&](int b, uint2 (&w)[2][2]) {
    const v16f_t s = dp_block(b);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      swap_halves(w[t]);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int v = 8 * t + 4 * g;
        delta += lo16(w[t][g].x) * s[v] + hi16(w[t][g].x) * s[v + 1];
        delta += lo16(w[t][g].y) * s[v + 2] + hi16(w[t][g].y) * s[v + 3];
      }
    }
  };
  v16f_t o[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) o[ob] = zero16();
  auto mul_block = [&](int b, uint2 (&w)[2][2]) {
    const v16f_t s = dp_block(b);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      swap_halves(w[t]);
      uint2 d[2];
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int v = 8 * t + 4 * g;
        d[g].x = pack2(lo16(w[t][g].x) * (s[v] - delta) * a.scale, hi16(w[t][g].x) * (s[v + 1] - delta) * a.scale);
        d[g].y = pack2(lo16(w[t][g].y) * (s[v + 2] - delta) * a.scale, hi16(w[t][g].y) * (s[v + 3] - delta) * a.scale);
      }
      if (32 * b + 16 * t < rows)
#pragma unroll
        for (int ob = 0; ob < OB; ++ob)
          o[ob] = mfma_bf16(frag_cols<KS>(Ks, 32 * b + 16 * t, 32 * ob, lane), make_uint4(d[0].x, d[0].y, d[1].x, d[1].y), o[ob]);
    }
  };
  uint2 w[2][2], nw[2][2], last[2][2];
  if (nblk > whole) {
#pragma unroll
    for (int t = 0; t < 2; ++t) load_p16(prow, 32 * whole + 16 * t, hi, NT, a.vec, last[t]);
  }
  if (whole > 0) load_block(0, w);
  auto walk = [&](auto block) {
    for (int b = 0; b < whole; ++b) {
      load_block(b + 1 < whole ? b + 1 : 0, nw);  // (at the end: the first for the second pass)
      block(b, w);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int g = 0; g < 2; ++g) w[t][g] = nw[t][g];
    }
    if (nblk > whole) {
      uint2 e[2][2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int g = 0; g < 2; ++g) e[t][g] = last[t][g];
      block(whole, e);
    }
  };
  walk(sum_block);
  delta += __shfl_xor(delta, 32, 64);
  if (q < NT && hi == 0) a.delta[(int64_t)z * NT + q] = delta;
  walk(mul_block);
  if (q < NT) {
    uint16_t* dst = a.out + ((int64_t)sample * NT + q) * tok + head * DH;
#pragma unroll
    for (int ob = 0; ob < OB; ++ob) store_cols<KS>(dst, ob, hi, o[ob]);
  }
}

// ---- backward, keys: dv = P^T d out, dk = dS^T q -----------------------------------------------------------------------
// A wavefront owns 32 keys (its lanes) and walks the queries: dP is contracted the other way round (rows = queries), so
// P and dS are again the column operand in the registers they are in, now reducing over queries.
template <int KS>
__global__ __launch_bounds__(256, KS <= 4 ? 3 : 2) void attn_bwd_dkv_kernel(const AttnArgs a) {
  using Tile = AttnTile<KS>;
  constexpr int OB = (KS + 1) / 2, DH = Tile::DH;
  extern __shared__ __attribute__((aligned(16))) unsigned char att_smem[];
  const int NT = a.NT, rows = (NT + 15) & ~15, nblk = (NT + 31) >> 5;
  uint16_t* Qs = reinterpret_cast<uint16_t*>(att_smem);
  uint16_t* Os = Qs + rows * Tile::PITCH;
  const int id = xcd_block_cyclic(blockIdx.x, gridDim.x, a.blocks);
  const int z = id / a.blocks, sample = z / a.heads, head = z % a.heads;
  const int lane = threadIdx.x & 63, l31 = lane & 31, hi = lane >> 5;
  const int k = ((id % a.blocks) * 4 + (threadIdx.x >> 6)) * 32 + l31;
  const int64_t tok = 3ll * a.D;
  const uint16_t* base = a.qkv + sample * NT * tok + head * DH;
  const int kc = min(k, NT - 1);  // lanes past the last key repeat it; nothing of them is stored
  const uint16_t* vrow = base + 2 * a.D + (int64_t)kc * tok;
  uint4 vf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) vf[ks] = *reinterpret_cast<const uint4*>(vrow + 16 * ks + 8 * hi);
  stage_two<KS>(Qs, Os, base, a.dout + (int64_t)sample * NT * a.D + head * DH, tok, a.D, NT, rows);
  // P[q][k] and delta[q] of a block of 32 queries, in accumulator order.  Uniform row address + one 32-bit offset per lane:
  // 64-bit addresses per element were a third of the kernel's vector instructions.
  const uint16_t* pbase = a.P + (int64_t)z * NT * NT;
  const float* dbase = a.delta + (int64_t)z * NT;
  const uint32_t plane = (uint32_t)(4 * hi * NT + kc) * 2u, dlane = 16u * hi;
  auto load_p = [&](int b, uint16_t (&p)[16]) {
    if (32 * b + 32 <= NT) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int q = 32 * b + 8 * (v >> 2) + (v & 3);
        p[v] = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(pbase + (int64_t)q * NT) + plane);
      }
    } else {  // rows past the last query: the last one's values, times zero rows of q and d out
#pragma unroll
      for (int v = 0; v < 16; ++v) p[v] = pbase[(uint32_t)(min(32 * b + 8 * (v >> 2) + 4 * hi + (v & 3), NT - 1) * NT + kc)];
    }
  };
  auto load_delta = [&](int b, float (&dl)[16]) {
    if (a.dvec && 32 * b + 32 <= NT) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 f = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(dbase + 32 * b + 8 * g) + dlane);
        dl[4 * g] = f.x; dl[4 * g + 1] = f.y; dl[4 * g + 2] = f.z; dl[4 * g + 3] = f.w;
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) dl[v] = dbase[min(32 * b + 8 * (v >> 2) + 4 * hi + (v & 3), NT - 1)];
    }
  };
  v16f_t dv[OB], dk[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) { dv[ob] = zero16(); dk[ob] = zero16(); }
  uint16_t p[16], np[16];
  // delta a block ahead where there are registers for it: for heads of width 48 and 80 the compiler else waits for the next
  // probabilities with it (333 tokens, 72 heads of 80, both kernels 58.0 -> 45.3 us).  At 64 the two registers too many cost more than the
  // round trip to cached lines (400 tokens, 64 heads 38.2 -> 40.8 us).
  constexpr bool DELTA_AHEAD = KS == 3 || KS == 5;
  float dl[16], ndl[16];
  load_p(0, p);
  if (DELTA_AHEAD) load_delta(0, dl);
  __syncthreads();
  for (int b = 0; b < nblk; ++b) {
    if (!DELTA_AHEAD) load_delta(b, dl);
    if (b + 1 < nblk) {
      load_p(b + 1, np);
      if (DELTA_AHEAD) load_delta(b + 1, ndl);
    }
    v16f_t s = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = mfma_bf16(frag_rows<KS>(Os, 32 * b, ks, lane, rows), vf[ks], s);
    uint32_t w[8], d[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      w[e] = (uint32_t)p[2 * e] | ((uint32_t)p[2 * e + 1] << 16);
      d[e] = pack2(lo16(w[e]) * (s[2 * e] - dl[2 * e]) * a.scale, hi16(w[e]) * (s[2 * e + 1] - dl[2 * e + 1]) * a.scale);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (32 * b + 16 * t >= rows) continue;
      const uint4 pw = make_uint4(w[4 * t], w[4 * t + 1], w[4 * t + 2], w[4 * t + 3]);
      const uint4 dw = make_uint4(d[4 * t], d[4 * t + 1], d[4 * t + 2], d[4 * t + 3]);
#pragma unroll
      for (int ob = 0; ob < OB; ++ob) {
        dv[ob] = mfma_bf16(frag_cols<KS>(Os, 32 * b + 16 * t, 32 * ob, lane), pw, dv[ob]);
        dk[ob] = mfma_bf16(frag_cols<KS>(Qs, 32 * b + 16 * t, 32 * ob, lane), dw, dk[ob]);
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p[v] = np[v];
      if (DELTA_AHEAD) dl[v] = ndl[v];
    }
  }
  if (k < NT) {
    uint16_t* dst = a.out + ((int64_t)sample * NT + k) * tok + head * DH;
#pragma unroll
    for (int ob = 0; ob < OB; ++ob) {
      store_cols<KS>(dst + a.D, ob, hi, dk[ob]);
      store_cols<KS>(dst + 2 * a.D, ob, hi, dv[ob]);
    }
  }
}

// ---- fp32 --------------------------------------------------------------------------------------------------------------
// The same products on 32x32x2, where a wavefront with all keys of its 32 queries would be a chain of a thousand matrix
// instructions: a workgroup owns 32 queries (or keys) of one head, its two to eight wavefronts take the blocks of 32 keys
// (or queries) in turn, and maxima, sums and partial results meet in LDS, added in wavefront order.  An accumulator register
// is an operand as it is (lane half hi holds rows 8 g + 4 hi + i), the other operand's value comes straight from memory,
// whole rows of the head at a time; row operands are 16-byte pieces whose columns both sides take in one order.  Loads of a
// block go out together, without a branch between them, and before the wait for the other wavefronts where there is one.
// The backward keeps the gradient of the scores (contracting it again for dk cost more than its trip through memory).
// What bounds it: 4 samples x 3 heads x 324 tokens of width 64 are 132 workgroups of three chained blocks, 5 us of matrix
// time forward under 16 us of loads, products and two waits in turn; the chip is half empty.  As three and five kernels
// 26.7 us forward and 51 us backward, 16.4 and 25.7 us so; 32 x 12 x 196 of width 64 107 / 182 -> 82 / 163 us (matrix time
// 36 / 72 us), 64 x 8 x 64 of width 32 24.6 / 29.9 -> 9.6 / 17.7 us.
struct AttnArgs32 {
  const float* qkv;   // [B][NT][3 D]
  float* P;           // [B][heads][NT][NT]: written forward, read backward
  const float* dout;  // backward: [B][NT][D]
  float* out;         // forward: [B][NT][D]; backward: d qkv [B][NT][3 D]
  float* ds;          // backward: [B][heads][NT][NT], gradient of the scores
  int NT, D, heads, dh;
  int blocks;         // of 32 tokens
  int vec;            // rows of P and ds are whole, aligned 16-byte groups
  float scale;
};
__device__ __forceinline__ v16f_t mfma32(float4 a, float4 b, v16f_t c) {
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, c, 0, 0, 0);
}
// Rows of the head: row r of `base` (clamped to the last token) as row operand pieces, column 8 s + 4 hi.
template <int OB>
__device__ __forceinline__ void load_row32(float4 (&f)[4 * OB], const float* row, int dh, int hi) {
#pragma unroll
  for (int s = 0; s < 4 * OB; ++s) {  // a select, no branch: the loads have to be in flight together
    f[s] = *reinterpret_cast<const float4*>(row + min(8 * s, dh - 8) + 4 * hi);
    const bool in = 8 * s < dh;
    f[s].x = in ? f[s].x : 0.f;
    f[s].y = in ? f[s].y : 0.f;
    f[s].z = in ? f[s].z : 0.f;
    f[s].w = in ? f[s].w : 0.f;
  }
}
// The same rows for every wavefront of the workgroup: fetched once, in whole lines, and handed out through LDS (a row operand
// straight from memory touches 32 lines a load).
template <int OB, int W32>
__device__ __forceinline__ void share_rows32(float4 (&f)[4 * OB], float* red, const float* src, int64_t ld, int row0, int NT, int dh) {
  constexpr int PITCH = 32 * OB + 4;
  for (int i = threadIdx.x; i < 32 * 8 * OB; i += 64 * W32) {
    const int r = i / (8 * OB), c = 4 * (i % (8 * OB));
    float4 x = *reinterpret_cast<const float4*>(src + (int64_t)min(row0 + r, NT - 1) * ld + min(c, dh - 4));
    if (c >= dh) x = make_float4(0.f, 0.f, 0.f, 0.f);
    *reinterpret_cast<float4*>(red + r * PITCH + c) = x;
  }
  __syncthreads();
  const int l31 = threadIdx.x & 31, hi = threadIdx.x >> 5 & 1;
#pragma unroll
  for (int s = 0; s < 4 * OB; ++s) f[s] = *reinterpret_cast<const float4*>(red + l31 * PITCH + 8 * s + 4 * hi);
}
// Products with rows past the last token are none: whatever the last token holds must not reach a sum.
__device__ __forceinline__ void clear32(v16f_t& s, int row0, int NT, int hi) {
  if (row0 + 32 <= NT) return;
#pragma unroll
  for (int v = 0; v < 16; ++v)
    if (row0 + 8 * (v >> 2) + 4 * hi + (v & 3) >= NT) s[v] = 0.f;
}
// a . b over the head width for one block of 32 rows (given by the lane's row) against the lane's column.
template <int OB>
__device__ __forceinline__ v16f_t rows32(const float* row, const float4 (&col)[4 * OB], int dh, int hi) {
  float4 f[4 * OB];
  load_row32<OB>(f, row, dh, hi);
  v16f_t s = zero16();
#pragma unroll
  for (int k = 0; k < 4 * OB; ++k) s = mfma32(f[k], col[k], s);
  return s;
}
// acc[ob][j][.] += sum over 32 rows of src[row][32 ob + j] * x[row]; x as an accumulator holds it.  Loads and products apart,
// so that the loads can be on their way before a wait that the products need.
template <int OB>
__device__ __forceinline__ void cols_load32(float (&f)[OB][16], const float* src, int64_t ld, int row0, int NT, int dh, int lane) {
  const int l31 = lane & 31, hi = lane >> 5;
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) {
    const float* p = src + min(32 * ob + l31, dh - 1);  // columns past the head only reach results that are not stored
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = row0 + 8 * (v >> 2) + 4 * hi + (v & 3);
      f[ob][v] = p[(int64_t)min(r, NT - 1) * ld];
    }
  }
}
template <int OB>
__device__ __forceinline__ void cols_mul32(v16f_t (&acc)[OB], const float (&f)[OB][16], const v16f_t& x, int row0, int NT, int hi) {
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) {
    v16f_t y;
#pragma unroll
    for (int v = 0; v < 16; ++v) y[v] = f[ob][v];
    clear32(y, row0, NT, hi);
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(y[v], x[v], acc[ob], 0, 0, 0);
  }
}
// The wavefronts' partial results, added in wavefront order: each finishes some groups of four columns of the lanes' tokens
// and stores them at dst + column (nullptr: nothing to store).
template <int OB, int W32>
__device__ __forceinline__ void finish32(const v16f_t (&acc)[OB], float* red, float* dst, int dh, int wave, int lane) {
  const int hi = lane >> 5;
  __syncthreads();  // red is free
#pragma unroll
  for (int ob = 0; ob < OB; ++ob)
#pragma unroll
    for (int v = 0; v < 16; ++v) red[((wave * OB + ob) * 16 + v) * 64 + lane] = acc[ob][v];
  __syncthreads();
  for (int g = wave; g < 4 * OB; g += W32) {
    const int j = 8 * g + 4 * hi;
    float r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* x = red + (4 * g + i) * 64 + lane;
      r[i] = x[0];
#pragma unroll
      for (int w = 1; w < W32; ++w) r[i] += x[w * OB * 1024];
    }
    if (dst != nullptr && j < dh) *reinterpret_cast<float4*>(dst + j) = make_float4(r[0], r[1], r[2], r[3]);
  }
}
// Probabilities of the lane's query (nullptr: none) for one block of keys, as an accumulator holds them; zero past the last.
__device__ __forceinline__ void load_p32(v16f_t& p, const float* row, int k0, int NT, int vec, int hi) {
  if (row == nullptr) {
    p = zero16();
    return;
  }
  if (vec) {  // NT is a multiple of four: a piece is all in or all out
    float4 f[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) f[g] = *reinterpret_cast<const float4*>(row + min(k0 + 8 * g + 4 * hi, NT - 4));
#pragma unroll
    for (int g = 0; g < 4; ++g) { p[4 * g] = f[g].x; p[4 * g + 1] = f[g].y; p[4 * g + 2] = f[g].z; p[4 * g + 3] = f[g].w; }
  } else {
#pragma unroll
    for (int v = 0; v < 16; ++v) p[v] = row[min(k0 + 8 * (v >> 2) + 4 * hi + (v & 3), NT - 1)];
  }
  clear32(p, k0, NT, hi);
}
__device__ __forceinline__ void store_p32(float* row, const v16f_t& p, int k0, int NT, int vec, int hi) {
  if (row == nullptr) return;
  if (vec) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (k0 + 8 * g + 4 * hi < NT)
        *reinterpret_cast<float4*>(row + k0 + 8 * g + 4 * hi) = make_float4(p[4 * g], p[4 * g + 1], p[4 * g + 2], p[4 * g + 3]);
    return;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v)
    if (const int k = k0 + 8 * (v >> 2) + 4 * hi + (v & 3); k < NT) row[k] = p[v];
}
// Sum / maximum over the lane pair of a query and the wavefronts; every lane of the query gets it.
template <bool MAX, int W32>
__device__ __forceinline__ float across32(float v, float* red, int wave, int lane) {
  const float o = __shfl_xor(v, 32, 64);
  v = MAX ? fmaxf(v, o) : v + o;
  __syncthreads();
  if (lane < 32) red[wave * 32 + lane] = v;
  __syncthreads();
  v = red[lane & 31];
#pragma unroll
  for (int w = 1; w < W32; ++w) {
    const float x = red[w * 32 + (lane & 31)];
    v = MAX ? fmaxf(v, x) : v + x;
  }
  return v;
}

template <int OB, int W32, int NBW>
__global__ __launch_bounds__(64 * W32, 2) void attn_fwd32_kernel(const AttnArgs32 a) {
  __shared__ __attribute__((aligned(16))) float red[W32 * OB * 1024];
  const int NT = a.NT, dh = a.dh;
  const int id = xcd_block_cyclic(blockIdx.x, gridDim.x, a.blocks), z = id / a.blocks, sample = z / a.heads, head = z % a.heads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l31 = lane & 31, hi = lane >> 5;
  const int q = (id % a.blocks) * 32 + l31;
  const int64_t tok = 3ll * a.D;
  const float* base = a.qkv + (int64_t)sample * NT * tok + head * dh;
  float4 qf[4 * OB];
  share_rows32<OB, W32>(qf, red, base, tok, q - l31, NT, dh);
  v16f_t s[NBW];
  float m = -INFINITY;
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int k0 = 32 * (wave + W32 * t);
    if (k0 >= NT) continue;
    s[t] = rows32<OB>(base + a.D + (int64_t)min(k0 + l31, NT - 1) * tok, qf, dh, hi);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      if (k0 + 8 * (v >> 2) + 4 * hi + (v & 3) >= NT) s[t][v] = -INFINITY;
      m = fmaxf(m, s[t][v]);
    }
  }
  const float c = a.scale * 1.44269504088896340736f;
  m = across32<true, W32>(m, red, wave, lane) * c;  // finite: key 0 is always there
  float sum = 0.f;
#pragma unroll
  for (int t = 0; t < NBW; ++t)
    if (32 * (wave + W32 * t) < NT) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[t][v] = exp2f(fmaf(s[t][v], c, -m));
        sum += s[t][v];
      }
    }
  float f[OB][16];
  cols_load32<OB>(f, base + 2 * a.D, tok, 32 * wave, NT, dh, lane);
  const float inv = 1.f / across32<false, W32>(sum, red, wave, lane);
  float* prow = q < NT ? a.P + ((int64_t)z * NT + q) * NT : nullptr;
  v16f_t o[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) o[ob] = zero16();
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int k0 = 32 * (wave + W32 * t);
    if (k0 >= NT) continue;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[t][v] *= inv;
    store_p32(prow, s[t], k0, NT, a.vec, hi);
    if (t > 0) cols_load32<OB>(f, base + 2 * a.D, tok, k0, NT, dh, lane);
    cols_mul32<OB>(o, f, s[t], k0, NT, hi);
  }
  finish32<OB, W32>(o, red, q < NT ? a.out + ((int64_t)sample * NT + q) * a.D + head * dh : nullptr, dh, wave, lane);
}

// dq of 32 queries, leaving the gradient of the scores behind; and dv or dk of 32 keys: the same sum over the queries, of
// probabilities times output gradient or of score gradient times q.  dv needs nothing of dq and shares its launch.
template <int OB, int W32, int NBW>
__device__ __forceinline__ void attn_dq32(const AttnArgs32& a, float* red, int id) {
  const int NT = a.NT, dh = a.dh, z = id / a.blocks, sample = z / a.heads, head = z % a.heads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l31 = lane & 31, hi = lane >> 5;
  const int q = (id % a.blocks) * 32 + l31;
  const int64_t tok = 3ll * a.D;
  const float* base = a.qkv + (int64_t)sample * NT * tok + head * dh;
  const float* prow = q < NT ? a.P + ((int64_t)z * NT + q) * NT : nullptr;
  float* drow = q < NT ? a.ds + ((int64_t)z * NT + q) * NT : nullptr;
  float4 df[4 * OB];
  share_rows32<OB, W32>(df, red, a.dout + (int64_t)sample * NT * a.D + head * dh, a.D, q - l31, NT, dh);
  v16f_t s[NBW], p[NBW];
  float delta = 0.f;
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int k0 = 32 * (wave + W32 * t);
    if (k0 >= NT) continue;
    load_p32(p[t], prow, k0, NT, a.vec, hi);
    s[t] = rows32<OB>(base + 2 * a.D + (int64_t)min(k0 + l31, NT - 1) * tok, df, dh, hi);
    clear32(s[t], k0, NT, hi);
#pragma unroll
    for (int v = 0; v < 16; ++v) delta = fmaf(p[t][v], s[t][v], delta);
  }
  float f[OB][16];
  cols_load32<OB>(f, base + a.D, tok, 32 * wave, NT, dh, lane);
  delta = across32<false, W32>(delta, red, wave, lane);
  v16f_t o[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) o[ob] = zero16();
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int k0 = 32 * (wave + W32 * t);
    if (k0 >= NT) continue;
    if (t > 0) cols_load32<OB>(f, base + a.D, tok, k0, NT, dh, lane);
#pragma unroll
    for (int v = 0; v < 16; ++v) s[t][v] = p[t][v] * (s[t][v] - delta) * a.scale;
    store_p32(drow, s[t], k0, NT, a.vec, hi);
    cols_mul32<OB>(o, f, s[t], k0, NT, hi);
  }
  finish32<OB, W32>(o, red, q < NT ? a.out + ((int64_t)sample * NT + q) * tok + head * dh : nullptr, dh, wave, lane);
}
template <int OB, int W32>
__device__ __forceinline__ void attn_dkv32(const AttnArgs32& a, float* red, int id, bool dv) {
  const int NT = a.NT, dh = a.dh, z = id / a.blocks, sample = z / a.heads, head = z % a.heads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l31 = lane & 31, hi = lane >> 5;
  const int k = (id % a.blocks) * 32 + l31;
  const int64_t tok = 3ll * a.D, ld = dv ? a.D : tok;
  const float* y = (dv ? a.dout : a.qkv) + (int64_t)sample * NT * ld + head * dh;
  const float* x = (dv ? a.P : a.ds) + (int64_t)z * NT * NT + min(k, NT - 1);
  auto load = [&](v16f_t& p, float (&f)[OB][16], int q0) {
#pragma unroll
    for (int v = 0; v < 16; ++v) p[v] = x[(int64_t)min(q0 + 8 * (v >> 2) + 4 * hi + (v & 3), NT - 1) * NT];
    cols_load32<OB>(f, y, ld, q0, NT, dh, lane);
  };
  v16f_t o[OB], p[2];
  float f0[OB][16], f1[OB][16];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) o[ob] = zero16();
  constexpr int STEP = 32 * W32;
  if (32 * wave < NT) {
    if constexpr (OB < 3) {
      load(p[0], f0, 32 * wave);
      for (int q0 = 32 * wave; q0 < NT; q0 += 2 * STEP) {
        if (q0 + STEP < NT) load(p[1], f1, q0 + STEP);
        clear32(p[0], q0, NT, hi);
        cols_mul32<OB>(o, f0, p[0], q0, NT, hi);
        if (q0 + STEP >= NT) break;
        if (q0 + 2 * STEP < NT) load(p[0], f0, q0 + 2 * STEP);
        clear32(p[1], q0 + STEP, NT, hi);
        cols_mul32<OB>(o, f1, p[1], q0 + STEP, NT, hi);
      }
    } else {  // two blocks of a wide head at once do not fit the registers
      for (int q0 = 32 * wave; q0 < NT; q0 += STEP) {
        load(p[0], f0, q0);
        clear32(p[0], q0, NT, hi);
        cols_mul32<OB>(o, f0, p[0], q0, NT, hi);
      }
    }
  }
  finish32<OB, W32>(o, red, k < NT ? a.out + ((int64_t)sample * NT + k) * tok + (dv ? 2 : 1) * a.D + head * dh : nullptr, dh, wave, lane);
}
template <int OB, int W32, int NBW>
__global__ __launch_bounds__(64 * W32, 2) void attn_bwd_dq_dv32_kernel(const AttnArgs32 a) {
  __shared__ __attribute__((aligned(16))) float red[W32 * OB * 1024];
  const int id = xcd_block_cyclic(blockIdx.x, gridDim.x, a.blocks), n = gridDim.x / 2;
  if (id < n) attn_dq32<OB, W32, NBW>(a, red, id);
  else attn_dkv32<OB, W32>(a, red, id - n, true);
}
template <int OB, int W32>
__global__ __launch_bounds__(64 * W32, 2) void attn_bwd_dk32_kernel(const AttnArgs32 a) {
  __shared__ __attribute__((aligned(16))) float red[W32 * OB * 1024];
  attn_dkv32<OB, W32>(a, red, xcd_block_cyclic(blockIdx.x, gridDim.x, a.blocks), false);
}

template <int OB, int W32, int NBW>
hipError_t launch_attn32_w(const AttnArgs32& a, bool backward, int batch, hipStream_t stream) {
  const unsigned n = (unsigned)batch * (unsigned)a.blocks;
  if (!backward) {
    hipLaunchKernelGGL((attn_fwd32_kernel<OB, W32, NBW>), dim3(n), dim3(64 * W32), 0, stream, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((attn_bwd_dq_dv32_kernel<OB, W32, NBW>), dim3(2 * n), dim3(64 * W32), 0, stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_bwd_dk32_kernel<OB, W32>), dim3(n), dim3(64 * W32), 0, stream, a);
  return hipGetLastError();
}
// As many wavefronts as there are blocks of 32 tokens, up to eight, and then as many blocks for each as it takes; with
// more than two workgroups per CU to run, two of four wavefronts on a CU rather than one of eight, whose waits the other
// one fills (32 x 12 x 196 of width 64: 94 / 230 -> 82 / 163 us, 16 x 8 x 512 161 / 333 -> 132 / 281 us).
template <int OB>
hipError_t launch_attn32_ob(const AttnArgs32& a, bool backward, int batch, hipStream_t stream) {
  if (a.blocks <= 2) return launch_attn32_w<OB, 2, 1>(a, backward, batch, stream);
  if (a.blocks <= 4) return launch_attn32_w<OB, 4, 1>(a, backward, batch, stream);
  if (a.blocks <= 8 && batch * a.blocks > 512) return launch_attn32_w<OB, 4, 2>(a, backward, batch, stream);
  if (a.blocks <= 8) return launch_attn32_w<OB, 8, 1>(a, backward, batch, stream);
  if (a.blocks <= 16 && batch * a.blocks > 512) return launch_attn32_w<OB, 4, 4>(a, backward, batch, stream);
  if (a.blocks <= 16) return launch_attn32_w<OB, 8, 2>(a, backward, batch, stream);
  return launch_attn32_w<OB, 8, 4>(a, backward, batch, stream);
}
hipError_t launch_attn32(const AttnArgs32& a, bool backward, int batch, hipStream_t stream) {
  if (batch <= 0 || batch > 65535 || a.blocks > 32) return hipErrorInvalidValue;
  if (a.dh <= 32) return launch_attn32_ob<1>(a, backward, batch, stream);
  if (a.dh <= 64) return launch_attn32_ob<2>(a, backward, batch, stream);
  return launch_attn32_ob<3>(a, backward, batch, stream);
}
constexpr size_t ATTN_LDS = 160 * 1024;
size_t attn_lds(int NT, int dh) {
  const size_t pitch = dh == 64 ? dh : dh + 8;
  // the transposing reads of a head whose width is an odd multiple of 16 run 16 columns past the last row
  return 2 * (size_t)((NT + 15) & ~15) * pitch * 2 + 64;
}

template <typename K>
hipError_t launch_attn(K kernel, const AttnArgs& a, int batch, size_t lds, hipStream_t stream) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3((unsigned)batch * (unsigned)a.blocks), dim3(256), lds, stream, a);
  return hipGetLastError();
}
template <int KS>
hipError_t launch_attn_ks(const AttnArgs& a, int pass, int batch, size_t lds, hipStream_t stream) {
  if (pass == 1) return launch_attn(&attn_bwd_dq_kernel<KS>, a, batch, lds, stream);
  if (pass == 2) return launch_attn(&attn_bwd_dkv_kernel<KS>, a, batch, lds, stream);
  if (a.NT <= 64) return launch_attn(&attn_fwd_kernel<KS, 2>, a, batch, lds, stream);
  if (a.NT <= 128) return launch_attn(&attn_fwd_kernel<KS, 4>, a, batch, lds, stream);
  if (a.NT <= 256) return launch_attn(&attn_fwd_kernel<KS, 8>, a, batch, lds, stream);
  return launch_attn(&attn_fwd_kernel<KS, 0>, a, batch, lds, stream);
}
hipError_t launch_attn_pass(const AttnArgs& a, int dh, int pass, int batch, hipStream_t stream) {
  if (batch <= 0 || batch > 65535) return hipErrorInvalidValue;
  const size_t lds = attn_lds(a.NT, dh);
  switch (dh / 16) {
    case 1: return launch_attn_ks<1>(a, pass, batch, lds, stream);
    case 2: return launch_attn_ks<2>(a, pass, batch, lds, stream);
    case 3: return launch_attn_ks<3>(a, pass, batch, lds, stream);
    case 4: return launch_attn_ks<4>(a, pass, batch, lds, stream);
    default: return launch_attn_ks<5>(a, pass, batch, lds, stream);
  }
}
bool aligned(const void* p, size_t n) { return reinterpret_cast<uintptr_t>(p) % n == 0; }
AttnArgs attn_args(const void* qkv, const void* P, int B, int NT, int D, int heads) {
  AttnArgs a;
  a.qkv = static_cast<const uint16_t*>(qkv);
  a.P = static_cast<uint16_t*>(const_cast<void*>(P));
  a.dout = nullptr; a.out = nullptr; a.delta = nullptr;
  a.NT = NT; a.D = D; a.heads = heads;
  a.blocks = (NT + 127) / 128;
  a.vec = NT % 4 == 0 && aligned(P, 8);
  a.dvec = 0;
  a.scale = 1.0f / sqrtf((float)(D / heads));
  return a;
}

AttnArgs32 attn_args32(const void* qkv, const void* P, int NT, int D, int heads) {
  AttnArgs32 a;
  a.qkv = static_cast<const float*>(qkv);
  a.P = static_cast<float*>(const_cast<void*>(P));
  a.dout = nullptr; a.out = nullptr; a.ds = nullptr;
  a.NT = NT; a.D = D; a.heads = heads; a.dh = D / heads;
  a.blocks = (NT + 31) / 32;
  a.vec = NT % 4 == 0 && aligned(P, 16);
  a.scale = 1.0f / sqrtf((float)a.dh);
  return a;
}

}  // namespace

// bf16: heads whose width is a whole number of 16-wide reduction steps up to 80 (the accumulators of a wider one leave a
// single workgroup per CU), two tiles of all tokens in LDS; the launches below also want aligned rows.
// fp32: three accumulators of 32 columns at most.  Long sequences in many heads run as well as products of whole matrices
// (16 x 8 x 512 of width 64: 270 us backward against 281 us, 4 x 8 x 1024 271 against 296 us; 16 x 8 x 384 157 against
// 148 us, 1 x 8 x 1024 134 against 73 us), unless their rows end inside a 16-byte piece (8 x 12 x 577: 495 against 399 us);
// forward the kernel is the faster one there too (152 against 142 us).
// bf16 backward of more tokens than leave room for a second workgroup on a CU, in rows of whole 8-byte groups (where separate kernels do
// not go element by element): heads of width 48, whose products are padded to 64 columns, are faster in separate kernels when the
// last round of workgroups is not full, and only up to 1.18 times slower when it is (us, separate / here: 72 heads x 416 tokens 88 / 124, 48 x 656
// 153 / 199, 96 x 500 141 / 156, 96 x 600 215 / 191, 4 x 624 70 / 63); heads of width 80 with a second round of few or a first of very
// few (72 x 416 124 / 137, 4 x 384 45 / 47; 64 x 416 120 / 72).
bool attention_fused(bool backward, int B, int NT, int D, int heads, int dtype) {
  if (heads <= 0 || NT <= 0 || D % heads) return false;
  const int dh = D / heads;
  if (dtype == DT_F32) {
    const int64_t blocks = (NT + 31) / 32;
    if (dh % 8 || dh > 96 || NT > 1024) return false;
    return !backward || blocks <= 8 || NT % 4 != 0 || (int64_t)B * heads * blocks * blocks <= 24576;
  }
  if (dh % 16 || dh > 80 || attn_lds(NT, dh) > ATTN_LDS) return false;
  if (backward && NT % 4 == 0 && attn_lds(NT, dh) > ATTN_LDS / 2) {
    const int64_t wgs = (int64_t)B * heads * ((NT + 127) / 128);
    if (dh == 48 || (dh == 80 && NT > 370 && (wgs < 32 || (wgs > 256 && wgs <= 320)))) return false;
  }
  return true;
}
bool attention_fused_fwd_ok(const void* qkv, const void* out, int B, int NT, int D, int heads, int dtype) {
  return attention_fused(false, B, NT, D, heads, dtype) && aligned(qkv, 16) && aligned(out, dtype == DT_F32 ? 16 : 8);
}
bool attention_fused_bwd_ok(const void* qkv, const void* dout, const void* dqkv, int B, int NT, int D, int heads, int dtype) {
  return attention_fused(true, B, NT, D, heads, dtype) && aligned(qkv, 16) && aligned(dout, 16) && aligned(dqkv, dtype == DT_F32 ? 16 : 8);
}

hipError_t launch_attention_fused_fwd(const void* qkv, void* P, void* out, int B, int NT, int D, int heads, int dtype, hipStream_t stream) {
  if (dtype == DT_F32) {
    AttnArgs32 f = attn_args32(qkv, P, NT, D, heads);
    f.out = static_cast<float*>(out);
    return launch_attn32(f, false, B * heads, stream);
  }
  AttnArgs a = attn_args(qkv, P, B, NT, D, heads);
  a.out = static_cast<uint16_t*>(out);
  return launch_attn_pass(a, D / heads, 0, B * heads, stream);
}
hipError_t launch_attention_fused_bwd(const void* qkv, const void* P, const void* dout, void* dqkv, float* ws, int B, int NT, int D, int heads,
                                      int dtype, hipStream_t stream) {
  if (dtype == DT_F32) {
    AttnArgs32 f = attn_args32(qkv, P, NT, D, heads);
    f.dout = static_cast<const float*>(dout);
    f.out = static_cast<float*>(dqkv);
    f.ds = ws;
    f.vec = f.vec && aligned(ws, 16);
    return launch_attn32(f, true, B * heads, stream);
  }
  AttnArgs a = attn_args(qkv, P, B, NT, D, heads);
  a.dout = static_cast<const uint16_t*>(dout);
  a.out = static_cast<uint16_t*>(dqkv);
  a.delta = ws;
  a.dvec = NT % 4 == 0 && aligned(ws, 16);
  hipError_t e = launch_attn_pass(a, D / heads, 1, B * heads, stream);
  return e != hipSuccess ? e : launch_attn_pass(a, D / heads, 2, B * heads, stream);
}

}  // namespace cdp
