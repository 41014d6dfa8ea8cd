// sk_affd_tt.hip -- AFFD transposes (eq. bami, adjoint) for D > 1024 and a last
// digit of 1024, up to kMaxPtrs layers per launch.
//
// Coordinates of a layer are (t, p, l): top digits t (TT values), digit p
// (dk1), last digit l (1024).  The D entries of z enter at one value h* of the
// top digits, so with unnormalised transforms
//   u[p, l] = (H_p (x) H_l) Scatter_{pi2_p, pi2_l} z          (one slab)
//   (H_TT G H_TT e_{h*}) u = M[t] u,  M = H_TT (c . g), c_t = (-1)^<h*, t>,
//   x[j] = b_j Y[t'][pi1_p(p), pi1_l(l)] / sqrt(N' D),
//   Y[t'] = (H_p (x) H_l)(M[t'] . u),  t' = pi1(top digits of j),
// the adjoint of the forward's slab sum, with the M that the forward stores.
// Three launches per group of layers:
//   A  rows a of z: columns scattered through pi2_l, H_l        -> U[a][l]
//   B  columns l: rows scattered through pi2_p, H_p, times M[t'] (or, TT = 1
//      and dk1 < 1024, the regenerated g), H_p                  -> W[t][p][l]
//   C  output rows h = (t, p): row pi1_p(p) of W[t], H_l, pi1_l, signs,
//      theta0, one write.
// Only slabs and rows behind real outputs are formed; slab t of W is the one
// of the source digits t, so that they are the first ceil(n / 2^20).
// Bytes per output: write and read W, read M and theta0, write x (20 with fp32
// outputs, against 8 for x and theta0 alone).  The per-layer chain of generic
// passes it replaces (a zero fill, a scatter, two N'-point transforms of two to
// three passes each, a multiply that regenerates N' Gaussians and an output
// pass: 7 to 11 launches and 60 bytes per padded entry) took 3.2 ms of a
// 3.8 ms intrinsic-dimension step over three GPT-2 blocks (38 layers, one
// vector); the launches here take 0.14 ms.
#include <algorithm>
#include <cmath>

#include "sk_kcommon.h"
#include "sk_launch.h"

namespace sk {

// The four transforms of a layer are unnormalised, sqrt(N' D) in all: 2^-10 of
// it goes in between the first two and the last two, so that intermediates stay
// near the input's size (powers of two: the same bits).
constexpr float kMidScale = 1.0f / 1024.0f;

// ---- A ---------------------------------------------------------------------
// Workgroup per 8 rows a, vector and layer: thread (i = tid / 32, c = tid % 32)
// reads columns c + 32 k of row i through pi2_l^{-1} (4 KB of z, in L1).
__global__ __launch_bounds__(256) void k_affdTT_zrows(const LayerDesc *__restrict__ layers,
                                                      const uint16_t *__restrict__ ptab, AffdTTGroup g,
                                                      const float *__restrict__ z, int R, int64_t D,
                                                      int64_t b_begin, float *__restrict__ ws) {
  using L = Lds1024<8>;
  __shared__ __align__(16) float s[L::kFloats];
  const LayerDesc &ld = layers[g.layer[blockIdx.z]];
  const uint16_t *inv = ptab + ld.poff[1][1][ld.K - 1];
  const int64_t v = blockIdx.y;
  const int i = threadIdx.x >> 5, c = threadIdx.x & 31;
  const int a = blockIdx.x * 8 + i;
  const float *zr = z + (b_begin + v) * D + (int64_t)(a < R ? a : 0) * 1024;
  float e[32];
#pragma unroll
  for (int k = 0; k < 32; ++k) e[k] = a < R ? zr[inv[c + 32 * k]] : 0.0f;
  fwht1024_lds_regs<8>(s, e);
  float *u = ws + g.u_off[blockIdx.z] + v * D;
  for (int r = 0; r < 8 && blockIdx.x * 8 + r < R; ++r)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int l = threadIdx.x + 256 * k;
      u[(int64_t)(blockIdx.x * 8 + r) * 1024 + l] = s[L::idx(r, l)];
    }
}

// ---- B, dk1 = 1024 with the stored M ------------------------------------------
// Workgroup (1024 threads) per 32 columns l, vector and run of spw slabs.
// Thread (ri = tid % 32, rc = tid / 32) works on column l = c0 + ri: u stays in
// registers (p = 32 rc + m) over the slabs; M[t'][l][.] (4 KB rows) is loaded
// by whole rows one slab ahead and turned through LDS; the product goes through
// H_p (low bits in registers, one LDS exchange, high bits) and row p = rc + 32 k
// of W leaves as one 128-byte line per half-wave.  One workgroup per CU: the
// M row loads of the next slab are in flight during the transform.
__global__ __launch_bounds__(1024) void k_affdTT_cols(const LayerDesc *__restrict__ layers,
                                                      const uint16_t *__restrict__ ptab, AffdTTGroup g,
                                                      int64_t D, float *__restrict__ ws) {
  using L = Lds1024R32;
  __shared__ float s[L::kFloats];
  int gl = 0;
  while (gl + 1 < g.n && blockIdx.x >= g.blk0[gl + 1]) ++gl;
  const LayerDesc &ld = layers[g.layer[gl]];
  const uint32_t b = blockIdx.x - g.blk0[gl];
  const int c0 = (int)(b & 31) * 32;
  const int t0 = (int)(b >> 5) * g.spw;
  const int nlive = (int)((ld.rows_live + 1023) >> 10);
  const int t1 = min(t0 + g.spw, nlive);
  const int64_t v = blockIdx.y;
  const int tid = threadIdx.x, ri = tid & 31, rc = tid >> 5;
  const uint16_t *inv2 = ptab + ld.poff[1][1][ld.K - 2];
  const uint16_t *inv1 = ptab + ld.poff[0][1][ld.K - 2];
  float *high = s + ri * L::kStride + rc;       // p = rc + 32 k at 33 k
  float *low = s + ri * L::kStride + 33 * rc;   // p = 32 rc + m at m
  auto slab = [&](int t) {  // pi1 of the top digits of t
    int64_t ts = 0, stride = 1;
    for (int k = ld.K - 3; k >= 0; --k) {
      const int64_t dig = (t / stride) & ((1ll << ld.lg[k]) - 1);
      ts += (int64_t)ptab[ld.poff[0][0][k] + dig] * stride;
      stride <<= ld.lg[k];
    }
    return ts;
  };
  float mreg[32], u[32];
  // row offsets in scalars: 96 values per thread leave no registers for addresses
  auto fetch = [&](int t) {
    const __amdgpu_buffer_rsrc_t mr = buf_rsrc(g.m[gl] + (slab(t) << 20) + (int64_t)c0 * 1024, 32 * 4096);
#pragma unroll
    for (int k = 0; k < 32; ++k) mreg[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(mr, tid * 4, k * 4096, 0));
  };
  {
    // rows a >= R lie past the resource and read zero
    const __amdgpu_buffer_rsrc_t ur = buf_rsrc(ws + g.u_off[gl] + v * D, (uint32_t)(D * 4));
#pragma unroll
    for (int k = 0; k < 32; ++k)
      u[k] = __uint_as_float(
          __builtin_amdgcn_raw_buffer_load_b32(ur, (int)inv2[rc + 32 * k] * 4096 + (c0 + ri) * 4, 0, 0));
  }
  fetch(t0);
  fwht_regs_t<32>(u);
#pragma unroll
  for (int k = 0; k < 32; ++k) high[33 * k] = u[k];
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 32; ++m) u[m] = low[m] * kMidScale;
  fwht_regs_t<32>(u);
  for (int t = t0; t < t1; ++t) {
    __syncthreads();  // the block's last readers are done
#pragma unroll
    for (int k = 0; k < 32; ++k) s[k * L::kStride + tid + (tid >> 5)] = mreg[k];
    if (t + 1 < t1) fetch(t + 1);
    __syncthreads();
    float x[32];
#pragma unroll
    for (int m = 0; m < 32; ++m) x[m] = low[m] * u[m];
    fwht_regs_t<32>(x);
#pragma unroll
    for (int m = 0; m < 32; ++m) low[m] = x[m];  // the places this thread has just read
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 32; ++k) x[k] = high[33 * k];
    fwht_regs_t<32>(x);
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(ws + g.w_off[gl] + ((v * nlive + t) << 20), 1u << 22);
    const int voff = rc * 4096 + (c0 + ri) * 4;
    const int64_t live = ld.rows_live - (int64_t)t * 1024;  // source rows of the slab
    if (live >= 1024) {
#pragma unroll
      for (int k = 0; k < 32; ++k)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[k]), wr, voff, k * 32 * 4096, 0);
    } else {
#pragma unroll
      for (int k = 0; k < 32; ++k)
        if (inv1[rc + 32 * k] < live)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[k]), wr, voff, k * 32 * 4096, 0);
    }
  }
}

// ---- B, one slab of dk1 < 1024 rows --------------------------------------------
// Workgroup per 2^lgcs columns (a tile of at most 2^LGT values in LDS), layer
// and every gridDim.y-th vector; the tile's g (from four consecutive columns'
// Philox block) stays in registers over the vectors.
template <int NG>
__device__ __forceinline__ void affd_tile_gauss(const LayerDesc &ld, int lgcs, int c0, int tot, Key key,
                                                float (&gg)[NG][4]) {
  const int cmask = (1 << lgcs) - 1;
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int e = 4 * threadIdx.x + 1024 * i;  // lgcs >= 5: four columns of one row
    if (e < tot) {
      gauss4((uint64_t)((e >> lgcs) * 1024 + c0 + (e & cmask)) >> 2, (uint32_t)ld.layer_id, ST_GAUSS, key, gg[i]);
#pragma unroll
      for (int q = 0; q < 4; ++q) gg[i][q] *= kMidScale;
    }
  }
}
// H_p, g, H_p on the filled tile (rows above bit lgcs); starts and ends synchronised.
template <int NG>
__device__ __forceinline__ void affd_tile_HgH(float *s, int lg, int lgcs, int tot, const float (&gg)[NG][4]) {
  lds_fwht_regs(s, lg, lgcs);
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int e = 4 * threadIdx.x + 1024 * i;
    if (e < tot) {
#pragma unroll
      for (int q = 0; q < 4; ++q) s[p16(e) + q] *= gg[i][q];
    }
  }
  lds_fwht_regs(s, lg, lgcs);
}

template <int LGT>
__global__ __launch_bounds__(256) void k_affdTT_cols_s(const LayerDesc *__restrict__ layers,
                                                       const uint16_t *__restrict__ ptab, AffdTTGroup g, int R,
                                                       int64_t D, int64_t bc, float *__restrict__ ws, Key key) {
  constexpr int NG = 1 << (LGT - 10);  // groups of four values per thread
  __shared__ __align__(16) float s[p16_floats(1 << LGT)];
  int gl = 0;
  while (gl + 1 < g.n && blockIdx.x >= g.blk0[gl + 1]) ++gl;
  const LayerDesc &ld = layers[g.layer[gl]];
  const int lgcs = min(10, LGT - ld.lgdk1);
  const int c0 = (int)(blockIdx.x - g.blk0[gl]) << lgcs;
  const int cmask = (1 << lgcs) - 1, tot = ld.dk1 << lgcs;
  const uint16_t *inv2 = ptab + ld.poff[1][1][ld.K - 2];
  const uint16_t *inv1 = ptab + ld.poff[0][1][ld.K - 2];
  float gg[NG][4];
  affd_tile_gauss<NG>(ld, lgcs, c0, tot, key, gg);
  for (int64_t v = blockIdx.y; v < bc; v += gridDim.y) {
    const float *u = ws + g.u_off[gl] + v * D + c0;
    for (int e = threadIdx.x; e < tot; e += 256) {
      const int a = inv2[e >> lgcs];
      s[p16(e)] = a < R ? u[(int64_t)a * 1024 + (e & cmask)] : 0.0f;
    }
    affd_tile_HgH<NG>(s, ld.lgdk1 + lgcs, lgcs, tot, gg);
    float *w = ws + g.w_off[gl] + v * ld.np + c0;
    for (int e = threadIdx.x; e < tot; e += 256) {
      const int p = e >> lgcs;
      if (inv1[p] < ld.rows_live) w[(int64_t)p * 1024 + (e & cmask)] = s[p16(e)];
    }
    __syncthreads();  // the tile is free for the next vector
  }
}

// ---- C ---------------------------------------------------------------------
// Workgroup per 8 output rows and vector: row h of the output is row pi1_p of
// its slab of W (4 KB, read in 128-byte pieces), H_l, then each thread gathers
// four consecutive outputs per row through pi1_l.
__global__ __launch_bounds__(256) void k_affdTT_out(const LayerDesc *__restrict__ layers,
                                                    const uint16_t *__restrict__ ptab, AffdTTGroup g, int64_t D,
                                                    int64_t b_begin, const float *__restrict__ ws, int out_dtype,
                                                    Key key) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  typedef uint16_t h4u __attribute__((ext_vector_type(4), aligned(2)));
  using L = Lds1024<8>;
  __shared__ __align__(16) float s[L::kFloats];
  __shared__ __align__(16) uint32_t sgn[8 * 32];
  int gl = 0;
  while (gl + 1 < g.n && blockIdx.x >= g.blk0[gl + 1]) ++gl;
  const LayerDesc &ld = layers[g.layer[gl]];
  const int64_t h0 = (int64_t)(blockIdx.x - g.blk0[gl]) * 8, v = blockIdx.y;
  const int i = threadIdx.x >> 5, c = threadIdx.x & 31;
  {
    const int64_t h = h0 + i;
    const int64_t per_v = ((ld.rows_live + ld.dk1 - 1) >> ld.lgdk1) << (ld.lgdk1 + 10);
    const float *w = ws + g.w_off[gl] + v * per_v;
    float e[32];
    if (h < ld.rows_live) {
      const int64_t p = ptab[ld.poff[0][0][ld.K - 2] + (h & (ld.dk1 - 1))];
      w += ((h >> ld.lgdk1) << (ld.lgdk1 + 10)) + p * 1024 + c;
#pragma unroll
      for (int k = 0; k < 32; ++k) e[k] = w[32 * k];
    } else {
#pragma unroll
      for (int k = 0; k < 32; ++k) e[k] = 0.0f;
    }
    if (threadIdx.x < 64) {  // one Philox block per 128 coordinates
      const W4 wd = philox((uint64_t)h0 * 8u + threadIdx.x, (uint32_t)ld.layer_id, ST_SIGN, key);
      *reinterpret_cast<uint4 *>(&sgn[4 * threadIdx.x]) = make_uint4(wd.w[0], wd.w[1], wd.w[2], wd.w[3]);
    }
    fwht1024_lds_regs<8>(s, e);
  }
  const float sc = g.scale[gl];
  const float *th = g.th[gl];
  const int col = 4 * threadIdx.x;
  int idx[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) idx[q] = ptab[ld.poff[0][0][ld.K - 1] + col + q];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int64_t j = (h0 + r) * 1024 + col;
    const int64_t lim = ld.n - j;
    if (lim <= 0) break;
    const uint32_t bits = sgn[r * 32 + (col >> 5)] >> (col & 31);
    float o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = flip(s[L::idx(r, idx[q])] * sc, (bits >> q) & 1u);
    const int64_t pos = (b_begin + v) * ld.n + j;
    if (lim >= 4) {
      if (th) {
        const f4u t = *reinterpret_cast<const f4u *>(th + j);
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] += t[q];
      }
      if (out_dtype == SK_BF16) {
        h4u w;
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = f32_to_bf16(o[q]);
        *reinterpret_cast<h4u *>((uint16_t *)g.out[gl] + pos) = w;
      } else {
        *reinterpret_cast<f4u *>((float *)g.out[gl] + pos) = f4u{o[0], o[1], o[2], o[3]};
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q < lim) store_out(g.out[gl], out_dtype, pos + q, th ? o[q] + th[j + q] : o[q]);
    }
  }
}

// ===========================================================================
// Forward for calls of few vectors (affd_F_grouped): the same passes backwards.
//   rows h: signs, pi1_l, H_l                                   -> W[t][p][l]
//   columns l: sum over t of M[t'] . H_p W[t] (dk1 < 1024: g . H_p W), H_p,
//     rows pi2_p(a)                                             -> G^T[l][a]
//   k_affdT_outm over all layers (sk_affd_t.hip).
// W keeps its rows whole, so one launch per pass takes every layer of the
// call; the slab kernels for larger batches share each M row among 8 vectors
// and W^T among the layers' launches, and for one vector their launches (two
// per layer) never fill the device.
// ===========================================================================
template <bool BF16>
__global__ __launch_bounds__(256) void k_affdF_rows(const LayerDesc *__restrict__ layers,
                                                    const uint16_t *__restrict__ ptab, AffdTTGroup g,
                                                    int64_t b_begin, float *__restrict__ ws, Key key) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  typedef uint16_t h4u __attribute__((ext_vector_type(4), aligned(2)));
  using L = Lds1024<8>;
  __shared__ __align__(16) float s[L::kFloats];
  __shared__ __align__(16) uint32_t sgn[8 * 32];
  int gl = 0;
  while (gl + 1 < g.n && blockIdx.x >= g.blk0[gl + 1]) ++gl;
  const LayerDesc &ld = layers[g.layer[gl]];
  const int64_t h0 = (int64_t)(blockIdx.x - g.blk0[gl]) * 8, v = blockIdx.y;
  const int col = 4 * threadIdx.x;
  const void *x = g.out[gl];
  const int64_t x0 = (b_begin + v) * ld.n;
  float e[8][4];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int64_t j = (h0 + r) * 1024 + col, lim = ld.n - j;
#pragma unroll
    for (int q = 0; q < 4; ++q) e[r][q] = 0.0f;
    if (lim >= 4) {
      if (BF16) {
        const h4u u = *reinterpret_cast<const h4u *>((const uint16_t *)x + x0 + j);
#pragma unroll
        for (int q = 0; q < 4; ++q) e[r][q] = bf16_to_f32(u[q]);
      } else {
        const f4u u = *reinterpret_cast<const f4u *>((const float *)x + x0 + j);
#pragma unroll
        for (int q = 0; q < 4; ++q) e[r][q] = u[q];
      }
    } else if (lim > 0) {
      load4<BF16, false>(x, x0 + j, lim, e[r]);
    }
  }
  if (threadIdx.x < 64) {  // one Philox block per 128 coordinates
    const W4 wd = philox((uint64_t)h0 * 8u + threadIdx.x, (uint32_t)ld.layer_id, ST_SIGN, key);
    *reinterpret_cast<uint4 *>(&sgn[4 * threadIdx.x]) = make_uint4(wd.w[0], wd.w[1], wd.w[2], wd.w[3]);
  }
  int idx[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) idx[q] = ptab[ld.poff[0][0][ld.K - 1] + col + q];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t bits = sgn[r * 32 + (col >> 5)] >> (col & 31);
#pragma unroll
    for (int q = 0; q < 4; ++q) s[L::idx(r, idx[q])] = flip(e[r][q], (bits >> q) & 1u);
  }
  __syncthreads();
  fwht1024_lds<8>(s);
  const int64_t per_v = ((ld.rows_live + ld.dk1 - 1) >> ld.lgdk1) << (ld.lgdk1 + 10);
  float *w = ws + g.w_off[gl] + v * per_v;
  for (int r = 0; r < 8 && h0 + r < ld.rows_live; ++r) {
    const int64_t h = h0 + r;
    const int64_t p = ptab[ld.poff[0][0][ld.K - 2] + (h & (ld.dk1 - 1))];
    float *wr = w + ((h >> ld.lgdk1) << (ld.lgdk1 + 10)) + p * 1024;
#pragma unroll
    for (int k = 0; k < 4; ++k) wr[threadIdx.x + 256 * k] = s[L::idx(r, threadIdx.x + 256 * k)];
  }
}

// Columns of a dk1 = 1024 layer, thread layout of k_affdTT_cols: F stays in
// registers (p = 32 rc + m) over the run's slabs; the next slab's rows of W load
// while M is turned through LDS, and M while W goes through H_p.
__global__ __launch_bounds__(1024) void k_affdF_cols(const LayerDesc *__restrict__ layers,
                                                     const uint16_t *__restrict__ ptab, AffdTTGroup g, int R,
                                                     float *__restrict__ ws) {
  using L = Lds1024R32;
  __shared__ float s[L::kFloats];
  int gl = 0;
  while (gl + 1 < g.n && blockIdx.x >= g.blk0[gl + 1]) ++gl;
  const LayerDesc &ld = layers[g.layer[gl]];
  const int c0 = (int)(blockIdx.x - g.blk0[gl]) * 32;
  const int nlive = (int)((ld.rows_live + 1023) >> 10);
  const int t0 = g.t0[gl], t1 = min(t0 + g.spw, nlive);
  const int64_t v = blockIdx.y;
  const int tid = threadIdx.x, ri = tid & 31, rc = tid >> 5;
  const uint16_t *inv2 = ptab + ld.poff[1][1][ld.K - 2];
  const uint16_t *inv1 = ptab + ld.poff[0][1][ld.K - 2];
  float *high = s + ri * L::kStride + rc;      // p = rc + 32 k at 33 k
  float *low = s + ri * L::kStride + 33 * rc;  // p = 32 rc + m at m
  float f[32], x[32], mreg[32];
  auto fetch_w = [&](int t) {
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(ws + g.w_off[gl] + ((v * nlive + t) << 20), 1u << 22);
    const int voff = rc * 4096 + (c0 + ri) * 4;
    const int64_t live = ld.rows_live - (int64_t)t * 1024;
    if (live >= 1024) {
#pragma unroll
      for (int k = 0; k < 32; ++k)
        x[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wr, voff, k * 32 * 4096, 0));
    } else {  // rows behind no source row were never written: read past the end (zero)
      int r0 = rc;
      asm volatile("" : "+v"(r0));  // keeps the 32 look-ups out of the slab loop's registers
#pragma unroll
      for (int k = 0; k < 32; ++k)
        x[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
            wr, inv1[r0 + 32 * k] < live ? voff + k * 32 * 4096 : 1 << 22, 0, 0));
    }
  };
  auto fetch_m = [&](int t) {
    int64_t ts = 0, stride = 1;  // pi1 of the top digits of t
    for (int k = ld.K - 3; k >= 0; --k) {
      const int64_t dig = (t / stride) & ((1ll << ld.lg[k]) - 1);
      ts += (int64_t)ptab[ld.poff[0][0][k] + dig] * stride;
      stride <<= ld.lg[k];
    }
    const __amdgpu_buffer_rsrc_t mr = buf_rsrc(g.m[gl] + (ts << 20) + (int64_t)c0 * 1024, 32 * 4096);
#pragma unroll
    for (int k = 0; k < 32; ++k) mreg[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(mr, tid * 4, k * 4096, 0));
  };
#pragma unroll
  for (int m = 0; m < 32; ++m) f[m] = 0.0f;
  fetch_w(t0);
  for (int t = t0; t < t1; ++t) {
    fetch_m(t);
    fwht_regs_t<32>(x);
    __syncthreads();  // the block's last readers are done
#pragma unroll
    for (int k = 0; k < 32; ++k) high[33 * k] = x[k];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 32; ++m) x[m] = low[m];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 32; ++k) s[k * L::kStride + tid + (tid >> 5)] = mreg[k];
    fwht_regs_t<32>(x);
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 32; ++m) f[m] += low[m] * x[m];
    if (t + 1 < t1) fetch_w(t + 1);
  }
  fwht_regs_t<32>(f);
#pragma unroll
  for (int m = 0; m < 32; ++m) low[m] = f[m] * kMidScale;  // the places this thread has just read
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 32; ++k) f[k] = high[33 * k];
  fwht_regs_t<32>(f);
  // rows a >= R: past the resource, dropped
  const __amdgpu_buffer_rsrc_t gr = buf_rsrc(ws + g.u_off[gl] + v * 1024 * R, (uint32_t)R << 12);
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const int a = inv2[rc + 32 * k];
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f[k]), gr, a < R ? ((c0 + ri) * R + a) * 4 : R << 12, 0, 0);
  }
}

template <int LGT>
__global__ __launch_bounds__(256) void k_affdF_cols_s(const LayerDesc *__restrict__ layers,
                                                      const uint16_t *__restrict__ ptab, AffdTTGroup g, int R,
                                                      int64_t bc, float *__restrict__ ws, Key key) {
  constexpr int NG = 1 << (LGT - 10);
  __shared__ __align__(16) float s[p16_floats(1 << LGT)];
  int gl = 0;
  while (gl + 1 < g.n && blockIdx.x >= g.blk0[gl + 1]) ++gl;
  const LayerDesc &ld = layers[g.layer[gl]];
  const int lgcs = min(10, LGT - ld.lgdk1);
  const int c0 = (int)(blockIdx.x - g.blk0[gl]) << lgcs;
  const int cmask = (1 << lgcs) - 1, tot = ld.dk1 << lgcs;
  const uint16_t *p2 = ptab + ld.poff[1][0][ld.K - 2];
  const uint16_t *inv1 = ptab + ld.poff[0][1][ld.K - 2];
  const int lgR = 31 - __clz(R);
  float gg[NG][4];
  affd_tile_gauss<NG>(ld, lgcs, c0, tot, key, gg);
  for (int64_t v = blockIdx.y; v < bc; v += gridDim.y) {
    const float *w = ws + g.w_off[gl] + v * ld.np + c0;
    for (int e = threadIdx.x; e < tot; e += 256) {
      const int p = e >> lgcs;
      s[p16(e)] = inv1[p] < ld.rows_live ? w[(int64_t)p * 1024 + (e & cmask)] : 0.0f;
    }
    affd_tile_HgH<NG>(s, ld.lgdk1 + lgcs, lgcs, tot, gg);
    float *go = ws + g.u_off[gl] + (v * 1024 + c0) * R;
    for (int e = threadIdx.x; e < R << lgcs; e += 256) {  // a fastest: a column's R values are contiguous
      const int c = e >> lgR, a = e & (R - 1);
      go[e] = s[p16((p2[a] << lgcs) + c)];
    }
    __syncthreads();  // the tile is free for the next vector
  }
}

// Layers of the transposed-slab path need the stored M; one-slab layers of
// 2 <= dk1 < 1024 regenerate g.
bool affd_T_grouped(const sk_sketch *s, int layer) {
  const LayerDesc &ld = s->layers[layer];
  if (affd_transposed_path(s, layer)) return s->d_mtab && s->mtab_off[layer] >= 0;
  return s->D > 1024 && ld.K == 2 && ld.L == 1024 && ld.dk1 >= 2 && ld.dk1 < 1024;
}

// Live slabs of a layer.
static int64_t affd_slabs(const LayerDesc &ld) { return (ld.rows_live + ld.dk1 - 1) / ld.dk1; }

// Forward, layers of one slab of fewer than 1024 rows (five launches each on the other paths) gain here at every
// size measured (widths 300 to 420, D = 2^12 to 2^17): 627 -> 117 us for one
// vector, 863 -> 419 for 8, 1343 -> 1175 for 16, 1853 -> 1776 and 2258 -> 2268
// for 32.  Biases (N' = D, at most 8 rows) keep their own kernels from four
// vectors on (D = 2^14, 8 vectors: 55 against 70 us).
// Layers of 1024-row slabs, up to three vectors, gain the launches that they
// share (some 40 us each), and lose that every vector reads M for itself (there
// 8 vectors share a row) and writes a sum of D values per four slabs: by the
// slopes of 1 to 9 layers some 3 us for each slab of every further vector (0.5 of
// the first), 11.5 for each such sum at D = 2^20; the rule is in halves of a us,
// its bounds where calls of GPT-2-like blocks and of equal matrices break even.  9 matrices, other path / here: D = 2^17, of 4
// slabs, one / two / three vectors 489 / 279, 539 / 502, 590 / 597; of 7, 537 /
// 370, 614 / 596, 689 / 802; of 16, three, 1298 / 1779; D = 2^20, of 4, one / two
// 509 / 374, 509 / 599; of 16, one, 927 / 1075.  With many layers the sums of the other path take
// several passes (48 matrices of one slab, D = 2^20, three vectors: 2198 / 2035,
// 9 of them 404 / 436).  A lone layer shares nothing, and of several slabs it has
// 32 workgroups per four of them (4096 x 1024, D = 2^17, one vector: 69 / 80; 1024
// x 1024, D = 2^17, 53 / 43, D = 2^20 61 / 66).
static bool affd_F_grouped(const sk_sketch *s, int layer, int64_t bc, int n) {
  if (!affd_T_grouped(s, layer)) return false;
  if (!affd_transposed_path(s, layer)) return bc <= 3 || (bc <= 32 && !affd_small_path(s, layer));
  const LayerDesc &ld = s->layers[layer];
  const int64_t slabs = (ld.rows_live + ld.dk1 - 1) / ld.dk1, sums = (slabs + 3) / 4;
  if (n == 1) return slabs == 1 && bc <= 3 && bc * s->D < 1 << 20;
  return bc <= 3 && slabs * (6 * bc - 5) + 23 * bc * sums * s->D / (1 << 20) < (bc == 1 ? 90 : n >= 16 ? 84 : 74);
}

std::vector<int> affd_F_layers(const sk_sketch *s, int l0, int l1, int64_t bc) {
  int n = 0;
  for (int l = l0; l < l1; ++l) n += affd_T_grouped(s, l);
  std::vector<int> fl;
  for (int l = l0; l < l1; ++l)
    if (affd_F_grouped(s, l, bc, n)) fl.push_back(l);
  return fl;
}

AffdTTGroup affd_T_group(const sk_sketch *s, int l0, int l1, int64_t bc, void *const *out, const void *const *theta0) {
  AffdTTGroup g{};
  int64_t off = 0;
  while (l0 + g.n < l1 && g.n < kMaxPtrs && affd_T_grouped(s, l0 + g.n)) {
    const LayerDesc &ld = s->layers[l0 + g.n];
    const int64_t w = ((ld.rows_live + ld.dk1 - 1) / ld.dk1) * ld.dk1 * 1024;  // slabs behind real outputs
    if (g.n && (off + bc * (s->D + w)) * 4 > s->ws_bytes) break;
    g.layer[g.n] = l0 + g.n;
    g.u_off[g.n] = off;
    g.w_off[g.n] = off + bc * s->D;
    off += bc * (s->D + w);
    g.m[g.n] = affd_transposed_path(s, l0 + g.n) ? s->d_mtab + s->mtab_off[l0 + g.n] : nullptr;
    g.out[g.n] = out[g.n];
    g.th[g.n] = theta0 ? (const float *)theta0[g.n] : nullptr;
    g.scale[g.n] = (float)(1.0 / std::sqrt((double)ld.np * (double)s->D)) / kMidScale;
    ++g.n;
  }
  return g;
}

namespace {
// Workgroups per tile of the one-slab column kernels: 2048 in all (eight per CU), at least one vector each.
unsigned vector_shares(int64_t tiles, int64_t bc) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(bc, 2048 / std::max<int64_t>(1, tiles)));
}

// The layers of g of one class with their first workgroups (count(ld) each).
template <class In, class Count>
AffdTTGroup sub_group(const sk_sketch *s, const AffdTTGroup &g, In in, Count count, int64_t &blocks) {
  AffdTTGroup r{};
  blocks = 0;
  for (int i = 0; i < g.n; ++i) {
    const LayerDesc &ld = s->layers[g.layer[i]];
    if (!in(ld, g.m[i])) continue;
    r.layer[r.n] = g.layer[i];
    r.u_off[r.n] = g.u_off[i];
    r.w_off[r.n] = g.w_off[i];
    r.m[r.n] = g.m[i];
    r.out[r.n] = g.out[i];
    r.th[r.n] = g.th[i];
    r.scale[r.n] = g.scale[i];
    r.t0[r.n] = g.t0[i];
    r.blk0[r.n++] = (uint32_t)blocks;
    blocks += count(ld);
  }
  return r;
}
}  // namespace

void run_affd_T(const sk_sketch *s, const AffdTTGroup &g, const float *z, int64_t b_begin, int64_t bc, int out_dtype,
                int phases, hipStream_t st) {
  const int R = (int)(s->D / 1024);
  float *ws = s->ws;
  int64_t blocks;
  if (phases & 1) {
    hipLaunchKernelGGL(k_affdTT_zrows, dim3((unsigned)((R + 7) / 8), (unsigned)bc, (unsigned)g.n), dim3(256), 0, st,
                       s->d_layers, s->d_ptab, g, z, R, s->D, b_begin, ws);
    // runs of one slab while the device is not full of 128 KB tiles, else four per u
    int64_t tiles = 0;
    for (int i = 0; i < g.n; ++i)
      if (g.m[i]) tiles += 32 * bc * ((s->layers[g.layer[i]].rows_live + 1023) >> 10);
    const int spw = tiles <= 1024 ? 1 : 4;
    AffdTTGroup b = sub_group(
        s, g, [](const LayerDesc &, const float *m) { return m != nullptr; },
        [&](const LayerDesc &ld) { return 32 * ((((ld.rows_live + 1023) >> 10) + spw - 1) / spw); }, blocks);
    b.spw = spw;
    if (b.n)
      hipLaunchKernelGGL(k_affdTT_cols, dim3((unsigned)blocks, (unsigned)bc), dim3(1024), 0, st, s->d_layers,
                         s->d_ptab, b, s->D, ws);
    // tiles of 4096 values (a bias at D = 2^14: four workgroups) while their rows keep 128 bytes (dk1 <= 128)
    b = sub_group(
        s, g, [](const LayerDesc &ld, const float *m) { return !m && ld.lgdk1 <= 7; },
        [](const LayerDesc &ld) { return 1024 >> std::min(10, 12 - ld.lgdk1); }, blocks);
    if (b.n)
      hipLaunchKernelGGL(k_affdTT_cols_s<12>, dim3((unsigned)blocks, vector_shares(blocks, bc)), dim3(256), 0, st,
                         s->d_layers, s->d_ptab, b, R, s->D, bc, ws, s->key);
    b = sub_group(
        s, g, [](const LayerDesc &ld, const float *m) { return !m && ld.lgdk1 > 7; },
        [](const LayerDesc &ld) { return 1024 >> std::min(10, 14 - ld.lgdk1); }, blocks);
    if (b.n)
      hipLaunchKernelGGL(k_affdTT_cols_s<14>, dim3((unsigned)blocks, vector_shares(blocks, bc)), dim3(256), 0, st,
                         s->d_layers, s->d_ptab, b, R, s->D, bc, ws, s->key);
  }
  if (phases & 2) {
    const AffdTTGroup c = sub_group(
        s, g, [](const LayerDesc &, const float *) { return true; },
        [](const LayerDesc &ld) { return (ld.rows_live + 7) / 8; }, blocks);
    hipLaunchKernelGGL(k_affdTT_out, dim3((unsigned)blocks, (unsigned)bc), dim3(256), 0, st, s->d_layers, s->d_ptab, c,
                       s->D, b_begin, ws, out_dtype, s->key);
  }
}

// Forward: entries of the group are (layer, run of spw slabs); each has a G^T
// slot (bc x D) and the layer's first entry its W.
AffdTTGroup affd_F_group(const sk_sketch *s, const int *layers, int count, int l0, int64_t bc, const void *const *x,
                         int *taken) {
  AffdTTGroup g{};
  g.spw = 4;
  int64_t w_all = 0, w_at[kMaxPtrs];
  int n = 0;
  for (; n < count; ++n) {
    const int l = layers[n];
    const LayerDesc &ld = s->layers[l];
    const bool big = affd_transposed_path(s, l);
    const int64_t slabs = (ld.rows_live + ld.dk1 - 1) / ld.dk1;
    const int runs = big ? (int)((slabs + g.spw - 1) / g.spw) : 1;
    const int64_t w = bc * slabs * ld.dk1 * 1024;
    if (g.n + runs > kMaxPtrs || (bc * s->D * (g.n + runs) + w_all + w) * 4 > s->ws_bytes) break;
    for (int r = 0; r < runs; ++r) {
      g.layer[g.n] = l;
      w_at[g.n] = w_all;
      g.t0[g.n] = r * g.spw;
      g.m[g.n] = big ? s->d_mtab + s->mtab_off[l] : nullptr;
      g.out[g.n] = const_cast<void *>(x[l - l0]);
      g.scale[g.n] = (float)(1.0 / std::sqrt((double)ld.np * (double)s->D)) / kMidScale;
      g.u_off[g.n] = g.n * bc * s->D;
      ++g.n;
    }
    w_all += w;
  }
  for (int i = 0; i < g.n; ++i) g.w_off[i] = bc * s->D * g.n + w_at[i];
  *taken = n;
  return g;
}

void run_affd_F(const sk_sketch *s, const AffdTTGroup &g, int dtype, int64_t b_begin, int64_t bc, int phases,
                hipStream_t st) {
  const int R = (int)(s->D / 1024);
  float *ws = s->ws;
  int64_t blocks;
  if (phases & 1) {
    AffdTTGroup c = g;  // one entry per layer
    c.n = 0;
    blocks = 0;
    for (int i = 0; i < g.n; ++i) {
      if (g.t0[i]) continue;
      c.layer[c.n] = g.layer[i];
      c.w_off[c.n] = g.w_off[i];
      c.out[c.n] = g.out[i];
      c.blk0[c.n++] = (uint32_t)blocks;
      blocks += (s->layers[g.layer[i]].rows_live + 7) / 8;
    }
    if (dtype == SK_BF16)
      hipLaunchKernelGGL(k_affdF_rows<true>, dim3((unsigned)blocks, (unsigned)bc), dim3(256), 0, st, s->d_layers,
                         s->d_ptab, c, b_begin, ws, s->key);
    else
      hipLaunchKernelGGL(k_affdF_rows<false>, dim3((unsigned)blocks, (unsigned)bc), dim3(256), 0, st, s->d_layers,
                         s->d_ptab, c, b_begin, ws, s->key);
  }
  if (phases & 2) {
    AffdTTGroup b = sub_group(
        s, g, [](const LayerDesc &, const float *m) { return m != nullptr; }, [](const LayerDesc &) { return 32; },
        blocks);
    b.spw = g.spw;
    if (b.n)
      hipLaunchKernelGGL(k_affdF_cols, dim3((unsigned)blocks, (unsigned)bc), dim3(1024), 0, st, s->d_layers, s->d_ptab,
                         b, R, ws);
    b = sub_group(
        s, g, [](const LayerDesc &ld, const float *m) { return !m && ld.lgdk1 <= 7; },
        [](const LayerDesc &ld) { return 1024 >> std::min(10, 12 - ld.lgdk1); }, blocks);
    if (b.n)
      hipLaunchKernelGGL(k_affdF_cols_s<12>, dim3((unsigned)blocks, vector_shares(blocks, bc)), dim3(256), 0, st,
                         s->d_layers, s->d_ptab, b, R, bc, ws, s->key);
    b = sub_group(
        s, g, [](const LayerDesc &ld, const float *m) { return !m && ld.lgdk1 > 7; },
        [](const LayerDesc &ld) { return 1024 >> std::min(10, 14 - ld.lgdk1); }, blocks);
    if (b.n)
      hipLaunchKernelGGL(k_affdF_cols_s<14>, dim3((unsigned)blocks, vector_shares(blocks, bc)), dim3(256), 0, st,
                         s->d_layers, s->d_ptab, b, R, bc, ws, s->key);
  }
}

}  // namespace sk
