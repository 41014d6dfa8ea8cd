// sk_qk.hip -- QK (Kronecker) sketch kernels: per weight matrix X (m x n),
// Y = A X B^T with A (dA x m) ~ N(0, 1/dA) and B (dB x n) ~ N(0, 1/dB)
// (eq. straight with two Kronecker factors; the contraction is that of
// eq. qk_proof_tensor_dec).  Factors are generated on the device at creation
// in fp32.  A and B are kept in fp32 and, for the bf16 matrix-core
// contractions of bf16 inputs, also as two bf16 terms, hi = bf16(F) and
// lo = bf16(F - hi) (both rounded to nearest even), so that X B^T =
// X hi^T + X lo^T sees B to 16 mantissa bits.  Products accumulate in fp32.
// fp32 inputs, shapes off the tiling below and the transpose multiply by the
// fp32 factors with fp64 sums (sk_qk64.hip).
#include <algorithm>

#include "sk_launch.h"

namespace sk {

__device__ __forceinline__ uint16_t qk_f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float qk_bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// A in fp32 and as bf16 hi / lo terms (for the contraction that applies A first)
__global__ void k_qk_factor_a(float *__restrict__ dst, uint16_t *__restrict__ hi, uint16_t *__restrict__ lo,
                              int64_t count, uint32_t layer, float scale, Key key) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float g = gauss((uint64_t)i, layer, ST_QKA, key) * scale;
  dst[i] = g;
  const uint16_t h = qk_f2bf(g);
  hi[i] = h;
  lo[i] = qk_f2bf(g - qk_bf2f(h));
}

// B in fp32 and as bf16 hi / lo terms
__global__ void k_qk_factor_b(float *__restrict__ dst, uint16_t *__restrict__ hi, uint16_t *__restrict__ lo,
                              int64_t count, uint32_t layer, float scale, Key key) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float g = gauss((uint64_t)i, layer, ST_QKB, key) * scale;
  dst[i] = g;
  const uint16_t h = qk_f2bf(g);
  hi[i] = h;
  lo[i] = qk_f2bf(g - qk_bf2f(h));
}

void launch_qk_factors(const sk_sketch *s, hipStream_t st) {
  for (const LayerDesc &ld : s->layers) {
    const int64_t na = (int64_t)ld.da * ld.m, nb = (int64_t)ld.db * ld.nc;
    hipLaunchKernelGGL(k_qk_factor_a, dim3((unsigned)((na + 255) / 256)), dim3(256), 0, st, s->d_qka + ld.fa_off,
                       s->d_qkah + ld.fa_off, s->d_qkah + s->qk_a_elems + ld.fa_off, na, (uint32_t)ld.layer_id,
                       (float)(1.0 / sqrt((double)ld.da)), s->key);
    hipLaunchKernelGGL(k_qk_factor_b, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, st, s->d_qkbf + ld.fb_off,
                       s->d_qkb + ld.fb_off, s->d_qkb + s->qk_b_elems + ld.fb_off, nb, (uint32_t)ld.layer_id,
                       (float)(1.0 / sqrt((double)ld.db)), s->key);
  }
  (void)hipGetLastError();
}

// ---------------------------------------------------------------------------
// MFMA path (bf16 X, n % 128 == 0, dA and dB multiples of 16, dB <= 128).
// Stage 1: T^T[v][c][i] = sum_j X[v][i][j] B[c][j], a tall-skinny GEMM over
// the stacked rows of the batch (M = bc m, N = dB, K = n) on
// v_mfma_f32_16x16x32_bf16.  Each wave owns 16 rows; each lane streams 64
// contiguous bytes of its row per 128-wide K step and splits them over four
// MFMAs.  The pairing of K positions to MFMA slots is a fixed permutation of
// the contraction index applied identically to X and B, so it does not change
// the sum.  Stage 2: Y[v][a][c] = sum_i A[a][i] T^T[v][c][i] on
// v_mfma_f32_16x16x4f32 (fp32 T, bf16 A widened exactly).
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

union Pack8 {
  uint4 u;
  bf16x8 v;
};

// Layers of a launch are tasks in the kernel arguments: one layer's contraction
// leaves the chip idle up to some 30 vectors (48 workgroups for a 768 x 768
// matrix and 16 vectors, and 45 us a layer whatever the batch).  12 GPT-2
// blocks (72 matrices), one launch per layer and contraction against groups:
// 3355 -> 594 us for 8 vectors, 3620 -> 1849 for 32; a 2048-wide decoder block,
// 64 vectors: 1628 -> 1452.  Dividing the first contraction's index instead
// writes more partial products than it reads inputs (3741 for the 32).
template <class Args>
__device__ __forceinline__ const auto &qk_task(const Args &a) {
  int i = 0;
  while (i + 1 < a.n && a.base + blockIdx.x >= a.t[i + 1].blk0) ++i;
  return a.t[i];
}

constexpr int kQkMR = 4;                  // 16-row tiles per wave
constexpr int kQkRows = 4 * kQkMR * 16;   // stacked rows per workgroup (4 waves)
constexpr int kQkBRow = 128 * 2 + 16;     // bytes of one B row chunk in LDS (padded)

template <int NT>
__global__ __launch_bounds__(256) void k_qk_s1(QkFirst a) {
  const QkFirstTask &task = qk_task(a);
  const uint32_t blk = a.base + blockIdx.x - task.blk0;
  const uint16_t *__restrict__ x = task.x, *__restrict__ B = task.fh, *__restrict__ Blo = task.fl;
  float *__restrict__ tt = task.t;
  const int64_t m = task.m, n = task.n, rows = a.bc * m;
  constexpr int DB = NT * 16;
  __shared__ __align__(16) unsigned char bs[2 * DB * kQkBRow];  // [hi|lo][row][128 bf16 + pad]
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const int64_t r0 = (int64_t)blk * kQkRows + wave * (kQkMR * 16);
  const uint16_t *xr[kQkMR];
  bool rv[kQkMR];
#pragma unroll
  for (int mr = 0; mr < kQkMR; ++mr) {
    const int64_t row = r0 + mr * 16 + li;
    rv[mr] = row < rows;
    xr[mr] = x + (rv[mr] ? row : 0) * n + g * 8;
  }
  floatx4 acc[kQkMR][NT];
#pragma unroll
  for (int mr = 0; mr < kQkMR; ++mr)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[mr][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int64_t k0 = 0; k0 < n; k0 += 128) {
    // this wave's X fragments: MFMA cc takes k = k0 + 32 cc + 8 g .. + 7 in lane (li, g), so each load
    // instruction reads 64 contiguous bytes of each of 16 rows (16 cache lines, not 32 half-used ones:
    // the address units bound this loop)
    Pack8 xf[kQkMR][4];
#pragma unroll
    for (int mr = 0; mr < kQkMR; ++mr)
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
        xf[mr][cc].u = rv[mr] ? *(const uint4 *)(xr[mr] + k0 + cc * 32) : make_uint4(0, 0, 0, 0);
    __syncthreads();  // previous chunk of B consumed
    // B[hi|lo][row][k0 .. k0+127] -> LDS, 16 bytes per thread per step
    for (int e = threadIdx.x; e < 2 * DB * 16; e += 256) {
      const int arr = e / (DB * 16), rem = e - arr * (DB * 16);
      const int row = rem >> 4, c16 = rem & 15;
      const uint16_t *src = (arr ? Blo : B) + (int64_t)row * n + k0 + c16 * 8;
      *(uint4 *)(bs + (arr * DB + row) * kQkBRow + c16 * 16) = *(const uint4 *)src;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const unsigned char *bh = bs + (t * 16 + li) * kQkBRow + g * 16;
      const unsigned char *bl = bh + DB * kQkBRow;
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) {
        Pack8 vh, vl;
        vh.u = *(const uint4 *)(bh + cc * 64);
        vl.u = *(const uint4 *)(bl + cc * 64);
#pragma unroll
        for (int mr = 0; mr < kQkMR; ++mr)
          acc[mr][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[mr][cc].v, vh.v, acc[mr][t], 0, 0, 0);
#pragma unroll
        for (int mr = 0; mr < kQkMR; ++mr)
          acc[mr][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[mr][cc].v, vl.v, acc[mr][t], 0, 0, 0);
      }
    }
  }
  // D layout: lane holds rows 4 g .. 4 g + 3 of column li of each 16 x 16 tile
#pragma unroll
  for (int mr = 0; mr < kQkMR; ++mr)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t R = r0 + mr * 16 + g * 4 + i;
      if (R >= rows) continue;
      const int64_t v = R / m, ii = R - (R / m) * m;
#pragma unroll
      for (int t = 0; t < NT; ++t) tt[(v * DB + t * 16 + li) * m + ii] = acc[mr][t][i];
    }
}

// A first (dA < dB, so A X costs fewer products than X B^T): stage 1
// U[v][a][j] = sum_i A[a][i] X[v][i][j] on v_mfma_f32_16x16x32_bf16 with A as
// bf16 hi + lo.  X's contiguous index j is the output column, so each lane
// reads 8 bytes (columns j0 .. j0 + 3) of 8 consecutive rows and packs the
// 16-bit halves into the K fragments of four MFMAs (one per column), i.e. four
// 16-column sets interleaved with stride 4.  Each step takes 64 rows; the
// next step's rows load during the current MFMAs.  Stage 2 is k_qk_s2 with U
// per vector and B in fp32.
template <int MT>
__global__ __launch_bounds__(256) void k_qk_s1a(QkFirst a) {
  const QkFirstTask &task = qk_task(a);
  const uint32_t blk = a.base + blockIdx.x - task.blk0;
  const uint16_t *__restrict__ x = task.x, *__restrict__ Ah = task.fh, *__restrict__ Al = task.fl;
  float *__restrict__ u = task.t;
  const int64_t m = task.m, n = task.n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const uint32_t ncol = (uint32_t)(n / 256);
  const int64_t v = blk / ncol;
  const int64_t j0 = (int64_t)(blk % ncol) * 256 + wave * 64 + 4 * li;  // this lane's four columns
  const uint16_t *xc = x + v * m * n + j0 + (int64_t)(g * 8) * n;
  const uint16_t *ah = Ah + (int64_t)li * m + g * 8;
  const uint16_t *al = Al + (int64_t)li * m + g * 8;
  floatx4 acc[MT][4];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[t][q] = floatx4{0.f, 0.f, 0.f, 0.f};
  uint2 w[2][8];  // rows k0 + 32 h + 8 g + r
  auto fetch = [&](int64_t k0) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 8; ++r) w[h][r] = *(const uint2 *)(xc + (k0 + 32 * h + r) * n);
  };
  fetch(0);
  for (int64_t k0 = 0; k0 < m; k0 += 64) {
    uint2 c[2][8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 8; ++r) c[h][r] = w[h][r];
    if (k0 + 64 < m) fetch(k0 + 64);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // K fragments (rows k0 + 32 h + 8 g .. + 7) of columns j0 + q
      Pack8 f[4];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        uint32_t e[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) e[r] = p ? c[h][r].y : c[h][r].x;
        f[2 * p].u = make_uint4(__builtin_amdgcn_perm(e[1], e[0], 0x05040100u),
                                __builtin_amdgcn_perm(e[3], e[2], 0x05040100u),
                                __builtin_amdgcn_perm(e[5], e[4], 0x05040100u),
                                __builtin_amdgcn_perm(e[7], e[6], 0x05040100u));
        f[2 * p + 1].u = make_uint4(__builtin_amdgcn_perm(e[1], e[0], 0x07060302u),
                                    __builtin_amdgcn_perm(e[3], e[2], 0x07060302u),
                                    __builtin_amdgcn_perm(e[5], e[4], 0x07060302u),
                                    __builtin_amdgcn_perm(e[7], e[6], 0x07060302u));
      }
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        Pack8 hv, lv;
        hv.u = *(const uint4 *)(ah + (int64_t)(t * 16) * m + k0 + 32 * h);
        lv.u = *(const uint4 *)(al + (int64_t)(t * 16) * m + k0 + 32 * h);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hv.v, f[q].v, acc[t][q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lv.v, f[q].v, acc[t][q], 0, 0, 0);
      }
    }
  }
  // D layout: lane holds rows 4 g .. 4 g + 3 (a) of its column in each set
  float *ub = u + v * (int64_t)(MT * 16) * n + j0;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = t * 16 + g * 4 + i;
      *(float4 *)(ub + row * n) = make_float4(acc[t][0][i], acc[t][1][i], acc[t][2][i], acc[t][3][i]);
    }
}

// The same stage with 16-byte loads: each lane reads eight columns j0 .. j0 + 7
// (two 128-byte lines per row for 16 lanes, half the load instructions of the
// 8-byte form for the same bytes), which gives eight 16-column sets per MFMA
// group; steps of 32 rows, the next step's rows loading during the MFMAs.
template <int MT>
__global__ __launch_bounds__(256) void k_qk_s1aw(QkFirst a) {
  const QkFirstTask &task = qk_task(a);
  const uint32_t blk = a.base + blockIdx.x - task.blk0;
  const uint16_t *__restrict__ x = task.x, *__restrict__ Ah = task.fh, *__restrict__ Al = task.fl;
  float *__restrict__ u = task.t;
  const int64_t m = task.m, n = task.n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const uint32_t ncol = (uint32_t)(n / 512);
  const int64_t v = blk / ncol;
  const int64_t j0 = (int64_t)(blk % ncol) * 512 + wave * 128 + 8 * li;  // this lane's eight columns
  const uint16_t *xc = x + v * m * n + j0 + (int64_t)(g * 8) * n;
  const uint16_t *ah = Ah + (int64_t)li * m + g * 8;
  const uint16_t *al = Al + (int64_t)li * m + g * 8;
  floatx4 acc[MT][8];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[t][q] = floatx4{0.f, 0.f, 0.f, 0.f};
  uint4 w[8];  // rows k0 + 8 g + r, columns j0 .. j0 + 7
  auto fetch = [&](int64_t k0) {
#pragma unroll
    for (int r = 0; r < 8; ++r) w[r] = *(const uint4 *)(xc + (k0 + r) * n);
  };
  fetch(0);
  for (int64_t k0 = 0; k0 < m; k0 += 32) {
    // K fragments (rows k0 + 8 g .. + 7) of columns j0 + q, q < 8
    Pack8 f[8];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t e[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) e[r] = p == 0 ? w[r].x : p == 1 ? w[r].y : p == 2 ? w[r].z : w[r].w;
      f[2 * p].u = make_uint4(__builtin_amdgcn_perm(e[1], e[0], 0x05040100u),
                              __builtin_amdgcn_perm(e[3], e[2], 0x05040100u),
                              __builtin_amdgcn_perm(e[5], e[4], 0x05040100u),
                              __builtin_amdgcn_perm(e[7], e[6], 0x05040100u));
      f[2 * p + 1].u = make_uint4(__builtin_amdgcn_perm(e[1], e[0], 0x07060302u),
                                  __builtin_amdgcn_perm(e[3], e[2], 0x07060302u),
                                  __builtin_amdgcn_perm(e[5], e[4], 0x07060302u),
                                  __builtin_amdgcn_perm(e[7], e[6], 0x07060302u));
    }
    if (k0 + 32 < m) fetch(k0 + 32);  // w is free once packed
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      Pack8 hv, lv;
      hv.u = *(const uint4 *)(ah + (int64_t)(t * 16) * m + k0);
      lv.u = *(const uint4 *)(al + (int64_t)(t * 16) * m + k0);
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hv.v, f[q].v, acc[t][q], 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lv.v, f[q].v, acc[t][q], 0, 0, 0);
    }
  }
  // D layout: lane holds rows 4 g .. 4 g + 3 (a) of its column in each set
  float *ub = u + v * (int64_t)(MT * 16) * n + j0;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = t * 16 + g * 4 + i;
      *(float4 *)(ub + row * n) = make_float4(acc[t][0][i], acc[t][1][i], acc[t][2][i], acc[t][3][i]);
      *(float4 *)(ub + row * n + 4) = make_float4(acc[t][4][i], acc[t][5][i], acc[t][6][i], acc[t][7][i]);
    }
}

// A first when it makes fewer products, and also when the 16-byte-load
// A-first kernel applies at most twice the products of the B-first order
// (the matrix cores are far from busy there; its whole-line X loads are not).
bool qk_afirst_ok(const LayerDesc &ld, int dtype) {
  if (dtype != SK_BF16 || ld.da % 16 != 0 || ld.db % 16 != 0 || ld.m % 64 != 0 || ld.nc % 256 != 0) return false;
  return (ld.da < ld.db && ld.da <= 64) || (ld.da <= 32 && ld.da <= 2 * ld.db && ld.nc % 512 == 0);
}

// Stage 2: Y[v][a][c] = sum_k P[a][k] Q[c][k] (P: dA rows, Q: dB rows, both
// with the contraction index contiguous; each may be per vector) on
// v_mfma_f32_16x16x4f32.  One workgroup per (vector, block of TA x TB output
// tiles of 16 x 16): each wave keeps the TA x TB accumulators of the block over
// a quarter of K, so every P and Q row is read once per workgroup, and the four
// partial blocks are added in a fixed order through LDS.  While the
// blocks of a launch are few, K is divided into nk ranges (kper terms, a
// multiple of 64) whose sums go to part[z][v][a db + c], added in order by
// k_qk_s2_sum: 128 workgroups with 8192 terms each (fc2 of a 2048-wide decoder,
// 64 vectors) took 110 us for 67 MB.
template <int TA, int TB>
__global__ __launch_bounds__(256) void k_qk_s2(QkSecond a) {
  __shared__ float red[4][TA * TB][64][4];
  const QkSecondTask &task = qk_task(a);
  const float *__restrict__ P = task.p, *__restrict__ Q = task.q;
  const int64_t p_vs = task.p_vs, q_vs = task.q_vs, K = task.K, kper = task.kper;
  const int da = task.da, db = task.db;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nbb = db / (16 * TB), nb = da / (16 * TA) * nbb;
  uint32_t e0 = a.base + blockIdx.x - task.blk0;
  const int blk = (int)(e0 % (uint32_t)nb);
  e0 /= (uint32_t)nb;
  const int64_t v = e0 % (uint32_t)a.bc, z = e0 / (uint32_t)a.bc;
  const int ba = blk / nbb, bb = blk - (blk / nbb) * nbb;
  const int li = lane & 15, g = lane >> 4;
  const float *pr = P + v * p_vs + (int64_t)(ba * TA * 16 + li) * K + g * 4;
  const float *qr = Q + v * q_vs + (int64_t)(bb * TB * 16 + li) * K + g * 4;
  const int64_t z0 = z * kper, z1 = z0 + kper < K ? z0 + kper : K;
  const int64_t per = ((z1 - z0 + 63) / 64) * 16;  // K range per wave, a multiple of 16
  const int64_t kb = z0 + wave * per, ke = kb + per < z1 ? kb + per : z1;
  floatx4 acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // U steps of 16 per iteration: all of an iteration's loads are in flight together
  constexpr int U = TA * TB >= 8 ? 2 : 4;
  int64_t k0 = kb;
  for (; k0 + 16 * U <= ke; k0 += 16 * U) {
    float4 pv[U][TA], qv[U][TB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < TA; ++i) pv[u][i] = *(const float4 *)(pr + (int64_t)(i * 16) * K + k0 + 16 * u);
#pragma unroll
      for (int j = 0; j < TB; ++j) qv[u][j] = *(const float4 *)(qr + (int64_t)(j * 16) * K + k0 + 16 * u);
    }
    // consecutive MFMAs go to different accumulators so none waits on the last
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[u][i].x, qv[u][j].x, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[u][i].y, qv[u][j].y, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[u][i].z, qv[u][j].z, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[u][i].w, qv[u][j].w, acc[i][j], 0, 0, 0);
    }
  }
  for (; k0 + 16 <= ke; k0 += 16) {
    float4 pv[TA], qv[TB];
#pragma unroll
    for (int i = 0; i < TA; ++i) pv[i] = *(const float4 *)(pr + (int64_t)(i * 16) * K + k0);
#pragma unroll
    for (int j = 0; j < TB; ++j) qv[j] = *(const float4 *)(qr + (int64_t)(j * 16) * K + k0);
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[i].x, qv[j].x, acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[i].y, qv[j].y, acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[i].z, qv[j].z, acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[i].w, qv[j].w, acc[i][j], 0, 0, 0);
      }
  }
  if (k0 < ke) {  // ragged end of K (K not a multiple of 16)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = k0 + g * 4 + e < ke;
      float pe[TA], qe[TB];
#pragma unroll
      for (int i = 0; i < TA; ++i) pe[i] = ok ? pr[(int64_t)(i * 16) * K + k0 + e] : 0.0f;
#pragma unroll
      for (int j = 0; j < TB; ++j) qe[j] = ok ? qr[(int64_t)(j * 16) * K + k0 + e] : 0.0f;
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pe[i], qe[j], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) red[wave][i * TB + j][lane][q] = acc[i][j][q];
  __syncthreads();
  // lane (li, g) of tile (i, j): rows 4 g .. 4 g + 3 of column li
  for (int e = threadIdx.x; e < TA * TB * 64; e += 256) {
    const int tile = e >> 6, ln = e & 63;
    const int i = tile / TB, j = tile - (tile / TB) * TB;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float y = ((red[0][tile][ln][q] + red[1][tile][ln][q]) + red[2][tile][ln][q]) + red[3][tile][ln][q];
      const int ra = (ba * TA + i) * 16 + (ln >> 4) * 4 + q, c = (bb * TB + j) * 16 + (ln & 15);
      if (task.part) {
        task.part[(z * a.bc + v) * ((int64_t)da * db) + (int64_t)ra * db + c] = y;
      } else {
        float *o = a.out + v * a.D + task.col + (int64_t)ra * db + c;
        *o = a.accumulate ? *o + y : y;
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_qk_s2_sum(QkSecond a) {
  const QkSecondTask &task = qk_task(a);
  const int64_t cnt = (int64_t)task.da * task.db;
  const int64_t e = (int64_t)(a.base + blockIdx.x - task.blk0) * 256 + threadIdx.x;
  if (e >= cnt * a.bc) return;
  float y = 0.0f;
#pragma unroll 8
  for (int z = 0; z < task.nk; ++z) y += task.part[(int64_t)z * a.bc * cnt + e];
  const int64_t v = e / cnt;
  float *o = a.out + v * a.D + task.col + (e - v * cnt);
  *o = a.accumulate ? *o + y : y;
}

// Tiles per block along a side of n16 tiles: the largest of 4, 2, 1 dividing it.
static int qk_block_tiles(int n16) { return n16 % 4 == 0 ? 4 : n16 % 2 == 0 ? 2 : 1; }

bool qk_mfma_ok(const LayerDesc &ld, int dtype) {
  return dtype == SK_BF16 && ld.nc % 128 == 0 && ld.m % 16 == 0 && ld.da % 16 == 0 && ld.db % 16 == 0 && ld.db <= 128;
}

// A call of one vector goes through the fp64-sum kernels: their workgroups
// split the contraction over four waves, and the length of one chain is what
// counts (fp64 sums / bf16, one vector: 12 GPT-2 blocks of width 768 250 / 398
// us, a 2048-wide decoder block 125 / 172, 8192 x 8192 (128, 128) 331 / 584).
// Layers that fill the device by themselves would be faster here (32768 x 768
// (64, 16) 49 / 36, 50304 x 2048 (256, 64) 307 / 148, 128256 x 4096 (256, 64)
// 1184 / 401), but with the first factor to 16 bits: errors of 2.5e-6 instead of
// 1e-7.  Two vectors: 400 / 443 (12 blocks), but 181 / 131 (4 of width 1024).
bool qk_bf16_path(const LayerDesc &ld, int dtype, int64_t batch) {
  return batch > 1 && (qk_afirst_ok(ld, dtype) || qk_mfma_ok(ld, dtype));
}

// First products held by a group: half of the memory-side cache, so that the second contraction finds them there.
// A layer that fills the chip alone needs no group: 145 matrices of a 2048-wide decoder, 256 vectors (33 to 268 MB of
// first products per matrix), took 154 to 160 ms in groups of up to 32, 156.5 layer by layer, 152.6 so.
constexpr int64_t kQkGroupBytes = 128ll << 20;

QkGroup qk_group(const sk_sketch *s, const int *layers, int count, int64_t bc, int64_t ws_bytes) {
  QkGroup g{};
  int64_t off = 0;
  while (g.n < count && g.n < kQkTasks) {
    const LayerDesc &ld = s->layers[layers[g.n]];
    const int64_t need = bc * (qk_afirst_ok(ld, SK_BF16) ? (int64_t)ld.da * ld.nc : (int64_t)ld.m * ld.db);
    if (g.n && (off + need) * 4 > std::min(ws_bytes, kQkGroupBytes)) break;
    g.layer[g.n] = layers[g.n];
    g.t_off[g.n] = off;
    off += (need + 3) & ~3ll;
    ++g.n;
  }
  g.spare = off;
  return g;
}

void launch_qk_first(const sk_sketch *s, const QkGroup &g, const void *const *x, int64_t b_begin, int64_t bc, float *ws,
                     hipStream_t st) {
  // one launch per kernel: 0-7 B first with 1-8 tiles of B, 8-11 A first with 1-4 tiles of A, 12-13 its wide form
  for (int cls = 0; cls < 14; ++cls) {
    QkFirst a{};
    a.bc = bc;
    int64_t blk = 0;
    for (int i = 0; i < g.n; ++i) {
      const LayerDesc &ld = s->layers[g.layer[i]];
      const bool af = qk_afirst_ok(ld, SK_BF16), wide = ld.nc % 512 == 0 && ld.da <= 32;
      if (cls != (!af ? ld.db / 16 - 1 : (wide ? 12 : 8) + ld.da / 16 - 1)) continue;
      QkFirstTask &t = a.t[a.n++];
      t.x = (const uint16_t *)x[i] + b_begin * ld.m * ld.nc;
      t.fh = af ? s->d_qkah + ld.fa_off : s->d_qkb + ld.fb_off;
      t.fl = t.fh + (af ? s->qk_a_elems : s->qk_b_elems);
      t.t = ws + g.t_off[i];
      t.m = ld.m;
      t.n = ld.nc;
      t.blk0 = (uint32_t)blk;
      blk += !af ? (bc * ld.m + kQkRows - 1) / kQkRows : bc * (ld.nc / (wide ? 512 : 256));
    }
    grid_parts(blk, [&](uint32_t first, uint32_t count) {
      const dim3 grid(count);
      a.base = first;
      switch (cls) {
        case 0: hipLaunchKernelGGL(k_qk_s1<1>, grid, dim3(256), 0, st, a); break;
        case 1: hipLaunchKernelGGL(k_qk_s1<2>, grid, dim3(256), 0, st, a); break;
        case 2: hipLaunchKernelGGL(k_qk_s1<3>, grid, dim3(256), 0, st, a); break;
        case 3: hipLaunchKernelGGL(k_qk_s1<4>, grid, dim3(256), 0, st, a); break;
        case 4: hipLaunchKernelGGL(k_qk_s1<5>, grid, dim3(256), 0, st, a); break;
        case 5: hipLaunchKernelGGL(k_qk_s1<6>, grid, dim3(256), 0, st, a); break;
        case 6: hipLaunchKernelGGL(k_qk_s1<7>, grid, dim3(256), 0, st, a); break;
        case 7: hipLaunchKernelGGL(k_qk_s1<8>, grid, dim3(256), 0, st, a); break;
        case 8: hipLaunchKernelGGL(k_qk_s1a<1>, grid, dim3(256), 0, st, a); break;
        case 9: hipLaunchKernelGGL(k_qk_s1a<2>, grid, dim3(256), 0, st, a); break;
        case 10: hipLaunchKernelGGL(k_qk_s1a<3>, grid, dim3(256), 0, st, a); break;
        case 11: hipLaunchKernelGGL(k_qk_s1a<4>, grid, dim3(256), 0, st, a); break;
        case 12: hipLaunchKernelGGL(k_qk_s1aw<1>, grid, dim3(256), 0, st, a); break;
        default: hipLaunchKernelGGL(k_qk_s1aw<2>, grid, dim3(256), 0, st, a); break;
      }
    });
  }
}

void launch_qk_second(const sk_sketch *s, const QkGroup &g, int64_t b_begin, int64_t bc, float *ws, float *out,
                      bool accumulate, hipStream_t st) {
  QkSecond sum{};
  sum.bc = bc;
  sum.D = s->D;
  sum.out = out + b_begin * s->D;
  sum.accumulate = accumulate;
  int64_t total = 0, sblk = 0, spare = g.spare;  // output blocks of the group; floats taken
  for (int i = 0; i < g.n; ++i) {
    const LayerDesc &ld = s->layers[g.layer[i]];
    total += bc * (ld.da / (16 * qk_block_tiles(ld.da / 16))) * (ld.db / (16 * qk_block_tiles(ld.db / 16)));
  }
  for (int cls = 0; cls < 9; ++cls) {  // (1, 2, 4) x (1, 2, 4) tiles per block
    const int ta = 1 << cls / 3, tb = 1 << cls % 3;
    QkSecond a = sum;
    a.n = 0;
    int64_t blk = 0;
    for (int i = 0; i < g.n; ++i) {
      const LayerDesc &ld = s->layers[g.layer[i]];
      if (qk_block_tiles(ld.da / 16) != ta || qk_block_tiles(ld.db / 16) != tb) continue;
      const float *im = ws + g.t_off[i];
      QkSecondTask &t = a.t[a.n++];
      t = QkSecondTask{};
      if (qk_afirst_ok(ld, SK_BF16)) {  // Y[v][a][c] = sum_j U[v][a][j] B[c][j]
        t.p = im;
        t.p_vs = (int64_t)ld.da * ld.nc;
        t.q = s->d_qkbf + ld.fb_off;
        t.K = ld.nc;
      } else {  // Y[v][a][c] = sum_i A[a][i] T^T[v][c][i]
        t.p = s->d_qka + ld.fa_off;
        t.q = im;
        t.q_vs = (int64_t)ld.db * ld.m;
        t.K = ld.m;
      }
      t.da = ld.da;
      t.db = ld.db;
      t.col = ld.qk_col;
      // ranges of K: 1024 workgroups in the group (four per CU), 512 terms or more each, as far as the partial
      // sums fit.  Blocks of 4 x 4 tiles (64 KB of LDS) that fill the CUs evenly are left whole: a 32000 x 1024
      // embedding (256, 64), 32 vectors (128 blocks) 1385 us whole and 1168 divided, 64 vectors 2028 and 2189, 96
      // vectors (384 blocks) 3472 and 3134, 128 vectors 4114 and 4173
      const int64_t cnt = (int64_t)ld.da * ld.db;
      int64_t nk = std::min({t.K / 512, 1024 / total, (s->ws_bytes / 4 - spare) / (bc * cnt)});
      if (nk < 2 || (ta * tb == 16 && total >= 256 && (total + 32) % 256 <= 32)) nk = 1;
      t.kper = ((t.K + nk - 1) / nk + 63) / 64 * 64;
      nk = (t.K + t.kper - 1) / t.kper;
      t.nk = (int)nk;
      t.blk0 = (uint32_t)blk;
      blk += (ld.da / (16 * ta)) * (ld.db / (16 * tb)) * bc * nk;
      if (nk > 1) {
        t.part = ws + spare;
        spare += nk * bc * cnt;
        QkSecondTask &u = sum.t[sum.n++];
        u = t;
        u.blk0 = (uint32_t)sblk;
        sblk += (bc * cnt + 255) / 256;
      }
    }
    grid_parts(blk, [&](uint32_t first, uint32_t count) {
      const dim3 grid(count);
      a.base = first;
      switch (cls) {
        case 0: hipLaunchKernelGGL((k_qk_s2<1, 1>), grid, dim3(256), 0, st, a); break;
        case 1: hipLaunchKernelGGL((k_qk_s2<1, 2>), grid, dim3(256), 0, st, a); break;
        case 2: hipLaunchKernelGGL((k_qk_s2<1, 4>), grid, dim3(256), 0, st, a); break;
        case 3: hipLaunchKernelGGL((k_qk_s2<2, 1>), grid, dim3(256), 0, st, a); break;
        case 4: hipLaunchKernelGGL((k_qk_s2<2, 2>), grid, dim3(256), 0, st, a); break;
        case 5: hipLaunchKernelGGL((k_qk_s2<2, 4>), grid, dim3(256), 0, st, a); break;
        case 6: hipLaunchKernelGGL((k_qk_s2<4, 1>), grid, dim3(256), 0, st, a); break;
        case 7: hipLaunchKernelGGL((k_qk_s2<4, 2>), grid, dim3(256), 0, st, a); break;
        default: hipLaunchKernelGGL((k_qk_s2<4, 4>), grid, dim3(256), 0, st, a); break;
      }
    });
  }
  grid_parts(sblk, [&](uint32_t first, uint32_t count) {
    sum.base = first;
    hipLaunchKernelGGL(k_qk_s2_sum, dim3(count), dim3(256), 0, st, sum);
  });
}

}  // namespace sk
