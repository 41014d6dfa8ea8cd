// sk_qk64.hip -- QK contractions with fp64 sums on v_mfma_f64_16x16x4_f64:
// fp32 inputs, bf16 inputs off the bf16 matrix-core tiling, and every
// transpose.  Operands are the fp32 factors and fp32 / bf16 values widened
// exactly; a sum is rounded once, so the error does not grow with the length
// of the contraction (fp32 accumulation over 50257 terms does not hold 1e-5).
//
// Two contractions cover both directions:
//   dot    out[p][q] = sum_k P[p][k] Q[q][k]   (k contiguous in P and Q)
//          T^T = B X^T (B first), then Y = A T^T or, A first, Y = U B^T;
//   outer  out[i][j] = sum_k P(k,i) Q[k][j]    (j contiguous in Q)
//          U = A X (A first), A^T Z or Z B, and the transposes' output pass.
// fp64 MFMA does 16 x 16 x 4 in 64 cycles (69 TFLOP/s measured on all CUs), so
// an operand fragment loaded straight from L1 / L2 costs less than the
// products it feeds and nothing is staged in LDS: a lane reads four
// consecutive k (or j) as one 16-byte load and feeds four MFMAs (the k order
// inside a step of 16 is permuted alike in both operands).  Contractions over
// an input split k over the four waves of a workgroup, added in a fixed order
// through LDS, so that a 768 x 768 matrix of one vector still gives 24
// workgroups short chains.  Up to kQk64Tasks layers go in one launch: one
// vector's matrix is 2 to 10 us of work, and 146 launches in a row for the 73
// matrices of GPT-2 small cost more than that.  Against one thread per output
// looping over k with fp64 FMAs (uncoalesced rows, no reuse of a row), an
// S^T z plus S x over those 73 matrices went from 54.2 ms to 0.80 ms (0.98 with each
// step's loads waited for before its products).
#include <algorithm>

#include "sk_launch.h"

namespace sk {

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
// rows of any length: 16-byte (fp32) and 8-byte (bf16) pieces at element alignment
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t shortx4u __attribute__((ext_vector_type(4), aligned(2)));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <bool BF16>
struct Elem;
template <>
struct Elem<false> {
  typedef float T;
  typedef floatx4u V;
  static __device__ __forceinline__ double at(const V &v, int i) { return (double)v[i]; }
  static __device__ __forceinline__ float one(const T *p) { return *p; }
};
template <>
struct Elem<true> {
  typedef uint16_t T;
  typedef shortx4u V;
  static __device__ __forceinline__ double at(const V &v, int i) { return (double)bf2f(v[i]); }
  static __device__ __forceinline__ float one(const T *p) { return bf2f(*p); }
};

__device__ __forceinline__ doublex4 mfma(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

}  // namespace

// ---------------------------------------------------------------------------
// dot: a workgroup owns TP x TQ output tiles of 16 x 16 over one k range; the
// waves take a quarter each.  Fragment of a step of 16: lane (li, g) holds
// k = k0 + 4 g .. + 3 of row li; MFMA s takes the s-th of them.  Result of the
// 16 x 16 x 4 fp64 MFMA: lane (li, g) holds rows g + 4 r of column li.
// ---------------------------------------------------------------------------
template <int TP, int TQ, bool QB>
__device__ __forceinline__ void qk64_dot(const Qk64Dot &t, int bp, int bq, int kc, int64_t v, int64_t nv,
                                         int accumulate, double (*red)[8][4][64]) {
  typedef Elem<QB> E;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const float *pr[TP];
  const typename E::T *qr[TQ];
#pragma unroll
  for (int i = 0; i < TP; ++i) {
    const int64_t row = min((int64_t)(bp * TP + i) * 16 + li, (int64_t)t.np - 1);  // past the end: loaded, not stored
    pr[i] = t.p + v * t.pvs + row * t.K + 4 * g;
  }
#pragma unroll
  for (int j = 0; j < TQ; ++j) {
    const int64_t row = min((int64_t)(bq * TQ + j) * 16 + li, (int64_t)t.nq - 1);
    qr[j] = (const typename E::T *)t.q + v * t.qvs + row * t.K + 4 * g;
  }
  const int64_t kb = kc * t.klen, ke = min(t.K, kb + t.klen);
  const int64_t per = ((ke - kb + 63) >> 6) << 4;  // a wave's share, a multiple of 16
  int64_t k = kb + wave * per;
  const int64_t k1 = min(k + per, ke);
  doublex4 acc[TP][TQ];
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TQ; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
  // U steps of 16 per buffer, the next buffer's loads in flight during the products
  constexpr int U = TP == 1 ? 4 : TP == 2 ? 2 : 1;
  floatx4u pv[2][U][TP];
  typename E::V qv[2][U][TQ];
  auto load = [&](int64_t kk, floatx4u(&p)[U][TP], typename E::V(&q)[U][TQ]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int j = 0; j < TQ; ++j) q[u][j] = *(const typename E::V *)(qr[j] + kk + 16 * u);
#pragma unroll
      for (int i = 0; i < TP; ++i) p[u][i] = *(const floatx4u *)(pr[i] + kk + 16 * u);
    }
  };
  auto products = [&](const floatx4u(&p)[U][TP], const typename E::V(&q)[U][TQ]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
          for (int j = 0; j < TQ; ++j) acc[i][j] = mfma((double)p[u][i][s], E::at(q[u][j], s), acc[i][j]);
  };
  if (k + 16 * U <= k1) {
    load(k, pv[0], qv[0]);
    for (;;) {
      k += 16 * U;
      const bool more = k + 16 * U <= k1;  // uniform over the wave
      if (more) load(k, pv[1], qv[1]);
      products(pv[0], qv[0]);
      if (!more) break;
      k += 16 * U;
      const bool more2 = k + 16 * U <= k1;
      if (more2) load(k, pv[0], qv[0]);
      products(pv[1], qv[1]);
      if (!more2) break;
    }
  }
  for (; k < k1; k += 16) {  // the last steps, guarded at the end of the range
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool ok = k + 4 * g + s < k1;
      double pe[TP], qe[TQ];
#pragma unroll
      for (int i = 0; i < TP; ++i) pe[i] = ok ? (double)pr[i][k + s] : 0.0;
#pragma unroll
      for (int j = 0; j < TQ; ++j) qe[j] = ok ? (double)E::one(qr[j] + k + s) : 0.0;
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j) acc[i][j] = mfma(pe[i], qe[j], acc[i][j]);
    }
  }
  // (w0 + w2) + (w1 + w3)
  if (wave >= 2) {
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TQ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave - 2][i * TQ + j][r][lane] = acc[i][j][r];
  }
  __syncthreads();
  if (wave < 2) {
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TQ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[i][j][r] += red[wave][i * TQ + j][r][lane];
          if (wave == 1) red[1][i * TQ + j][r][lane] = acc[i][j][r];
        }
  }
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TQ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t p = (int64_t)(bp * TP + i) * 16 + g + 4 * r, q = (int64_t)(bq * TQ + j) * 16 + li;
        if (p >= t.np || q >= t.nq) continue;
        const double y = acc[i][j][r] + red[1][i * TQ + j][r][lane];
        if (t.part) {
          t.part[((int64_t)kc * nv + v) * ((int64_t)t.np * t.nq) + p * t.nq + q] = y;
        } else {
          float *o = t.o + v * t.ovs + p * t.ldo + q;
          *o = accumulate ? *o + (float)y : (float)y;
        }
      }
}

template <bool QB>
__global__ __launch_bounds__(256, 3) void k_qk64_dot(Qk64DotArgs a) {
  __shared__ double red[2][8][4][64];
  const uint32_t blk = a.base + blockIdx.x;
  int ti = 0;
  while (ti + 1 < a.n && blk >= a.blk0[ti + 1]) ++ti;
  const Qk64Dot &t = a.t[ti];
  uint32_t e = blk - a.blk0[ti];
  const int bp = (int)(e % (uint32_t)t.nbp);
  e /= (uint32_t)t.nbp;
  const int bq = (int)(e % (uint32_t)t.nbq);
  e /= (uint32_t)t.nbq;
  const int kc = (int)(e % (uint32_t)t.nk);
  const int64_t v = e / (uint32_t)t.nk;
  // tiles per workgroup by the operands' heights (uniform over the workgroup)
  if (t.tp == 1)
    qk64_dot<1, 2, QB>(t, bp, bq, kc, v, a.nv, a.accumulate, red);
  else if (t.tp == 2)
    qk64_dot<2, 2, QB>(t, bp, bq, kc, v, a.nv, a.accumulate, red);
  else
    qk64_dot<4, 2, QB>(t, bp, bq, kc, v, a.nv, a.accumulate, red);
}

// Sums the k ranges' partial products in order, in fp64, into out.
__global__ __launch_bounds__(256) void k_qk64_sum(Qk64DotArgs a) {
  const uint32_t blk = a.base + blockIdx.x;
  int ti = 0;
  while (ti + 1 < a.n && blk >= a.blk0[ti + 1]) ++ti;
  const Qk64Dot &t = a.t[ti];
  const int64_t cnt = (int64_t)t.np * t.nq;
  const int64_t e = (int64_t)(blk - a.blk0[ti]) * 256 + threadIdx.x;
  if (e >= cnt * a.nv) return;
  double y = 0.0;
#pragma unroll 8
  for (int k = 0; k < t.nk; ++k) y += t.part[(int64_t)k * a.nv * cnt + e];
  const int64_t v = e / cnt;
  float *o = t.o + v * t.ovs + (e - v * cnt);
  *o = a.accumulate ? *o + (float)y : (float)y;
}

// ---------------------------------------------------------------------------
// outer: a wave owns 16 TM rows x 64 columns; lane (li, g) reads columns
// 4 li .. + 3 of row k0 + 4 g + s (256 contiguous bytes of fp32 per row), one
// 16-column set per component.  KS: the waves split k (long contractions of
// A first); else they take consecutive row tiles (short k, output-bound).
// ---------------------------------------------------------------------------
template <int TM, bool KS, bool PK, bool QB>
__device__ __forceinline__ void qk64_outer(const Qk64Outer &t, int bm, int64_t bn, int64_t v, int out_bf16,
                                           double (*red)[8][4][64]) {
  typedef Elem<QB> E;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const int64_t j0 = bn * 64 + 4 * li;
  const int64_t i0 = (int64_t)(KS ? bm : bm * 4 + wave) * (TM * 16);
  if (!KS && i0 >= t.M) return;
  const bool full = j0 + 3 < t.N;
  const typename E::T *q = (const typename E::T *)t.q + v * t.qvs + (j0 < t.N ? j0 : 0);
  const float *p[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t row = min(i0 + i * 16 + li, (int64_t)t.M - 1);
    p[i] = t.p + v * t.pvs + row * t.psi;
  }
  int64_t k = 0, k1 = t.K;
  if (KS) {
    const int64_t per = ((t.K + 63) >> 6) << 4;
    k = wave * per;
    k1 = min(k + per, t.K);
  }
  doublex4 acc[TM][4];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[i][c] = doublex4{0.0, 0.0, 0.0, 0.0};
  // one step of 16 per buffer, the next step's loads in flight during the products
  typename E::V qv[2][4];
  float pv[2][TM][4];
  auto load = [&](int64_t kk, typename E::V(&qb)[4], float(&pb)[TM][4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const typename E::T *qs = q + (kk + 4 * g + s) * t.N;
      if (full) {
        qb[s] = *(const typename E::V *)qs;
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) qb[s][c] = j0 + c < t.N ? qs[c] : (typename E::T)0;
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (PK) {
        const floatx4u x = *(const floatx4u *)(p[i] + kk + 4 * g);
#pragma unroll
        for (int s = 0; s < 4; ++s) pb[i][s] = x[s];
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) pb[i][s] = p[i][(kk + 4 * g + s) * t.psk];
      }
    }
  };
  auto products = [&](const typename E::V(&qb)[4], const float(&pb)[TM][4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[i][c] = mfma((double)pb[i][s], E::at(qb[s], c), acc[i][c]);
  };
  if (k + 16 <= k1) {
    load(k, qv[0], pv[0]);
    for (;;) {
      k += 16;
      const bool more = k + 16 <= k1;
      if (more) load(k, qv[1], pv[1]);
      products(qv[0], pv[0]);
      if (!more) break;
      k += 16;
      const bool more2 = k + 16 <= k1;
      if (more2) load(k, qv[0], pv[0]);
      products(qv[1], pv[1]);
      if (!more2) break;
    }
  }
  if (k < k1) {  // ragged end of the range
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int64_t kk = k + 4 * g + s;
      const bool ok = kk < k1;
      const typename E::T *qs = q + (ok ? kk : k) * t.N;
      double qe[4], pe[TM];
#pragma unroll
      for (int c = 0; c < 4; ++c) qe[c] = ok && j0 + c < t.N ? (double)E::one(qs + c) : 0.0;
#pragma unroll
      for (int i = 0; i < TM; ++i) pe[i] = ok ? (double)p[i][PK ? kk : kk * t.psk] : 0.0;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[i][c] = mfma(pe[i], qe[c], acc[i][c]);
    }
  }
  if (KS) {  // (w0 + w2) + (w1 + w3)
    if (wave >= 2) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) red[wave - 2][i * 4 + c][r][lane] = acc[i][c][r];
    }
    __syncthreads();
    if (wave < 2) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            acc[i][c][r] += red[wave][i * 4 + c][r][lane];
            if (wave == 1) red[1][i * 4 + c][r][lane] = acc[i][c][r];
          }
    }
    __syncthreads();
    if (wave) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][c][r] += red[1][i * 4 + c][r][lane];
  }
  if (j0 >= t.N) return;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = i0 + i * 16 + g + 4 * r;
      if (row >= t.M) continue;
      const int64_t at = row * t.N + j0;
      double y[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) y[c] = acc[i][c][r];
      if (t.theta) {
        if (full) {
          const floatx4u th = *(const floatx4u *)(t.theta + at);
#pragma unroll
          for (int c = 0; c < 4; ++c) y[c] += (double)th[c];
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (j0 + c < t.N) y[c] += (double)t.theta[at + c];
        }
      }
      if (out_bf16) {
        uint16_t *o = (uint16_t *)t.o + v * t.ovs + at;
        shortx4u w;
#pragma unroll
        for (int c = 0; c < 4; ++c) w[c] = f2bf((float)y[c]);
        if (full) {
          *(shortx4u *)o = w;
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (j0 + c < t.N) o[c] = w[c];
        }
      } else {
        float *o = (float *)t.o + v * t.ovs + at;
        if (full) {
          *(floatx4u *)o = floatx4u{(float)y[0], (float)y[1], (float)y[2], (float)y[3]};
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (j0 + c < t.N) o[c] = (float)y[c];
        }
      }
    }
}

// Thin outputs of transposes (outer_thin): a thread per output and VB vectors,
// the factor's entry read once for them, sums in the order of k as above.
template <int VB>
__global__ __launch_bounds__(256) void k_qk64_thin(Qk64OuterArgs a) {
  const uint32_t blk = a.base + blockIdx.x;
  int ti = 0;
  while (ti + 1 < a.n && blk >= a.blk0[ti + 1]) ++ti;
  const Qk64Outer &t = a.t[ti];
  const uint32_t e = blk - a.blk0[ti], nb = (uint32_t)t.nbn;
  const int64_t at = (int64_t)(e % nb) * 256 + threadIdx.x;
  if (at >= (int64_t)t.M * t.N) return;
  const int64_t i = at / t.N, j = at - i * t.N, v0 = (int64_t)(e / nb) * VB;
  const bool qs = t.qvs == 0;  // the factor is Q
  const float *f = qs ? (const float *)t.q + j : t.p + i * t.psi;
  const int64_t fstep = qs ? t.N : t.psk, step = qs ? t.psk : t.N;
  const float *x[VB];
  double y[VB];
#pragma unroll
  for (int u = 0; u < VB; ++u) {
    const int64_t v = min(v0 + u, a.nv - 1);
    x[u] = qs ? t.p + v * t.pvs + i * t.psi : (const float *)t.q + v * t.qvs + j;
    y[u] = 0.0;
  }
#pragma unroll 8
  for (int k = 0; k < (int)t.K; ++k) {
    const double fv = (double)*f;
    f += fstep;
#pragma unroll
    for (int u = 0; u < VB; ++u) {
      y[u] += (double)*x[u] * fv;
      x[u] += step;
    }
  }
  const double th = t.theta ? (double)t.theta[at] : 0.0;
#pragma unroll
  for (int u = 0; u < VB; ++u) {
    if (v0 + u >= a.nv) break;
    const float o = (float)(y[u] + th);
    if (a.out_bf16)
      ((uint16_t *)t.o)[(v0 + u) * t.ovs + at] = f2bf(o);
    else
      ((float *)t.o)[(v0 + u) * t.ovs + at] = o;
  }
}

template <bool KS, bool QB>
__global__ __launch_bounds__(256, 3) void k_qk64_outer(Qk64OuterArgs a) {
  __shared__ double red[KS ? 2 : 1][8][4][64];
  const uint32_t blk = a.base + blockIdx.x;
  int ti = 0;
  while (ti + 1 < a.n && blk >= a.blk0[ti + 1]) ++ti;
  const Qk64Outer &t = a.t[ti];
  const uint32_t e = blk - a.blk0[ti], nm = (uint32_t)t.nbm, nn = (uint32_t)t.nbn;
  const int64_t v = e / (nm * nn);
  const uint32_t r = e % (nm * nn);
  // KS: the row blocks of one column block (the same input) next to each other
  const int bm = (int)(KS ? r % nm : r / nn);
  const int64_t bn = KS ? r / nm : r % nn;
  if constexpr (KS) {  // A first: k contiguous in A
    if (t.tm == 1)
      qk64_outer<1, true, true, QB>(t, bm, bn, v, a.out_bf16, red);
    else
      qk64_outer<2, true, true, QB>(t, bm, bn, v, a.out_bf16, red);
  } else {
    if (t.psk == 1)
      qk64_outer<1, false, true, QB>(t, bm, bn, v, a.out_bf16, nullptr);
    else if (t.tm == 1)
      qk64_outer<1, false, false, QB>(t, bm, bn, v, a.out_bf16, nullptr);
    else
      qk64_outer<2, false, false, QB>(t, bm, bn, v, a.out_bf16, nullptr);
  }
}

namespace {

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Workgroup numbers of a group stay below 2^32 (a call's chunks have at most 2^20 vectors, and a workgroup writes 64
// bytes or more of a matrix of more than one), but not its threads: a matrix of few columns makes a workgroup of
// every 32 rows, and eight of 2^19 rows with 256 vectors are 2^33 threads.
void launch_dot(Qk64DotArgs &a, bool qb, hipStream_t st) {
  int64_t blk = 0;
  for (int i = 0; i < a.n; ++i) {
    Qk64Dot &t = a.t[i];
    t.tp = t.np <= 16 ? 1 : t.np <= 32 ? 2 : 4;
    t.nbp = (int)cdiv(t.np, 16 * t.tp);
    t.nbq = (int)cdiv(t.nq, 32);
    a.blk0[i] = (uint32_t)blk;
    blk += (int64_t)t.nbp * t.nbq * t.nk * a.nv;
  }
  grid_parts(blk, [&](uint32_t first, uint32_t count) {
    a.base = first;
    if (qb)
      hipLaunchKernelGGL(k_qk64_dot<true>, dim3(count), dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL(k_qk64_dot<false>, dim3(count), dim3(256), 0, st, a);
  });
}

template <bool KS>
void launch_outer(Qk64OuterArgs &a, bool qb, hipStream_t st) {
  int64_t blk = 0;
  for (int i = 0; i < a.n; ++i) {
    Qk64Outer &t = a.t[i];
    t.tm = t.M <= 16 || (!KS && t.psk == 1) ? 1 : 2;
    t.nbm = (int)cdiv(t.M, 16 * t.tm * (KS ? 1 : 4));
    t.nbn = (int)cdiv(t.N, 64);
    a.blk0[i] = (uint32_t)blk;
    blk += (int64_t)t.nbn * t.nbm * a.nv;
  }
  grid_parts(blk, [&](uint32_t first, uint32_t count) {
    a.base = first;
    if (qb)
      hipLaunchKernelGGL((k_qk64_outer<KS, true>), dim3(count), dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL((k_qk64_outer<KS, false>), dim3(count), dim3(256), 0, st, a);
  });
}

// Fewer rows than 16, columns than 64 or terms than 16 leave matrix-core tiles padded, and a factor of one or few rows
// then takes longer than a thread per output.  In ns of the whole device, by the slopes of 64 vectors: a thread per output
// (K + 7) / 4000 each (a factor entry read for every vector: more than twice that), a tile of 16 x 64 one and one more for every 16 terms, half
// as much again where three of the workgroup's waves have no rows.  64 vectors, tiles / threads: a 1 x 40000 matrix (1, 64) 167 /
// 37 us, 40000 x 1 449 / 37, 8 x 40000 (4, 64) 265 / 157, 16 x 40000 (4, 8) 205 / 110, 768 x 768 (3, 3) 59 / 72.
bool outer_thin(const Qk64Outer &t, int vb) {
  const double tiles = (double)cdiv(t.M, 16) * (double)cdiv(t.N, 64) * (t.M <= 16 ? 1.5 : 1.0);
  return (vb == 4 ? 0.25e-3 : 0.6e-3) * t.M * t.N * (double)(t.K + 7) < tiles * (double)(1 + cdiv(t.K, 16));
}

// Transposes (fp32 operands): thin outputs by k_qk64_thin.
void launch_outer_T(const Qk64OuterArgs &a, hipStream_t st) {
  Qk64OuterArgs wide{}, thin{};
  wide.nv = thin.nv = a.nv;
  wide.out_bf16 = thin.out_bf16 = a.out_bf16;
  const int vb = a.nv >= 4 ? 4 : 1;
  int64_t blk = 0;
  for (int i = 0; i < a.n; ++i) {
    if (!outer_thin(a.t[i], vb)) {
      wide.t[wide.n++] = a.t[i];
      continue;
    }
    Qk64Outer &t = thin.t[thin.n];
    t = a.t[i];
    t.nbn = (int)cdiv((int64_t)t.M * t.N, 256);
    thin.blk0[thin.n++] = (uint32_t)blk;
    blk += t.nbn * cdiv(a.nv, vb);
  }
  launch_outer<false>(wide, false, st);
  grid_parts(blk, [&](uint32_t first, uint32_t count) {
    thin.base = first;
    if (vb == 4)
      hipLaunchKernelGGL(k_qk64_thin<4>, dim3(count), dim3(256), 0, st, thin);
    else
      hipLaunchKernelGGL(k_qk64_thin<1>, dim3(count), dim3(256), 0, st, thin);
  });
}

}  // namespace

// The order with fewer products: A first U = A X (dA x n), else T = X B^T (m x dB).
static bool qk64_afirst(const LayerDesc &ld) {
  const double m = ld.m, n = ld.nc, da = ld.da, db = ld.db;
  return m * n * da + n * da * db < m * n * db + m * da * db;
}

Qk64Group qk64_group(const sk_sketch *s, const int *layers, int count, int64_t bc, int64_t ws_bytes) {
  Qk64Group g{};
  int64_t off = 0;  // floats
  while (g.n < count && g.n < kQk64Tasks) {
    const LayerDesc &ld = s->layers[layers[g.n]];
    const bool af = qk64_afirst(ld);
    const int64_t need = bc * (af ? (int64_t)ld.da * ld.nc : (int64_t)ld.m * ld.db);
    if (g.n && (off + need) * 4 > ws_bytes) break;  // one layer always fits: the caller sized bc for it
    g.layer[g.n] = layers[g.n];
    g.afirst[g.n] = af;
    g.t_off[g.n] = off;
    off += (need + 3) & ~3ll;
    ++g.n;
  }
  // second contraction: k ranges of 512 beyond 1024 terms (a workgroup's chain of dependent MFMAs is
  // 64 cycles x tiles per four terms and wave), as far as the partial sums fit behind the intermediates
  int64_t room = ws_bytes - off * 4;
  for (int i = 0; i < g.n; ++i) {
    const LayerDesc &ld = s->layers[g.layer[i]];
    const int64_t K = g.afirst[i] ? ld.nc : ld.m, per = bc * ld.da * ld.db * 8;
    int64_t nk = K <= 1024 ? 1 : cdiv(K, 512);
    if (nk > 1 && nk * per > room) nk = room >= 2 * per ? room / per : 1;
    const int64_t klen = cdiv(cdiv(K, nk), 16) * 16;
    nk = cdiv(K, klen);
    g.klen[i] = klen;
    g.nk[i] = (int32_t)nk;
    g.part_off[i] = -1;
    if (nk > 1) {
      g.part_off[i] = off;
      off += nk * per / 4;
      room -= nk * per;
    }
  }
  return g;
}

void launch_qk64_first(const sk_sketch *s, const Qk64Group &g, const void *const *x, int dtype, int64_t b_begin,
                       int64_t bc, float *ws, hipStream_t st) {
  const bool bf = dtype == SK_BF16;
  Qk64DotArgs d{};
  Qk64OuterArgs o{};
  d.nv = o.nv = bc;
  for (int i = 0; i < g.n; ++i) {
    const LayerDesc &ld = s->layers[g.layer[i]];
    const int64_t mn = (int64_t)ld.m * ld.nc;
    const void *xv = (const char *)x[i] + b_begin * mn * (bf ? 2 : 4);
    if (g.afirst[i]) {  // U[a][j] = sum_i A[a][i] X[i][j]
      Qk64Outer &t = o.t[o.n++];
      t.p = s->d_qka + ld.fa_off;
      t.psk = 1;
      t.psi = ld.m;
      t.q = xv;
      t.qvs = mn;
      t.o = ws + g.t_off[i];
      t.ovs = (int64_t)ld.da * ld.nc;
      t.M = ld.da;
      t.N = ld.nc;
      t.K = ld.m;
    } else {  // T^T[c][i] = sum_j B[c][j] X[i][j]
      Qk64Dot &t = d.t[d.n++];
      t.p = s->d_qkbf + ld.fb_off;
      t.q = xv;
      t.qvs = mn;
      t.o = ws + g.t_off[i];
      t.ovs = (int64_t)ld.m * ld.db;
      t.ldo = ld.m;
      t.np = ld.db;
      t.nq = ld.m;
      t.K = ld.nc;
      t.nk = 1;
      t.klen = cdiv(ld.nc, 16) * 16;
    }
  }
  launch_dot(d, bf, st);
  launch_outer<true>(o, bf, st);
}

void launch_qk64_second(const sk_sketch *s, const Qk64Group &g, int64_t b_begin, int64_t bc, float *ws, float *out,
                        bool accumulate, hipStream_t st) {
  Qk64DotArgs d{}, r{};
  d.nv = r.nv = bc;
  d.accumulate = r.accumulate = accumulate;
  int64_t blk = 0;
  for (int i = 0; i < g.n; ++i) {
    const LayerDesc &ld = s->layers[g.layer[i]];
    Qk64Dot &t = d.t[d.n++];
    const float *im = ws + g.t_off[i];
    if (g.afirst[i]) {  // Y[a][c] = sum_j U[a][j] B[c][j]
      t.p = im;
      t.pvs = (int64_t)ld.da * ld.nc;
      t.q = s->d_qkbf + ld.fb_off;
      t.K = ld.nc;
    } else {  // Y[a][c] = sum_i A[a][i] T^T[c][i]
      t.p = s->d_qka + ld.fa_off;
      t.q = im;
      t.qvs = (int64_t)ld.m * ld.db;
      t.K = ld.m;
    }
    t.o = out + b_begin * s->D + ld.qk_col;
    t.ovs = s->D;
    t.ldo = ld.db;
    t.np = ld.da;
    t.nq = ld.db;
    t.nk = g.nk[i];
    t.klen = g.klen[i];
    if (g.part_off[i] >= 0) {
      t.part = (double *)(ws + g.part_off[i]);
      r.t[r.n] = t;
      r.blk0[r.n++] = (uint32_t)blk;
      blk += cdiv((int64_t)ld.da * ld.db * bc, 256);
    }
  }
  launch_dot(d, false, st);
  grid_parts(blk, [&](uint32_t first, uint32_t count) {
    r.base = first;
    hipLaunchKernelGGL(k_qk64_sum, dim3(count), dim3(256), 0, st, r);
  });
}

Qk64Group qk64_group_T(const sk_sketch *s, int l0, int count, int64_t bc, int64_t ws_bytes) {
  Qk64Group g{};
  int64_t off = 0;
  while (g.n < count && g.n < kQk64Tasks) {
    const LayerDesc &ld = s->layers[l0 + g.n];
    const double m = ld.m, n = ld.nc, da = ld.da, db = ld.db;
    const bool af = da * db * n + m * n * da < da * db * m + m * n * db;  // Z B first, then A^T (Z B)
    const int64_t need = bc * (af ? (int64_t)ld.da * ld.nc : (int64_t)ld.m * ld.db);
    if (g.n && (off + need) * 4 > ws_bytes) break;
    g.layer[g.n] = l0 + g.n;
    g.afirst[g.n] = af;
    g.t_off[g.n] = off;
    off += (need + 3) & ~3ll;
    ++g.n;
  }
  return g;
}

void launch_qk64_T(const sk_sketch *s, const Qk64Group &g, const float *z, int64_t b_begin, int64_t bc, float *ws,
                   void *const *out, int out_dtype, const void *const *theta0, hipStream_t st) {
  Qk64OuterArgs a{}, b{};
  a.nv = b.nv = bc;
  a.n = b.n = g.n;
  b.out_bf16 = out_dtype == SK_BF16;
  for (int i = 0; i < g.n; ++i) {
    const LayerDesc &ld = s->layers[g.layer[i]];
    const float *A = s->d_qka + ld.fa_off, *B = s->d_qkbf + ld.fb_off;
    Qk64Outer &t = a.t[i], &u = b.t[i];
    t.p = z + b_begin * s->D + ld.qk_col;
    t.pvs = s->D;
    t.o = ws + g.t_off[i];
    if (g.afirst[i]) {  // V[a][j] = sum_c Z[a][c] B[c][j]
      t.psk = 1;
      t.psi = ld.db;
      t.q = B;
      t.M = ld.da;
      t.N = ld.nc;
      t.K = ld.db;
      u.p = A;  // X'[i][j] = sum_a A[a][i] V[a][j]
      u.q = t.o;
      u.qvs = (int64_t)ld.da * ld.nc;
      u.K = ld.da;
    } else {  // U^T[c][i] = sum_a Z[a][c] A[a][i]
      t.psk = ld.db;
      t.psi = 1;
      t.q = A;
      t.M = ld.db;
      t.N = ld.m;
      t.K = ld.da;
      u.p = ws + g.t_off[i];  // X'[i][j] = sum_c U^T[c][i] B[c][j]
      u.pvs = (int64_t)ld.m * ld.db;
      u.q = B;
      u.K = ld.db;
    }
    t.ovs = (int64_t)t.M * t.N;
    u.psk = ld.m;
    u.psi = 1;
    u.o = (char *)out[i] + b_begin * (int64_t)ld.m * ld.nc * (out_dtype == SK_BF16 ? 2 : 4);
    u.ovs = (int64_t)ld.m * ld.nc;
    u.theta = theta0 ? (const float *)theta0[i] : nullptr;
    u.M = ld.m;
    u.N = ld.nc;
  }
  launch_outer_T(a, st);
  launch_outer_T(b, st);
}

}  // namespace sk
