// sk_ffd_m.hip -- FFD (eq. fastfood) with 2^14 <= D <= 2^19.
//
// A block's coordinates are i = (r, c), r < R = D / 1024, c < 1024, and
// H_D = H_R (x) H_1024: a row kernel transforms 8 rows of 1024 in LDS, a column
// kernel a tile of 2^lgcs columns by R rows.  Four passes per direction over
// the live blocks; g carries 1/D (a power of two) for both unnormalised
// transforms, so that intermediates stay within sqrt(D) of the input either way.
// Normalised row passes would keep them closer, but cost 2 us of 42 to 86 each
// (153 blocks of 2^16, 4 vectors):
//   forward     rows(x) -> columns, times g -> rows gathered through
//               pi_b^{-1} -> columns, signs, summed over a run of blocks
//   transpose   rows(B_b z) -> columns -> rows gathered through pi_b, times g
//               -> columns, theta0, written
// The gather stays inside one block (64 KB to 2 MB), whose workgroups are
// placed on one XCD (workgroups go to the XCDs in turn) so that it hits that
// XCD's L2, unless that leaves the device idle (local_blocks).  The Feistel network's eight round functions depend on one half of
// the index only, so a workgroup tabulates them in LDS (2 KB to 12 KB, where
// the row tile goes afterwards: 1 k to 6 k hashes for its 8192 coordinates
// instead of 64 k; two 32-bit multiplies per hash made the permutation the
// largest VALU item).  Against the passes over single blocks that this
// replaces (a copy, two transforms of two passes, a scatter, a sum over the
// blocks by one thread per output and sign hashes per coordinate), S^T z + S x
// of 1e7 parameters at D = 2^16 (one vector) went from 521 to 234 us.
#include <algorithm>
#include <type_traits>

#include "sk_kcommon.h"
#include "sk_launch.h"

namespace sk {

namespace {

// Workgroup -> (block b, part t of 2^lgT): the parts of each of the first
// `local` blocks (a multiple of 8) on one XCD, those of the others in a row.
// False past the last block.
__device__ __forceinline__ bool place(uint32_t id, int lgT, int64_t nblk, int64_t local, int64_t &b, int &t) {
  const bool spread = id >= (uint32_t)local << lgT;
  const uint32_t q = spread ? id - ((uint32_t)local << lgT) : id >> 3;
  b = spread ? local + (q >> lgT) : (int64_t)(q >> lgT) * 8 + (id & 7);
  t = (int)(q & ((1u << lgT) - 1));
  return b < nblk;
}

// The round functions of a permutation of lgD bits as tables in LDS: rounds
// 0, 2, .. (indexed by the low half) then 1, 3, .. (by the high half).
struct FeistelLds {
  const uint16_t *t;
  int wl, nl, nh;
  __device__ __forceinline__ uint32_t fwd(uint32_t x) const {
    uint32_t hi = x >> wl, lo = x & (nl - 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      hi ^= t[r * nl + lo];
      lo ^= t[4 * nl + r * nh + hi];
    }
    return (hi << wl) | lo;
  }
  __device__ __forceinline__ uint32_t inv(uint32_t y) const {
    uint32_t hi = y >> wl, lo = y & (nl - 1);
#pragma unroll
    for (int r = 3; r >= 0; --r) {
      lo ^= t[4 * nl + r * nh + hi];
      hi ^= t[r * nl + lo];
    }
    return (hi << wl) | lo;
  }
};

// Filled by the whole workgroup; the caller synchronises.
__device__ __forceinline__ FeistelLds feistel_fill(uint16_t *t, uint32_t layer, uint32_t pid, int lgD, Key key) {
  const PermKey pk = perm_key(layer, ST_FFDPERM, pid, (uint32_t)lgD, key);
  FeistelLds f{t, lgD / 2, 1 << (lgD / 2), 1 << (lgD - lgD / 2)};
  for (int e = threadIdx.x; e < f.nl; e += blockDim.x)
#pragma unroll
    for (int r = 0; r < 4; ++r) t[r * f.nl + e] = (uint16_t)(fmix32((uint32_t)e ^ pk.k[2 * r]) & pk.mh);
  for (int e = threadIdx.x; e < f.nh; e += blockDim.x)
#pragma unroll
    for (int r = 0; r < 4; ++r) t[4 * f.nl + r * f.nh + e] = (uint16_t)(fmix32((uint32_t)e ^ pk.k[2 * r + 1]) & pk.ml);
  return f;
}

enum { kRowsX = 0, kRowsZ = 1, kRowsInv = 2, kRowsFwd = 3 };

}  // namespace

// Row kernel: workgroup per 8 rows of a block (and every gridDim.y-th vector);
// thread: columns 4 tid .. + 3 of each row.
//   kRowsX    x of the layer (zero past its end)
//   kRowsZ    B_b z
//   kRowsInv  src gathered through pi_b^{-1}
//   kRowsFwd  g / D . (src gathered through pi_b)
template <int SRC, bool BF16>
__global__ __launch_bounds__(256, SRC == kRowsFwd ? 3 : 4) void k_ffdM_rows(const LayerDesc *__restrict__ layers, int layer,
                                                   const void *__restrict__ src, int lgD, int64_t nblk,
                                                   int64_t local, int64_t b_begin, int64_t bc, float *__restrict__ w,
                                                   Key key) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  typedef uint16_t h4u __attribute__((ext_vector_type(4), aligned(2)));
  using L = Lds1024<8>;
  __shared__ __align__(16) float s[L::kFloats];
  __shared__ __align__(16) uint32_t sgn[SRC == kRowsZ ? 256 : 1];
  const LayerDesc &ld = layers[layer];
  int64_t b;
  int t;
  if (!place(blockIdx.x, lgD - 13, nblk, local, b, t)) return;  // uniform
  const int64_t D = 1ll << lgD;
  const int col = 4 * threadIdx.x;
  const int i0 = t * 8192;  // first coordinate of the rows, within the block
  uint32_t idx[8][4];
  float g[8][4];
  if (SRC == kRowsInv || SRC == kRowsFwd) {
    const FeistelLds f = feistel_fill((uint16_t *)s, (uint32_t)ld.layer_id, (uint32_t)b, lgD, key);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t i = (uint32_t)(i0 + r * 1024 + col + q);
        idx[r][q] = SRC == kRowsInv ? f.inv(i) : f.fwd(i);
      }
    __syncthreads();  // the tables make room for the rows
  }
  if (SRC == kRowsFwd) {
    const float gs = 1.0f / (float)(1 << lgD);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      gauss4((uint64_t)(b * D + i0 + r * 1024 + col) >> 2, (uint32_t)ld.layer_id, ST_GAUSS, key, g[r]);
#pragma unroll
      for (int q = 0; q < 4; ++q) g[r][q] *= gs;
    }
  }
  if (SRC == kRowsZ) {
    if (threadIdx.x < 64) {  // one Philox block per 128 coordinates
      const W4 wd = philox((uint64_t)(b * D + i0) / 128 + threadIdx.x, (uint32_t)ld.layer_id, ST_SIGN, key);
      *reinterpret_cast<uint4 *>(&sgn[4 * threadIdx.x]) = make_uint4(wd.w[0], wd.w[1], wd.w[2], wd.w[3]);
    }
    __syncthreads();
  }
  for (int64_t v = blockIdx.y; v < bc; v += gridDim.y) {
    float e[8][4];
    if (SRC == kRowsX) {
      const int64_t x0 = (b_begin + v) * ld.n;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int64_t j = b * D + i0 + r * 1024 + col, lim = ld.n - j;
#pragma unroll
        for (int q = 0; q < 4; ++q) e[r][q] = 0.0f;
        if (lim >= 4) {
          if (BF16) {
            const h4u u = *reinterpret_cast<const h4u *>((const uint16_t *)src + x0 + j);
#pragma unroll
            for (int q = 0; q < 4; ++q) e[r][q] = bf16_to_f32(u[q]);
          } else {
            const f4u u = *reinterpret_cast<const f4u *>((const float *)src + x0 + j);
#pragma unroll
            for (int q = 0; q < 4; ++q) e[r][q] = u[q];
          }
        } else if (lim > 0) {
          load4<BF16, false>(src, x0 + j, lim, e[r]);
        }
      }
    } else if (SRC == kRowsZ) {
      const float *z = (const float *)src + (b_begin + v) * D + i0 + col;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const f4u u = *reinterpret_cast<const f4u *>(z + r * 1024);  // z may start at any element
        const uint32_t bits = sgn[r * 32 + (col >> 5)] >> (col & 31);
#pragma unroll
        for (int q = 0; q < 4; ++q) e[r][q] = flip(u[q], (bits >> q) & 1u);
      }
    } else {
      const float *blk = (const float *)src + (v * nblk + b) * D;
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) e[r][q] = blk[idx[r][q]];
      if (SRC == kRowsFwd) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
          for (int q = 0; q < 4; ++q) e[r][q] *= g[r][q];
      }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) s[L::idx(r, col + q)] = e[r][q];
    __syncthreads();
    fwht1024_lds<8>(s);
    float *dst = w + (v * nblk + b) * D + i0;
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        dst[r * 1024 + threadIdx.x + 256 * k] = s[L::idx(r, threadIdx.x + 256 * k)];
    __syncthreads();
  }
}

// Column kernels: tile of 2^LGCS columns x R rows (2^LGT values) at LDS places
// p16(e), e = (r << LGCS) | c.  Everything is a constant of D: a thread's
// elements tid + 256 i (or 4 tid + 1024 i) then differ by constants in LDS and
// in the block, which ride on instruction and scalar offsets; computed per
// element they filled the registers (108 to 140 spilled: the last pass of the
// transpose 87 us against 23, the block sum 72 against 21, at D = 2^16).  Tiles
// of 2^13 values keep pieces of 128 bytes up to D = 2^18; 2^19 takes 2^14.
namespace {
template <int LGD>
struct Tile {
  static constexpr int LGT = LGD <= 18 ? 13 : 14, LGCS = LGT - (LGD - 10), R = 1 << (LGD - 10);
  static constexpr int NE = 1 << (LGT - 8), NG = NE / 4, TILES = 1024 >> LGCS, FLOATS = p16_floats(1 << LGT);
  static constexpr int OCC = LGT == 13 ? 4 : 2;  // workgroups per CU, by LDS
  // element offset in the block of e = tid + 256 i from that of e = tid
  static constexpr int off1(int i) { return LGCS <= 8 ? i << (10 + 8 - LGCS) : (i >> 1) * 1024 + (i & 1) * 256; }
  // of e = 4 tid + 1024 i from e = 4 tid
  static constexpr int off4(int i) { return i << (20 - LGCS); }
  static __device__ __forceinline__ int place1() { return (threadIdx.x >> LGCS) * 1024 + (threadIdx.x & ((1 << LGCS) - 1)); }
  static __device__ __forceinline__ int place4() {
    const int e = 4 * threadIdx.x;
    return (e >> LGCS) * 1024 + (e & ((1 << LGCS) - 1));
  }
  // the tile at column c0 of block `blk` into registers, and from there into LDS
  static __device__ __forceinline__ void load(const float *blk, int c0, float (&x)[NE]) {
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(blk, 4u << LGD);
    const int voff = (place1() + c0) * 4;
#pragma unroll
    for (int i = 0; i < NE; ++i) x[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, off1(i) * 4, 0));
  }
  static __device__ __forceinline__ void stage(float *s, const float (&x)[NE]) {
    float *d = s + p16(threadIdx.x);
#pragma unroll
    for (int i = 0; i < NE; ++i) d[272 * i] = x[i];
  }
};
}  // namespace

// In place: H_R along the rows, times g / D (forward).
template <int LGD, bool G>
__global__ __launch_bounds__(256, Tile<LGD>::OCC) void k_ffdM_cols(const LayerDesc *__restrict__ layers, int layer,
                                                                   int64_t nblk, int64_t local, int64_t bc,
                                                                   float *__restrict__ w, Key key) {
  using T = Tile<LGD>;
  __shared__ __align__(16) float s[T::FLOATS];
  const LayerDesc &ld = layers[layer];
  int64_t b;
  int t;
  if (!place(blockIdx.x, 10 - T::LGCS, nblk, local, b, t)) return;
  const int c0 = t << T::LGCS;
  float x[T::NE];
  int64_t v = blockIdx.y;
  T::load(w + ((v * nblk + b) << LGD), c0, x);
  float gg[T::NG][4];
  if (G) {
    const uint64_t q0 = ((uint64_t)(b << LGD) + (uint64_t)(T::place4() + c0)) >> 2;
#pragma unroll
    for (int i = 0; i < T::NG; ++i) {
      gauss4(q0 + T::off4(i) / 4, (uint32_t)ld.layer_id, ST_GAUSS, key, gg[i]);
#pragma unroll
      for (int q = 0; q < 4; ++q) gg[i][q] *= 1.0f / (float)(1 << LGD);
    }
  }
  for (;;) {
    T::stage(s, x);
    lds_fwht_regs(s, T::LGT, T::LGCS);
    // Global stores: a 16-byte buffer store with its offset in a scalar register must not be followed at once by
    // a write to its data registers, and the compiler inserts no wait for that form (seen as wrong third entries of
    // a piece, in a few of 10^7, when the next LDS address went to that register).
    float *o = w + ((v * nblk + b) << LGD) + c0 + T::place4();
    const float *d = s + p16(4 * threadIdx.x);
#pragma unroll
    for (int i = 0; i < T::NG; ++i) {
      float4 y = make_float4(d[1088 * i], d[1088 * i + 1], d[1088 * i + 2], d[1088 * i + 3]);
      if (G) y = make_float4(y.x * gg[i][0], y.y * gg[i][1], y.z * gg[i][2], y.w * gg[i][3]);
      *reinterpret_cast<float4 *>(o + T::off4(i)) = y;
    }
    v += gridDim.y;
    if (v >= bc) return;
    __syncthreads();
    T::load(w + ((v * nblk + b) << LGD), c0, x);
  }
}

// Transpose, last pass: H_R, theta0, the layer's outputs.
template <int LGD>
__global__ __launch_bounds__(256, Tile<LGD>::OCC) void k_ffdM_out(const LayerDesc *__restrict__ layers, int layer,
                                                                  int64_t nblk, int64_t local, int64_t b_begin,
                                                                  int64_t bc, const float *__restrict__ w, void *__restrict__ out,
                                                                  int out_dtype, const float *__restrict__ theta0) {
  using T = Tile<LGD>;
  __shared__ __align__(16) float s[T::FLOATS];
  const int64_t n = layers[layer].n;
  int64_t b;
  int t;
  if (!place(blockIdx.x, 10 - T::LGCS, nblk, local, b, t)) return;
  const int64_t j0 = b << LGD;
  const int lim = (int)(n - j0 < (1ll << LGD) ? n - j0 : 1ll << LGD);  // entries of the block
  const int i0 = T::place1() + (t << T::LGCS);
  // a whole block takes scalar offsets; the last one compares every entry with its end
  const bool full = lim == 1 << LGD;
  float x[T::NE], th[T::NE];
  int64_t v = blockIdx.y;
  T::load(w + ((v * nblk + b) << LGD), t << T::LGCS, x);
#pragma unroll
  for (int i = 0; i < T::NE; ++i) th[i] = 0.0f;
  if (theta0 && full) T::load(theta0 + j0, t << T::LGCS, th);
  for (;;) {
    T::stage(s, x);
    lds_fwht_regs(s, T::LGT, T::LGCS);
    const float *d = s + p16(threadIdx.x);
    const int64_t o0 = (b_begin + v) * n + j0;
    if (!full) {
#pragma unroll 1
      for (int i = 0; i < T::NE; ++i) {
        const int k = i0 + T::off1(i);
        if (k < lim) store_out(out, out_dtype, o0 + k, d[272 * i] + (theta0 ? theta0[j0 + k] : 0.0f));
      }
    } else if (out_dtype == SK_BF16) {
      uint16_t *o = (uint16_t *)out + o0;
#pragma unroll
      for (int i = 0; i < T::NE; ++i) (o + T::off1(i))[i0] = f32_to_bf16(d[272 * i] + th[i]);
    } else {
      const __amdgpu_buffer_rsrc_t r = buf_rsrc((float *)out + o0, 4u << LGD);
#pragma unroll
      for (int i = 0; i < T::NE; ++i)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d[272 * i] + th[i]), r, i0 * 4, T::off1(i) * 4, 0);
    }
    v += gridDim.y;
    if (v >= bc) return;
    __syncthreads();
    T::load(w + ((v * nblk + b) << LGD), t << T::LGCS, x);
  }
}

// Forward, last pass: H_R and the signs of the blocks of run blockIdx.z, summed
// in registers in block order, to part[run][v][D].  gridDim.x =
// tiles: a run's tile stays on one workgroup, its next block in flight.
template <int LGD>
__global__ __launch_bounds__(256, Tile<LGD>::OCC) void k_ffdM_sum(const LayerDesc *__restrict__ layers, int layer,
                                                                  int64_t nblk, int64_t per, int64_t bc,
                                                                  const float *__restrict__ w,
                                                                  float *__restrict__ part, Key key) {
  using T = Tile<LGD>;
  constexpr int WPR = T::LGCS > 7 ? 1 << (T::LGCS - 5) : 4;  // sign words per row (whole Philox blocks)
  constexpr int NB = T::R * WPR / 4;
  __shared__ __align__(16) float s[T::FLOATS];
  __shared__ __align__(16) uint32_t sgn[T::R * WPR];
  const LayerDesc &ld = layers[layer];
  const int c0 = blockIdx.x << T::LGCS;
  const int64_t v = blockIdx.y;
  const int64_t b0 = blockIdx.z * per, b1 = b0 + per < nblk ? b0 + per : nblk;
  const int c = c0 + (threadIdx.x & ((1 << T::LGCS) - 1));
  const uint32_t *sw = sgn + (threadIdx.x >> T::LGCS) * WPR + (T::LGCS > 7 ? (c - c0) >> 5 : (c >> 5) & 3);
  float acc[T::NE], x[T::NE];
#pragma unroll
  for (int i = 0; i < T::NE; ++i) acc[i] = 0.0f;
  T::load(w + ((v * nblk + b0) << LGD), c0, x);
  for (int64_t b = b0; b < b1; ++b) {
    for (int u = threadIdx.x; u < NB; u += 256) {
      const int r = u / (WPR / 4), k = u % (WPR / 4);
      const W4 wd = philox((((uint64_t)b << LGD) + (uint64_t)(r * 1024 + c0)) / 128 + (uint64_t)k,
                           (uint32_t)ld.layer_id, ST_SIGN, key);
      *reinterpret_cast<uint4 *>(&sgn[4 * u]) = make_uint4(wd.w[0], wd.w[1], wd.w[2], wd.w[3]);
    }
    T::stage(s, x);
    if (b + 1 < b1) T::load(w + ((v * nblk + b + 1) << LGD), c0, x);
    lds_fwht_regs(s, T::LGT, T::LGCS);
    const float *d = s + p16(threadIdx.x);
#pragma unroll
    for (int i = 0; i < T::NE; ++i) {
      // rows step by off1 / 1024; LGCS = 9: odd i is 256 columns (8 words) on
      const int wi = T::LGCS <= 8 ? (T::off1(i) >> 10) * WPR : (i >> 1) * WPR + (i & 1) * 8;
      acc[i] += flip(d[272 * i], (sw[wi] >> (c & 31)) & 1u);
    }
    __syncthreads();
  }
  float *o = part + (((int64_t)blockIdx.z * bc + v) << LGD) + T::place1() + c0;
#pragma unroll
  for (int i = 0; i < T::NE; ++i) o[T::off1(i)] = acc[i];
}

namespace {
// Vectors of a call share a block's g and indices; more workgroups than 2048 (eight per CU) are not needed.
unsigned shares(int64_t blocks, int64_t bc) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(bc, 2048 / std::max<int64_t>(1, blocks)));
}
// Blocks whose parts share an XCD (place); the grid has max(nblk, local) blocks.  Beyond the last eight, one to three
// blocks on an XCD each leave most of the device idle, which costs more than a gather outside the XCD's L2 once the
// call has 2^19 values per block: D = 2^19, one block, 1 / 4 / 16 vectors, transpose: 73 / 174 / 617 us on one XCD, 57 /
// 75 / 161 spread; nine blocks of 2^17, 16 vectors, 258 / 178.  Fewer values stay in L2 (D = 2^16, one block, one vector
// 32.5 / 38), and four blocks or more fill enough of the device (D = 2^18, four, 16 vectors forward 258 / 292; D = 2^17,
// seven, 4 vectors 61 / 79).
int64_t local_blocks(int64_t nblk, int64_t D, int64_t bc) {
  const int64_t rest = nblk & 7;
  return rest <= 3 && D * bc >= 1 << 19 ? nblk - rest : (nblk + 7) & ~7ll;
}
}  // namespace

bool ffd_mid_path(const sk_sketch *s) { return s->D > (1ll << kFfdSmallMax) && s->D < (1ll << 20); }

namespace {
template <class F>
void with_lgD(int lgD, F f) {
  switch (lgD) {
    case 14: f(std::integral_constant<int, 14>()); break;
    case 15: f(std::integral_constant<int, 15>()); break;
    case 16: f(std::integral_constant<int, 16>()); break;
    case 17: f(std::integral_constant<int, 17>()); break;
    case 18: f(std::integral_constant<int, 18>()); break;
    default: f(std::integral_constant<int, 19>()); break;
  }
}
}  // namespace

void run_ffd_mid_fwd(const sk_sketch *s, int layer, const void *x, int dtype, int64_t b_begin, int64_t bc, float *out,
                     bool accumulate, int phases, hipStream_t st) {
  int lgD = 14;
  while ((1ll << lgD) < s->D) ++lgD;
  const int64_t nblk = ffd_live_blocks(s, layer);
  const int64_t local = local_blocks(nblk, s->D, bc), gblk = std::max(nblk, local);
  float *w = s->ws, *w2 = s->ws + bc * nblk * s->D;
  const int64_t rgrid = gblk << (lgD - 13);
  const dim3 gr((unsigned)rgrid, shares(rgrid, bc));
  if (phases & 1) {
    if (dtype == SK_BF16)
      hipLaunchKernelGGL((k_ffdM_rows<kRowsX, true>), gr, dim3(256), 0, st, s->d_layers, layer, x, lgD, nblk, local,
                         b_begin, bc, w, s->key);
    else
      hipLaunchKernelGGL((k_ffdM_rows<kRowsX, false>), gr, dim3(256), 0, st, s->d_layers, layer, x, lgD, nblk, local,
                         b_begin, bc, w, s->key);
  }
  if (!(phases & 2)) return;
  with_lgD(lgD, [&](auto lg) {
    constexpr int LGD = decltype(lg)::value;
    const int64_t tiles = Tile<LGD>::TILES, cgrid = gblk * tiles;
    hipLaunchKernelGGL((k_ffdM_cols<LGD, true>), dim3((unsigned)cgrid, shares(cgrid, bc)), dim3(256), 0, st,
                       s->d_layers, layer, nblk, local, bc, w, s->key);
    hipLaunchKernelGGL((k_ffdM_rows<kRowsInv, false>), gr, dim3(256), 0, st, s->d_layers, layer, w, lgD, nblk, local,
                       b_begin, bc, w2, s->key);
    // runs of blocks: 1024 workgroups while each has a block; the partial sums take the place of w
    int64_t runs = std::max<int64_t>(1, std::min<int64_t>(nblk, 1024 / std::max<int64_t>(1, tiles * bc)));
    const int64_t per = (nblk + runs - 1) / runs;
    runs = (nblk + per - 1) / per;
    hipLaunchKernelGGL((k_ffdM_sum<LGD>), dim3((unsigned)tiles, (unsigned)bc, (unsigned)runs), dim3(256), 0, st,
                       s->d_layers, layer, nblk, per, bc, w2, w, s->key);
    launch_reduce_partials(w, runs, bc, s->D, b_begin, out, accumulate, st);
  });
}

void run_ffd_mid_T(const sk_sketch *s, int layer, const float *z, int64_t b_begin, int64_t bc, void *out, int out_dtype,
                   const float *theta0, int phases, hipStream_t st) {
  int lgD = 14;
  while ((1ll << lgD) < s->D) ++lgD;
  const int64_t nblk = ffd_live_blocks(s, layer);
  const int64_t local = local_blocks(nblk, s->D, bc), gblk = std::max(nblk, local);
  float *w = s->ws, *w2 = s->ws + bc * nblk * s->D;
  const int64_t rgrid = gblk << (lgD - 13);
  const dim3 gr((unsigned)rgrid, shares(rgrid, bc));
  with_lgD(lgD, [&](auto lg) {
    constexpr int LGD = decltype(lg)::value;
    const int64_t cgrid = gblk * Tile<LGD>::TILES;
    const dim3 gc((unsigned)cgrid, shares(cgrid, bc));
    if (phases & 1) {
      hipLaunchKernelGGL((k_ffdM_rows<kRowsZ, false>), gr, dim3(256), 0, st, s->d_layers, layer, z, lgD, nblk, local,
                         b_begin, bc, w, s->key);
      hipLaunchKernelGGL((k_ffdM_cols<LGD, false>), gc, dim3(256), 0, st, s->d_layers, layer, nblk, local, bc, w, s->key);
      hipLaunchKernelGGL((k_ffdM_rows<kRowsFwd, false>), gr, dim3(256), 0, st, s->d_layers, layer, w, lgD, nblk, local,
                         b_begin, bc, w2, s->key);
    }
    if (phases & 2)
      hipLaunchKernelGGL((k_ffdM_out<LGD>), gc, dim3(256), 0, st, s->d_layers, layer, nblk, local, b_begin, bc, w2,
                         out, out_dtype, theta0);
  });
}

}  // namespace sk
