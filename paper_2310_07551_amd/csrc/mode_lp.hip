// Reduced-precision mu-mode products (same operation and job tables as
// mode_f64.hip): operands and intermediates in FP32, the last mode of a
// Tucker written in FP64 on top of an FP64 base.
//
//   SETD_PREC_F32     v_mfma_f32_16x16x4f32, FP32 accumulate.
//   SETD_PREC_BF16X3  v_mfma_f32_16x16x32_bf16 with the three-term split
//                     x = h + m + l (h = bf16(x), m = bf16(x - h),
//                     l = bf16(x - h - m)) and the six products of order
//                     <= 2^-16: hh + hm + mh + hl + lh + mm, FP32 accumulate
//                     (about FP32 accuracy).
//   SETD_PREC_BF16X2  the two-term split x = h + l with hh + hl + lh (about
//                     16 significant bits, half the matrix-core work).
//                     The matrix is split once when it is packed; the tensor
//                     operand is split in registers right after its load.
//
// Per-term scale factors multiply FP32 partial sums (never a bf16 piece, and
// never inside a load, where the multiply would make the wave wait for it).
//
// Operand layouts (probed on gfx950): FP32 16x16x4 and BF16 16x16x32 put
// tile row 4 g + r in register r of lane (g, l); in the bf16 form lane (g, l)
// supplies A[l][8 g + j] and B[8 g + j][l] in slot j.
//
// Every mode has MFMA rows = i (matrix, packed tile by tile in the order the
// lanes read it), columns = the other index, k = p.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "common.hpp"

namespace setd {
namespace {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int64_t remap_xcd_lp(int64_t bid, int64_t per_xcd) {
  return (bid & 7) * per_xcd + (bid >> 3);
}

__device__ __forceinline__ int find_job_lp(const ModeJobs& J, int64_t t) { return find_job(J, t); }

// x = p[0] + p[1] (+ p[2]): each piece the bf16 rounding (RNE) of the FP32
// remainder left by the previous ones.
template <int NP>
__device__ __forceinline__ void split_bf16(const f8& x, bf8 (&p)[NP]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float r = x[j];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const __bf16 h = (__bf16)r;
      p[k][j] = h;
      r -= (float)h;
    }
  }
}

__device__ __forceinline__ f4 mfma_bf(const bf8& a, const bf8& b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// One k-chunk of the split product.  The bf16 matrix-core accumulation was
// measured on gfx950 to round with a small bias toward zero (positive-data
// mode products: mean relative error -2e-8 at n = 256, growing with the
// number of chained accumulations; FP32 MFMA: 1e-10).  A bias does not average
// out over the Tuckers and steps of the integrator, so the leading product
// h*h is formed per chunk from a zero accumulator and added to `main` with an
// FP32 VALU add (round to nearest), and the cross products of order <= 2^-8
// (NP = 2) or <= 2^-16 (NP = 3) chain in their own, 2^8 times smaller,
// accumulator `small` (unscaled; the caller applies the term's scale to it
// once).  `main` receives sc * (chunk of h*h).
// p: matrix pieces, x: tensor pieces.  Of two cross products of one order the
// first is the one with the leading piece of the matrix in mode 1, of the
// tensor in modes >= 2.
template <int NP, bool M1>
__device__ __forceinline__ void mfma_split(const bf8 (&p)[NP], const bf8 (&x)[NP], float sc, f4& main, f4& small) {
  if constexpr (NP == 3) {
    small = mfma_bf(p[1], x[1], small);
    small = M1 ? mfma_bf(p[0], x[2], small) : mfma_bf(p[2], x[0], small);
    small = M1 ? mfma_bf(p[2], x[0], small) : mfma_bf(p[0], x[2], small);
  }
  small = M1 ? mfma_bf(p[0], x[1], small) : mfma_bf(p[1], x[0], small);
  small = M1 ? mfma_bf(p[1], x[0], small) : mfma_bf(p[0], x[1], small);
  main += sc * mfma_bf(p[0], x[0], f4{0.f, 0.f, 0.f, 0.f});
}

// Writes `cnt` consecutive results starting at Y + off (all in range when
// full) as FP32 or, for an FP64 output, base + value.
template <typename TOut, typename TV>
__device__ __forceinline__ void store_run(TOut* __restrict__ Y, const double* __restrict__ base, int64_t off,
                                          const TV* v, int cnt, int valid, bool vec) {
  if (vec && valid >= cnt) {
    if constexpr (sizeof(TOut) == 4) {
      for (int e = 0; e < cnt; e += 4)
        *(f4*)(Y + off + e) = f4{(float)v[e], (float)v[e + 1], (float)v[e + 2], (float)v[e + 3]};
    } else {
      for (int e = 0; e < cnt; e += 2) {
        d2 w = d2{(double)v[e], (double)v[e + 1]};
        if (base) w += *(const d2*)(base + off + e);
        *(d2*)(Y + off + e) = w;
      }
    }
  } else {
    for (int e = 0; e < cnt; ++e) {
      if (e < valid) {
        if constexpr (sizeof(TOut) == 4) {
          Y[off + e] = (float)v[e];
        } else {
          double w = (double)v[e];
          if (base) w += base[off + e];
          Y[off + e] = w;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// FP32 with the accumulation chained on the matrix cores
// ---------------------------------------------------------------------------
// One wave computes 16 TI values of i by 16 TO of the other index, four waves
// per workgroup on neighbouring tiles; modes >= 2 tile a and b together as in
// the FP64 kernels.  MFMA rows = i (matrix), columns = the other index: lane
// (g, l) register r of the accumulator holds D[4 g + r][l].
//
// Packed FP32 matrix: entry (tile t, chunk c, lane, j) = M[16 t + l][p], zero
// past n, p = 16 c + 4 g + j in mode 1 (whose lanes read four consecutive p of
// X) and p = 16 c + 4 j + g in modes >= 2 (whose MFMA takes four consecutive
// p): the order of every sum, and with it every bit of the result, depends on
// the mode and n alone, not on the tile.
//
// Every size takes the same loop: columns and rows past the end are clamped to
// the last one (their results are not stored), and the last n % 16 values of p
// are one masked chunk.  Mode 1 loads it ahead of the loop, modes >= 2 after it:
// without the registers that hold it 7 x 2 tiles run three waves per SIMD, which
// takes modes >= 2 from 0.68 to 0.61 ms at 200^3, and mode 1, whose lanes read
// half-lines of 16 rows that three waves push out of the L1, from 0.64 to 0.97.
// In modes >= 2 the TO columns of a lane are neighbours (V), one load for all of
// them, wherever no slab ends between them; one load each was what bound the
// large sizes (256^3 last mode 1.78 -> 1.42 ms).  Whole steps against kernels of one 4 x 4 tile that
// checked every load unless n was a multiple of 32: 200^3 4.83 -> 3.40 ms,
// 150^3 2.74 -> 1.37, 256^3 8.02 -> 7.4, 100^3 0.52 -> 0.38, 300^2 0.40 -> 0.10.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // four floats at any address

__device__ __forceinline__ f4 mfma32(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <bool M1, bool V, int TI, int TO, typename Off, typename TOut>
__global__ void __launch_bounds__(256, 2) mode_f32_kernel(const ModeJobs J, int64_t per_xcd) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t t = (uint32_t)remap_xcd_lp(blockIdx.x, per_xcd) * 4 + wave;
  if (t >= (uint32_t)J.total_tiles) return;
  const ModeJob& jb = J.job[find_job_lp(J, t)];
  const uint32_t lt = t - (uint32_t)jb.tile_begin;
  const int g = lane >> 4, l = lane & 15;
  const int n = jb.n, nch = (n + 15) >> 4, nfull = n >> 4;
  const uint32_t ti = (uint32_t)jb.tiles_i;
  const uint32_t ot = lt / ti;
  const int t0 = (int)(lt - ot * ti) * TI;
  const int64_t na = M1 ? 1 : jb.na;
  const int64_t ext = M1 ? jb.nb : na * jb.nb;
  const int64_t q0 = (int64_t)ot * (16 * TO);
  const uint32_t b0 = M1 || jb.nb == 1 ? 0 : (uint32_t)((uint64_t)q0 / (uint32_t)na);
  const int64_t r0 = q0 - (int64_t)b0 * na;   // a of the tile's first column
  const int64_t origin = M1 ? q0 * n : (int64_t)b0 * na * n + r0;
  // element offset of column k of the tile (clamped to the extent) from its first
  auto column = [&](int k) -> Off {
    const int64_t rel = min(q0 + k, ext - 1) - q0;
    if (M1) return (Off)(rel * n);
    if (jb.nb == 1) return (Off)rel;
    const Off q = (Off)(r0 + rel);
    const Off bb = q / (Off)na;
    return (Off)(bb * (Off)(na * n) + (q - bb * (Off)na) - (Off)r0);
  };
  // columns of the lane: 16 o + l, or with V the TO consecutive ones from
  // TO l on (the last lanes move back to end with the last column; they keep
  // the first `skip` of theirs to themselves)
  constexpr int NX = V ? 1 : TO;
  // the moved lanes of a tile with fewer than TO columns begin before it, so
  // that with V offsets count from TO elements before the tile's first
  constexpr int kBack = V ? TO : 0;
  typedef float fv __attribute__((ext_vector_type(TO), aligned(4)));
  const int k0 = V ? (int)(min(q0 + TO * l, ext - TO) - q0) : 0, skip = TO * l - k0;
  Off xo[NX];   // byte offset of the lane's first element of each column block
#pragma unroll
  for (int o = 0; o < NX; ++o) xo[o] = (column(V ? k0 : 16 * o + l) + (Off)kBack + (M1 ? (Off)(4 * g) : (Off)na * (Off)g)) * 4;
  f4 acc[TI][TO];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int o = 0; o < TO; ++o) acc[i][o] = f4{0.f, 0.f, 0.f, 0.f};
  __builtin_amdgcn_s_setprio(1);   // products ahead of another wave's epilogue on the SIMD
  const int nterms = M1 ? 1 : jb.nterms;
  const int nt = nch;              // tiles of i
  for (int term = 0; term < nterms; ++term) {
    const float* __restrict__ x0 = (const float*)jb.X[term] + (origin - kBack);
    const float sc = (float)jb.scale[term];
    const float* at[TI];
#pragma unroll
    for (int i = 0; i < TI; ++i)
      at[i] = (const float*)jb.P[term] + (int64_t)min(t0 + i, nt - 1) * nch * 256 + 4 * lane;
    auto load_m = [&](int c, f4 (&pr)[TI]) {
#pragma unroll
      for (int i = 0; i < TI; ++i) pr[i] = *(const f4*)(at[i] + (int64_t)c * 256);
    };
    auto load = [&](int c, f4 (&xr)[TO], f4 (&pr)[TI]) {
      load_m(c, pr);
      if constexpr (M1) {
        const char* xb = (const char*)(x0 + 16 * c);
#pragma unroll
        for (int o = 0; o < TO; ++o) xr[o] = *(const f4u*)(xb + xo[o]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const char* xb = (const char*)(x0 + na * (16 * (int64_t)c + 4 * j));
          if constexpr (V) {
            const fv v = *(const fv*)(xb + xo[0]);
#pragma unroll
            for (int o = 0; o < TO; ++o) xr[o][j] = v[o];
          } else {
#pragma unroll
            for (int o = 0; o < TO; ++o) xr[o][j] = *(const float*)(xb + xo[o]);
          }
        }
      }
    };
    // the term's scale goes on the matrix in modes >= 2 and on the sum in mode 1
    auto mma = [&](const f4 (&xr)[TO], const f4 (&pr)[TI]) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < TI; ++i) {
          const float pv = M1 ? pr[i][j] : pr[i][j] * sc;
#pragma unroll
          for (int o = 0; o < TO; ++o) acc[i][o] = mfma32(pv, xr[o][j], acc[i][o]);
        }
    };
    // the last n % 16 values of p: clamped loads, zero past n
    auto load_tail = [&](f4 (&xt)[TO], f4 (&pt)[TI]) {
      load_m(nfull, pt);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = M1 ? 4 * g + j : 4 * j + g, p = 16 * nfull + k;
        const float* xp = x0 + (M1 ? 1 : na) * (min(p, n - 1) - (M1 ? 4 * g : g));   // xo holds the lane's part
#pragma unroll
        for (int o = 0; o < TO; ++o) {
          const float v = *(const float*)((const char*)(V ? xp + o : xp) + xo[V ? 0 : o]);
          xt[o][j] = p < n ? v : 0.f;
        }
      }
    };
    // chunks alternate between two register sets, each loaded one chunk ahead
    f4 xr[2][TO], pr[2][TI];
    const bool tail = nch > nfull;
    if (nfull > 0) load(0, xr[0], pr[0]);
    f4 xt[M1 ? TO : 1], pt[M1 ? TI : 1];
    if constexpr (M1) {
      if (tail) load_tail(xt, pt);
    }
    int c = 0;
    for (; c + 2 <= nfull; c += 2) {
      load(c + 1, xr[1], pr[1]);
      mma(xr[0], pr[0]);
      load(min(c + 2, nfull - 1), xr[0], pr[0]);   // the last one re-reads a valid chunk: no branch
      mma(xr[1], pr[1]);
    }
    if constexpr (M1) {
      if (c < nfull) mma(xr[0], pr[0]);
      if (tail) mma(xt, pt);
    } else {
      if (tail) load_tail(xr[1], pr[1]);
      if (c < nfull) mma(xr[0], pr[0]);
      if (tail) mma(xr[1], pr[1]);
    }
  }
  __builtin_amdgcn_s_setprio(0);
  const float sc1 = M1 ? (float)jb.scale[0] : 1.f;
  const int imax = n - 16 * t0;                               // i of the tile below it
  const int omax = (int)min(ext - q0, (int64_t)(16 * TO));    // columns of the tile
  const double* __restrict__ base = (const double*)jb.base;
  if constexpr (M1) {
    TOut* __restrict__ Y = (TOut*)jb.Y + origin + 16 * t0;
    const double* __restrict__ bs = base + origin + 16 * t0;
#pragma unroll
    for (int o = 0; o < TO; ++o) {
      if (16 * o + l >= omax) continue;
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const int i0 = 16 * i + 4 * g;
        const int64_t at = (int64_t)(16 * o + l) * n + i0;
        const f4 v = sc1 * acc[i][o];
        if constexpr (sizeof(TOut) == 4) {
          if (i0 + 4 <= imax) {
            *(f4u*)(Y + at) = v;
            continue;
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (i0 + r < imax) Y[at + r] = sizeof(TOut) == 8 && base ? (TOut)((double)v[r] + bs[at + r]) : (TOut)v[r];
      }
    }
  } else {
    TOut* __restrict__ Y = (TOut*)jb.Y + (origin - kBack) + na * 16 * t0;
    const double* __restrict__ bs = base + (origin - kBack) + na * 16 * t0;
    Off yo[NX];
#pragma unroll
    for (int o = 0; o < NX; ++o) yo[o] = column(V ? k0 : 16 * o + l) + (Off)kBack;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      // the base values of a block of rows are read together, from clamped
      // indices, so that they are one wait and not one each
      double bv[4][TO];
      if (sizeof(TOut) == 8 && base) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int o = 0; o < TO; ++o)
            bv[r][o] = bs[min(16 * i + 4 * g + r, imax - 1) * na + yo[V ? 0 : o] + (V ? o : 0)];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int o = 0; o < TO; ++o) bv[r][o] = -0.0;   // the sum is then the product itself
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + 4 * g + r;
        if (row >= imax) continue;
        TOut w[TO];
#pragma unroll
        for (int o = 0; o < TO; ++o) {
          const float v = acc[i][o][r];
          w[o] = sizeof(TOut) == 8 ? (TOut)((double)v + bv[r][o]) : (TOut)v;
        }
        if constexpr (V) {
          typedef TOut tv __attribute__((ext_vector_type(TO), aligned(sizeof(TOut))));
          TOut* y = Y + row * na + yo[0];
          if (skip == 0) {
            tv x;
#pragma unroll
            for (int o = 0; o < TO; ++o) x[o] = w[o];
            *(tv*)y = x;
          } else {
#pragma unroll
            for (int o = 0; o < TO; ++o)
              if (o >= skip) y[o] = w[o];
          }
        } else {
#pragma unroll
          for (int o = 0; o < TO; ++o)
            if (16 * o + l < omax) Y[row * na + yo[o]] = w[o];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// FP32 mode 1 with the matrix panel in LDS: the scheme of the FP64 panel
// kernel (mode_f64.hip) on FP32 operands, for interior jobs with
// 192 <= n <= 256, n % 64 == 0 and 4 x 4 tiles.  A workgroup of 8 waves
// shares one 64-row panel of P (64 KB), stored in LDS in the order the MFMA
// reads it, so no wave holds P in registers; each wave computes `reps`
// 64 x 64 tiles of the workgroup's column group, its tensor loads one 16-p
// chunk ahead of the products.  The products and their order, and the scale
// applied to the FP32 accumulators, are those of the register kernel: the two
// agree bit for bit.  Measured at 3D FHN 256^3: 110 TFLOP/s against 97 for
// the register kernel (two waves per SIMD; at four, 128 registers forced
// spills: 100).  The same panel for modes >= 2 ran at 90.5 (two waves) and
// 93.6 (four) against 95.2 for the register kernel and is not used.
constexpr int kLds32Waves = 8, kLds32MinN = 192, kLds32MaxN = 256, kLds32Reps = 4;

template <typename TOut>
__global__ void __launch_bounds__(512, 1) mode1_lds32_kernel(const ModeJobs J, int64_t per_xcd, int reps) {
  __shared__ f4 panel[(kLds32MaxN / 16) * 4 * 64];   // 64 KB
  const int64_t w = remap_xcd_lp(blockIdx.x, per_xcd);
  if (w >= J.total_tiles) return;   // uniform over the workgroup
  const ModeJob& jb = J.job[find_job_lp(J, w)];
  const int64_t lw = w - jb.tile_begin;
  const int it = (int)(lw % jb.tiles_i);
  const int64_t bg = lw / jb.tiles_i;
  const int n = jb.n, nchunk = n / 16;
  const int i0 = it * 64;
  // fill: entry q = (c * 4 + m) * 64 + lane holds P[i0 + 4 l + m][16 c + 4 g + 0..3]
  {
    const float* __restrict__ PT = (const float*)jb.P[0];
    for (int q = threadIdx.x; q < nchunk * 256; q += 512) {
      const int ln = q & 63, m = (q >> 6) & 3, c = q >> 8;
      const int i = i0 + 4 * (ln & 15) + m;
      panel[q] = *(const f4*)(PT + ((int64_t)(i >> 4) * nchunk + c) * 256 + ((ln >> 4) * 16 + (i & 15)) * 4);
    }
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, l = lane & 15;
  const float sc = (float)jb.scale[0];
  for (int rep = 0; rep < reps; ++rep) {
    const int64_t bt = (bg * reps + rep) * kLds32Waves + wave;
    if (bt >= jb.tiles_a) return;   // no barrier follows
    const int64_t b0 = bt * 64;
    const float* __restrict__ X = (const float*)jb.X[0];
    const float* pb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) pb[u] = X + (b0 + 16 * u + l) * (int64_t)n + 4 * g;
    f4 acc[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[m][u] = f4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](int c, f4 (&xr)[4]) {
#pragma unroll
      for (int u = 0; u < 4; ++u) xr[u] = *(const f4*)(pb[u] + 16 * c);
    };
    auto mma = [&](int c, const f4 (&xr)[4]) {
      f4 a[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) a[m] = panel[(c * 4 + m) * 64 + lane];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[m][u] = mfma32(a[m][jj], xr[u][jj], acc[m][u]);
    };
    f4 x0[4], x1[4];
    load(0, x0);
    for (int c = 0; c < nchunk; c += 2) {   // nchunk is even (n % 32 == 0)
      load(c + 1, x1);
      mma(c, x0);
      load(c + 2 < nchunk ? c + 2 : c, x0);
      mma(c + 1, x1);
    }
    // lane (g, l) owns rows i0 + 16 g + 4 r + m of column b0 + 16 u + l
    TOut* __restrict__ Y = (TOut*)jb.Y;
    const double* __restrict__ base = (const double*)jb.base;
    const int ir = i0 + 16 * g;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float v[16];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int m = 0; m < 4; ++m) v[4 * r + m] = sc * acc[m][u][r];
      store_run<TOut>(Y, base, (b0 + 16 * u + l) * (int64_t)n + ir, v, 16, n - ir, true);
    }
  }
}

// ---------------------------------------------------------------------------
// BF16 splits
// ---------------------------------------------------------------------------
// The FP32 kernel's tiling and addressing with chunks of 32 p (lane (g, l)
// holds p = 32 c + 8 g + j in both operands) and the tensor operand split in
// registers.  Packed matrix: plane k, entry (tile t, chunk c, lane, j) = piece
// k of M[16 t + l][p], zero past n.  SUM: jobs of several terms, whose cross
// products are scaled term by term.  Tiles of 8 blocks or more run one wave per
// SIMD: bounded to two (256 registers) they spill (3D FHN 256^3: 26 against
// 115 steps/s).
template <int NP, bool M1, bool V, bool SUM, int TI, int TO, typename Off, typename TOut>
__global__ void __launch_bounds__(256, TI * TO >= 8 ? 1 : 2) mode_bf16_kernel(const ModeJobs J, int64_t per_xcd) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t t = (uint32_t)remap_xcd_lp(blockIdx.x, per_xcd) * 4 + wave;
  if (t >= (uint32_t)J.total_tiles) return;
  const ModeJob& jb = J.job[find_job_lp(J, t)];
  const uint32_t lt = t - (uint32_t)jb.tile_begin;
  const int g = lane >> 4, l = lane & 15;
  const int n = jb.n, nch = (n + 31) >> 5, nfull = n >> 5;
  const uint32_t ti = (uint32_t)jb.tiles_i;
  const uint32_t ot = lt / ti;
  const int t0 = (int)(lt - ot * ti) * TI;
  const int64_t na = M1 ? 1 : jb.na;
  const int64_t ext = M1 ? jb.nb : na * jb.nb;
  const int64_t q0 = (int64_t)ot * (16 * TO);
  const uint32_t b0 = M1 || jb.nb == 1 ? 0 : (uint32_t)((uint64_t)q0 / (uint32_t)na);
  const int64_t r0 = q0 - (int64_t)b0 * na;   // a of the tile's first column
  const int64_t origin = M1 ? q0 * n : (int64_t)b0 * na * n + r0;
  // element offset of column k of the tile (clamped to the extent) from its first
  auto column = [&](int k) -> Off {
    const int64_t rel = min(q0 + k, ext - 1) - q0;
    if (M1) return (Off)(rel * n);
    if (jb.nb == 1) return (Off)rel;
    const Off q = (Off)(r0 + rel);
    const Off bb = q / (Off)na;
    return (Off)(bb * (Off)(na * n) + (q - bb * (Off)na) - (Off)r0);
  };
  // columns of the lane: 16 o + l, or with V the TO consecutive ones from
  // TO l on (the last lanes move back to end with the last column; they keep
  // the first `skip` of theirs to themselves)
  constexpr int NX = V ? 1 : TO;
  // the moved lanes of a tile with fewer than TO columns begin before it, so
  // that with V offsets count from TO elements before the tile's first
  constexpr int kBack = V ? TO : 0;
  typedef float fv __attribute__((ext_vector_type(TO), aligned(4)));
  const int k0 = V ? (int)(min(q0 + TO * l, ext - TO) - q0) : 0, skip = TO * l - k0;
  Off xo[NX];   // byte offset of the lane's first element of each column block
#pragma unroll
  for (int o = 0; o < NX; ++o) xo[o] = (column(V ? k0 : 16 * o + l) + (Off)kBack + (M1 ? (Off)(8 * g) : (Off)na * (Off)(8 * g))) * 4;
  f4 acc[TI][TO], accs[TI][TO], acct[SUM ? TI : 1][SUM ? TO : 1];   // leading, cross, finished terms' cross products
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int o = 0; o < TO; ++o) {
      acc[i][o] = accs[i][o] = f4{0.f, 0.f, 0.f, 0.f};
      if constexpr (SUM) acct[i][o] = f4{0.f, 0.f, 0.f, 0.f};
    }
  __builtin_amdgcn_s_setprio(1);   // products ahead of another wave's epilogue on the SIMD
  const int nterms = SUM ? jb.nterms : 1;
  const int nt = (n + 15) >> 4;    // tiles of i
  const int64_t plane = (int64_t)nt * nch * 512;
  float sc = 0.f;
  for (int term = 0; term < nterms; ++term) {
    const float* __restrict__ x0 = (const float*)jb.X[term] + (origin - kBack);
    sc = (float)jb.scale[term];
    const __bf16* at[TI];
#pragma unroll
    for (int i = 0; i < TI; ++i)
      at[i] = (const __bf16*)jb.P[term] + (int64_t)min(t0 + i, nt - 1) * nch * 512 + 8 * lane;
    auto load_m = [&](int c, bf8 (&pr)[TI][NP]) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int k = 0; k < NP; ++k) pr[i][k] = *(const bf8*)(at[i] + k * plane + (int64_t)c * 512);
    };
    auto load = [&](int c, f8 (&xr)[TO], bf8 (&pr)[TI][NP]) {
      load_m(c, pr);
      if constexpr (M1) {
        const char* xb = (const char*)(x0 + 32 * c);
#pragma unroll
        for (int o = 0; o < TO; ++o) {
          const f4 lo = *(const f4u*)(xb + xo[o]), hi = *(const f4u*)(xb + xo[o] + 16);
          xr[o] = f8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const char* xb = (const char*)(x0 + na * (32 * (int64_t)c + j));
          if constexpr (V) {
            const fv v = *(const fv*)(xb + xo[0]);
#pragma unroll
            for (int o = 0; o < TO; ++o) xr[o][j] = v[o];
          } else {
#pragma unroll
            for (int o = 0; o < TO; ++o) xr[o][j] = *(const float*)(xb + xo[o]);
          }
        }
      }
    };
    // the last n % 32 values of p: clamped loads, zero past n
    auto load_tail = [&](f8 (&xr)[TO], bf8 (&pr)[TI][NP]) {
      load_m(nfull, pr);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int p = 32 * nfull + 8 * g + j;
        const float* xp = x0 + (M1 ? 1 : na) * (min(p, n - 1) - 8 * g);   // xo holds the lane's part
#pragma unroll
        for (int o = 0; o < TO; ++o) {
          const float v = *(const float*)((const char*)(V ? xp + o : xp) + xo[V ? 0 : o]);
          xr[o][j] = p < n ? v : 0.f;
        }
      }
    };
    auto mma = [&](const f8 (&xr)[TO], const bf8 (&pr)[TI][NP]) {
      bf8 xp[TO][NP];
#pragma unroll
      for (int o = 0; o < TO; ++o) split_bf16<NP>(xr[o], xp[o]);
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int o = 0; o < TO; ++o) mfma_split<NP, M1>(pr[i], xp[o], sc, acc[i][o], accs[i][o]);
    };
    // chunks alternate between two register sets, each loaded one chunk ahead
    f8 xa[TO], xc[TO];
    bf8 pa[TI][NP], pc[TI][NP];
    if (nfull > 0) load(0, xa, pa);
    int c = 0;
    for (; c + 2 <= nfull; c += 2) {
      load(c + 1, xc, pc);
      __builtin_amdgcn_sched_barrier(0);
      mma(xa, pa);
      load(min(c + 2, nfull - 1), xa, pa);   // the last one re-reads a valid chunk: no branch
      __builtin_amdgcn_sched_barrier(0);
      mma(xc, pc);
    }
    const bool tail = nch > nfull;
    if (tail) load_tail(xc, pc);
    if (c < nfull) mma(xa, pa);
    if (tail) mma(xc, pc);
    if constexpr (SUM) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int o = 0; o < TO; ++o) {
          acct[i][o] += sc * accs[i][o];
          accs[i][o] = f4{0.f, 0.f, 0.f, 0.f};
        }
    }
  }
  __builtin_amdgcn_s_setprio(0);
  // one value: mode 1 adds the scaled cross products in one rounding, modes >= 2
  // round them first
  auto value = [&](int i, int o, int r) {
    if constexpr (M1) return acc[i][o][r] + sc * accs[i][o][r];
    else if constexpr (SUM) return acc[i][o][r] + acct[i][o][r];
    else return acc[i][o][r] + __builtin_fmaf(sc, accs[i][o][r], 0.f);
  };
  const int imax = n - 16 * t0;                               // i of the tile below it
  const int omax = (int)min(ext - q0, (int64_t)(16 * TO));    // columns of the tile
  const double* __restrict__ base = (const double*)jb.base;
  if constexpr (M1) {
    TOut* __restrict__ Y = (TOut*)jb.Y + origin + 16 * t0;
    const double* __restrict__ bs = base + origin + 16 * t0;
#pragma unroll
    for (int o = 0; o < TO; ++o) {
      if (16 * o + l >= omax) continue;
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const int i0 = 16 * i + 4 * g;
        const int64_t at = (int64_t)(16 * o + l) * n + i0;
        const f4 v = f4{value(i, o, 0), value(i, o, 1), value(i, o, 2), value(i, o, 3)};
        if constexpr (sizeof(TOut) == 4) {
          if (i0 + 4 <= imax) {
            *(f4u*)(Y + at) = v;
            continue;
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (i0 + r < imax) Y[at + r] = sizeof(TOut) == 8 && base ? (TOut)((double)v[r] + bs[at + r]) : (TOut)v[r];
      }
    }
  } else {
    TOut* __restrict__ Y = (TOut*)jb.Y + (origin - kBack) + na * 16 * t0;
    const double* __restrict__ bs = base + (origin - kBack) + na * 16 * t0;
    Off yo[NX];
#pragma unroll
    for (int o = 0; o < NX; ++o) yo[o] = column(V ? k0 : 16 * o + l) + (Off)kBack;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      // the base values of a block of rows are read together, from clamped
      // indices, so that they are one wait and not one each
      double bv[4][TO];
      if (sizeof(TOut) == 8 && base) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int o = 0; o < TO; ++o)
            bv[r][o] = bs[min(16 * i + 4 * g + r, imax - 1) * na + yo[V ? 0 : o] + (V ? o : 0)];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int o = 0; o < TO; ++o) bv[r][o] = -0.0;   // the sum is then the product itself
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + 4 * g + r;
        if (row >= imax) continue;
        TOut w[TO];
#pragma unroll
        for (int o = 0; o < TO; ++o) {
          const float v = value(i, o, r);
          w[o] = sizeof(TOut) == 8 ? (TOut)((double)v + bv[r][o]) : (TOut)v;
        }
        if constexpr (V) {
          typedef TOut tv __attribute__((ext_vector_type(TO), aligned(sizeof(TOut))));
          TOut* y = Y + row * na + yo[0];
          if (skip == 0) {
            tv x;
#pragma unroll
            for (int o = 0; o < TO; ++o) x[o] = w[o];
            *(tv*)y = x;
          } else {
#pragma unroll
            for (int o = 0; o < TO; ++o)
              if (o >= skip) y[o] = w[o];
          }
        } else {
#pragma unroll
          for (int o = 0; o < TO; ++o)
            if (16 * o + l < omax) Y[row * na + yo[o]] = w[o];
        }
      }
    }
  }
}

bool aligned_lp(const void* p, uintptr_t a) { return ((uintptr_t)p % a) == 0; }

// A tile's byte offsets span more than 32 bits.
bool big_tiles(const ModeJobs& J) {
  for (int j = 0; j < J.njobs; ++j) {
    const ModeJob& jb = J.job[j];
    if (jb.na > (int64_t(1) << 26) / 8 || (jb.nb > 1 && (ceil_div(64, jb.na) + 1) * jb.na * jb.n > (int64_t(1) << 28)))
      return true;
  }
  return false;
}

// Tiles of the FP32 kernel {blocks of i, of the other index}, and the part of
// the matrix-core rate that their loop reaches in mode 1 and in modes >= 2.
// Measured with 18 jobs: 128^3 modes >= 2 110 us with 4 x 4, 117 with 8 x 2, 140
// with 4 x 2 (8 tiles of i); 200^3 (13 tiles) mode 1 0.64 ms with 7 x 2, 0.68
// with 5 x 4, 0.76 with 4 x 4, modes >= 2 0.61, 0.73 and 0.72; 150^3 (10 tiles)
// modes >= 2 0.25 ms with 5 x 2, 0.29 with 5 x 4; 500 x 400, 6 jobs 38 us with
// 1 x 1, 96 with 4 x 4.  1 x 4 for modes >= 2 of one block of i, bound by memory: a
// whole operator on mode 2 of 1024 x 2 x 3200 61 us, 114 with 1 x 1.
struct TileF32 {
  int ti, to;
  double rate1, rateB;
};
constexpr TileF32 kTilesF32[] = {{1, 1, .50, .50}, {2, 2, .80, .80}, {4, 2, .85, .90}, {4, 4, .92, .98},
                                 {5, 2, .88, .88}, {5, 4, .95, .87}, {7, 2, .93, .92}, {8, 2, .92, .97},
                                 {1, 4, .50, .80}};

int64_t tile_count(const ModeJobs& J, bool mode1, const TileF32& t) {
  int64_t w = 0;
  for (int j = 0; j < J.njobs; ++j) {
    const ModeJob& jb = J.job[j];
    w += ceil_div(jb.n, 16 * t.ti) * ceil_div(mode1 ? jb.nb : jb.na * jb.nb, 16 * t.to);
  }
  return w;
}

// The tile whose launch should take least time, by the model of the FP64
// kernels (a chunk of 16 p is four MFMAs of 32 cycles per block); overridable
// with SETD_TILE_F32_MODE1 / SETD_TILE_F32_MODEB ("4x2" etc.).
TileF32 tile_f32(const ModeJobs& J, bool mode1) {
  const char* e = std::getenv(mode1 ? "SETD_TILE_F32_MODE1" : "SETD_TILE_F32_MODEB");
  int a = 0, b = 0;
  if (e && std::sscanf(e, "%dx%d", &a, &b) == 2)
    for (const TileF32& t : kTilesF32)
      if (t.ti == a && t.to == b) return t;
  bool wide = !mode1;   // 1 x 4: modes >= 2 of one block of i
  for (int j = 0; j < J.njobs; ++j) wide = wide && J.job[j].n <= 16;
  TileF32 best = kTilesF32[3];   // 4 x 4
  double bt = 1e300;
  for (const TileF32& t : kTilesF32) {
    if (t.ti == 1 && t.to == 4 && !wide) continue;
    const int64_t tiles = tile_count(J, mode1, t);
    if (!fits_grid(tiles, 1)) continue;
    const double w = (double)tiles / 1024.0;
    double wave = 0.0;
    for (int j = 0; j < J.njobs; ++j) {
      const ModeJob& jb = J.job[j];
      wave = std::max(wave, t.ti * t.to * ((double)jb.nterms * ceil_div(jb.n, 16) * 128.0 / (mode1 ? t.rate1 : t.rateB) +
                                           700.0 * (jb.base ? 1.6 : 1.0)));
    }
    const double time = ((w < 6.0 ? std::ceil(w) : w) + 0.3) * wave;
    if (time < bt) {
      bt = time;
      best = t;
    }
  }
  return best;
}

int finish_tiles_f32(ModeJobs& J, bool mode1, const TileF32& t) {
  J.total_tiles = assign_tiles_f64(J.job, J.njobs, mode1, t.ti, t.to);
  J.tiles_per_job = J.njobs > 0 ? J.total_tiles / J.njobs : 0;
  for (int j = 0; j < J.njobs; ++j)
    if (J.job[j].tile_begin != (int64_t)j * J.tiles_per_job) J.tiles_per_job = 0;
  return SETD_OK;
}

template <bool M1, bool V, int TI, int TO, typename Off, typename T>
int launch_tile_f32(const ModeJobs& J, hipStream_t s) {
  const int64_t per = ceil_div(ceil_div(J.total_tiles, 4), 8);
  hipLaunchKernelGGL((mode_f32_kernel<M1, V, TI, TO, Off, T>), dim3((unsigned)(per * 8)), dim3(256), 0, s, J, per);
  SETD_LAUNCHED();
  return SETD_OK;
}

template <bool M1, bool V, typename T>
int launch_f32(const ModeJobs& J, const TileF32& t, hipStream_t s) {
#define SETD_TILE(TI_, TO_) \
  if (t.ti == TI_ && t.to == TO_) return launch_tile_f32<M1, V && (TO_ > 1), TI_, TO_, uint32_t, T>(J, s);
  SETD_TILE(1, 1)
  SETD_TILE(1, 4)
  SETD_TILE(2, 2)
  SETD_TILE(4, 2)
  SETD_TILE(4, 4)
  SETD_TILE(5, 2)
  SETD_TILE(5, 4)
  SETD_TILE(7, 2)
  SETD_TILE(8, 2)
#undef SETD_TILE
  set_error("unsupported tile %dx%d", t.ti, t.to);
  return SETD_EUNSUPPORTED;
}

int launch_mode1_f32c(ModeJobs& J, DType out, hipStream_t s) {
  if (J.njobs == 0) return SETD_OK;
  double fl = 0.0, by = 0.0;
  if (prof_on()) job_work(J, 4, out == DType::F64 ? 8 : 4, 4, fl, by);
  const TileF32 cfg = tile_f32(J, true);
  bool lds = std::getenv("SETD_TILE_F32_MODE1") == nullptr;
  for (int j = 0; j < J.njobs; ++j) {
    const ModeJob& jb = J.job[j];
    lds = lds && jb.n >= kLds32MinN && jb.n <= kLds32MaxN && jb.n % 64 == 0 && jb.nb % 64 == 0 &&
          aligned_lp(jb.X[0], 16) && aligned_lp(jb.Y, 16) && aligned_lp(jb.base, 16);
  }
  if (lds) {   // workgroups: per job tiles_i panels x column groups of 8 * reps tiles
    const int reps = kLds32Reps;
    int64_t tot = 0;
    for (int j = 0; j < J.njobs; ++j) {
      ModeJob& jb = J.job[j];
      jb.tiles_i = jb.n / 64;
      jb.tiles_a = (int)(jb.nb / 64);
      jb.tile_begin = tot;
      tot += (int64_t)jb.tiles_i * ceil_div(jb.tiles_a, kLds32Waves * reps);
    }
    J.total_tiles = tot;
    J.tiles_per_job = J.njobs > 0 ? tot / J.njobs : 0;
    for (int j = 0; j < J.njobs; ++j)
      if (J.job[j].tile_begin != (int64_t)j * J.tiles_per_job) J.tiles_per_job = 0;
    if (tot == 0) return SETD_OK;
    ProfScope prof(s, kProfMode1LP, fl, by);
    const int64_t per = ceil_div(tot, 8);
    if (out == DType::F32)
      hipLaunchKernelGGL(mode1_lds32_kernel<float>, dim3((unsigned)(per * 8)), dim3(64 * kLds32Waves), 0, s, J, per,
                         reps);
    else
      hipLaunchKernelGGL(mode1_lds32_kernel<double>, dim3((unsigned)(per * 8)), dim3(64 * kLds32Waves), 0, s, J, per,
                         reps);
    SETD_LAUNCHED();
    return SETD_OK;
  }
  finish_tiles_f32(J, true, cfg);
  if (J.total_tiles == 0) return SETD_OK;
  ProfScope prof(s, kProfMode1LP, fl, by);
  return out == DType::F32 ? launch_f32<true, false, float>(J, cfg, s) : launch_f32<true, false, double>(J, cfg, s);
}

int launch_modeB_f32c(ModeJobs& J, DType out, hipStream_t s) {
  if (J.njobs == 0) return SETD_OK;
  double fl = 0.0, by = 0.0;
  if (prof_on()) job_work(J, 4, out == DType::F64 ? 8 : 4, 4, fl, by);
  const bool big = big_tiles(J);
  const TileF32 cfg = big ? kTilesF32[fits_grid(tile_count(J, false, kTilesF32[2]), 1) ? 2 : 3] : tile_f32(J, false);
  finish_tiles_f32(J, false, cfg);
  if (J.total_tiles == 0) return SETD_OK;
  ProfScope prof(s, kProfModeBLP, fl, by);
  if (big && cfg.to == 4)
    return out == DType::F32 ? launch_tile_f32<false, false, 4, 4, uint64_t, float>(J, s)
                             : launch_tile_f32<false, false, 4, 4, uint64_t, double>(J, s);
  if (big)
    return out == DType::F32 ? launch_tile_f32<false, false, 4, 2, uint64_t, float>(J, s)
                             : launch_tile_f32<false, false, 4, 2, uint64_t, double>(J, s);
  const bool vec = vector_columns(J, cfg.to);
  if (vec) return out == DType::F32 ? launch_f32<false, true, float>(J, cfg, s) : launch_f32<false, true, double>(J, cfg, s);
  return out == DType::F32 ? launch_f32<false, false, float>(J, cfg, s) : launch_f32<false, false, double>(J, cfg, s);
}

// Tiles of the bf16 kernel and the part of its rate that their loop reaches
// (the larger the tile, the less often a value is split and a piece read).
// Measured, three pieces, 18 jobs: 256^3 mode 1 1.17 ms with 4 x 4, 1.44 with
// 4 x 2, 1.67 with 2 x 2; 96 x 226 x 66 mode 1 78 us with 4 x 4 (6 tiles of i),
// 60 with 2 x 2; 128 x 82, 6 jobs 4.4 us with 1 x 1, 11 with 4 x 4.
constexpr TileF32 kTilesBf16[] = {{1, 1, .25, .25}, {2, 2, .60, .60}, {4, 2, .70, .70}, {4, 4, 1.0, 1.0}};

TileF32 tile_bf16(const ModeJobs& J, bool mode1, int np) {
  const char* e = std::getenv(mode1 ? "SETD_TILE_BF16_MODE1" : "SETD_TILE_BF16_MODEB");
  int a = 0, b = 0;
  if (e && std::sscanf(e, "%dx%d", &a, &b) == 2)
    for (const TileF32& t : kTilesBf16)
      if (t.ti == a && t.to == b) return t;
  TileF32 best = kTilesBf16[3];   // 4 x 4
  double bt = 1e300;
  for (const TileF32& t : kTilesBf16) {
    const int64_t tiles = tile_count(J, mode1, t);
    if (!fits_grid(tiles, 1)) continue;
    const double w = (double)tiles / 1024.0;
    double wave = 0.0;
    for (int j = 0; j < J.njobs; ++j) {
      const ModeJob& jb = J.job[j];
      wave = std::max(wave, t.ti * t.to * ((double)jb.nterms * ceil_div(jb.n, 32) * (np == 3 ? 112.0 : 64.0) / t.rate1 +
                                           700.0 * (jb.base ? 1.6 : 1.0)));
    }
    const double time = ((w < 6.0 ? std::ceil(w) : w) + 0.3) * wave;
    if (time < bt) {
      bt = time;
      best = t;
    }
  }
  return best;
}

template <int NP, bool M1, bool V, bool SUM, int TI, int TO, typename Off, typename T>
int launch_tile_bf16(const ModeJobs& J, hipStream_t s) {
  const int64_t per = ceil_div(ceil_div(J.total_tiles, 4), 8);
  hipLaunchKernelGGL((mode_bf16_kernel<NP, M1, V, SUM, TI, TO, Off, T>), dim3((unsigned)(per * 8)), dim3(256), 0, s, J,
                     per);
  SETD_LAUNCHED();
  return SETD_OK;
}

template <int NP, bool M1, bool V, bool SUM, typename T>
int launch_bf16(const ModeJobs& J, const TileF32& t, hipStream_t s) {
#define SETD_TILE(TI_, TO_) \
  if (t.ti == TI_ && t.to == TO_) return launch_tile_bf16<NP, M1, V && (TO_ > 1), SUM, TI_, TO_, uint32_t, T>(J, s);
  SETD_TILE(1, 1)
  SETD_TILE(2, 2)
  SETD_TILE(4, 2)
  SETD_TILE(4, 4)
#undef SETD_TILE
  set_error("unsupported tile %dx%d", t.ti, t.to);
  return SETD_EUNSUPPORTED;
}

template <int NP, typename T>
int launch_modeB_bf16(const ModeJobs& J, const TileF32& t, bool big, bool vec, bool sum, hipStream_t s) {
  if (big && t.to == 4) return launch_tile_bf16<NP, false, false, true, 4, 4, uint64_t, T>(J, s);
  if (big) return launch_tile_bf16<NP, false, false, true, 4, 2, uint64_t, T>(J, s);
  if (vec) return sum ? launch_bf16<NP, false, true, true, T>(J, t, s) : launch_bf16<NP, false, true, false, T>(J, t, s);
  return sum ? launch_bf16<NP, false, false, true, T>(J, t, s) : launch_bf16<NP, false, false, false, T>(J, t, s);
}

}  // namespace

int launch_mode1_lp(ModeJobs& J, int prec, DType out, hipStream_t s) {
  if (prec == SETD_PREC_F32) return launch_mode1_f32c(J, out, s);
  if (J.njobs == 0) return SETD_OK;
  const bool x3 = prec == SETD_PREC_BF16X3;
  const TileF32 cfg = tile_bf16(J, true, x3 ? 3 : 2);
  finish_tiles_f32(J, true, cfg);
  if (J.total_tiles == 0) return SETD_OK;
  double fl = 0.0, by = 0.0;
  if (prof_on()) job_work(J, 4, out == DType::F64 ? 8 : 4, 4, fl, by);
  ProfScope prof(s, kProfMode1LP, fl, by);
  if (x3)
    return out == DType::F32 ? launch_bf16<3, true, false, false, float>(J, cfg, s)
                             : launch_bf16<3, true, false, false, double>(J, cfg, s);
  return out == DType::F32 ? launch_bf16<2, true, false, false, float>(J, cfg, s)
                           : launch_bf16<2, true, false, false, double>(J, cfg, s);
}

int launch_modeB_lp(ModeJobs& J, int prec, DType out, hipStream_t s) {
  if (prec == SETD_PREC_F32) return launch_modeB_f32c(J, out, s);
  if (J.njobs == 0) return SETD_OK;
  const bool x3 = prec == SETD_PREC_BF16X3, big = big_tiles(J);
  const TileF32 cfg =
      big ? kTilesBf16[fits_grid(tile_count(J, false, kTilesBf16[2]), 1) ? 2 : 3] : tile_bf16(J, false, x3 ? 3 : 2);
  finish_tiles_f32(J, false, cfg);
  if (J.total_tiles == 0) return SETD_OK;
  double fl = 0.0, by = 0.0;
  if (prof_on()) job_work(J, 4, out == DType::F64 ? 8 : 4, 4, fl, by);
  ProfScope prof(s, kProfModeBLP, fl, by);
  bool sum = false;
  for (int j = 0; j < J.njobs; ++j) sum = sum || J.job[j].nterms > 1;
  const bool vec = vector_columns(J, cfg.to);
  if (x3)
    return out == DType::F32 ? launch_modeB_bf16<3, float>(J, cfg, big, vec, sum, s)
                             : launch_modeB_bf16<3, double>(J, cfg, big, vec, sum, s);
  return out == DType::F32 ? launch_modeB_bf16<2, float>(J, cfg, big, vec, sum, s)
                           : launch_modeB_bf16<2, double>(J, cfg, big, vec, sum, s);
}

}  // namespace setd
