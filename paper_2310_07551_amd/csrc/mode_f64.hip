// FP64 mu-mode products on the CDNA4 matrix cores (v_mfma_f64_16x16x4_f64).
//
// A mu-mode product S = T x_mu L (Section 2) applies L to every mu-fiber:
// with a = (i_1..i_{mu-1}) flattened (stride 1), i = i_mu and b =
// (i_{mu+1}..i_d) flattened,
//
//     Y[a, i, b] = sum_p L[i, p] X[a, p, b].
//
// Operand layout.  The matrix is packed in the order the matrix cores read
// it: entry (tile t, chunk c, lane, j) = L[16 t + lane % 16][8 c + 2 (lane / 16)
// + j], j in {0, 1}, zero past n.  One 16-byte load per lane (1 KB contiguous
// per wave) is the operand of two k-steps, whichever side of the product the
// matrix is on, so mode 1 and the other modes share one layout.  The tensor
// is read in place, with the same assignment of p to k-steps:
//   * mode 1 (no a index): Y = L X as a GEMM over the column-major unfolding
//     X_(1) (n x N/n), no copy.  MFMA rows = b, columns = i: a lane loads two
//     consecutive p of its column of X, and the 16 lanes of a group hold 16
//     consecutive i of the result.
//   * modes >= 2: for each b, Y[:, :, b] = X[:, :, b] L^T with a contiguous.
//     MFMA rows = i, columns = a: 16 lanes load 128 contiguous bytes of a row
//     of X, and store 128 contiguous bytes of the result.
// Either way no load or store needs more than 8-byte alignment, so odd sizes
// run the same code as round ones: indices past an edge are clamped (their
// results are not stored), and the last n % 8 contraction indices are taken
// first, as one masked chunk.
//
// Each wave owns TI x TO accumulators (16 TI of i, 16 TO of the other index)
// and keeps a ring of D chunks of operands in registers, each loaded D - 1
// chunks of products before its use.  With KS > 1 the waves of a workgroup
// share a tile, each a part of the contraction, and add their accumulators
// through LDS in a fixed order.
//
// Each launch runs a table of independent jobs (up to kMaxJobs outputs; each
// may sum up to kMaxTerms inputs along the contraction, which is how the
// terms of a split phi action are accumulated into one output), four waves
// per workgroup on neighbouring tiles, with the block index remapped so that
// each XCD gets a contiguous range of tiles (neighbouring tiles share X or L
// in that XCD's L2).
//
// What bounds them: the matrix cores (64 cycles per MFMA and SIMD) from n =
// 192 on; below that also the tensor traffic (n / 8 flops per byte), and on
// small grids the latency of one wave (about 2 us besides its products), so
// that the tile is chosen per launch (choose_tile).  Steps of two components
// against kernels with one fixed tile per contraction length and vector
// accesses for aligned sizes only: 300^2 595 -> 109 us (the last mode alone
// 151 -> 20 and 9 us), and with the one-pass kernels below 64^2 107 -> 36 us,
// 100^3 739 -> 538 us, 128^3 1060 -> 884 us, 256^3 11.93 -> 11.72 ms.
#include "common.hpp"
#include "pointwise.hpp"

#include <algorithm>
#include <cstdlib>

namespace setd {

__device__ __forceinline__ int64_t remap_xcd(int64_t bid, int64_t per_xcd) {
  return (bid & 7) * per_xcd + (bid >> 3);
}

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));   // a pair at any 8-byte address

// Packed FP64 matrix: tile t starts at t * chunks(n) * 128 doubles.
__device__ __forceinline__ int chunks_of(int n) { return (n + 7) >> 3; }
__device__ __forceinline__ double packed_at(const double* P, int n, int i, int p) {
  return P[((int64_t)(i >> 4) * chunks_of(n) + (p >> 3)) * 128 + ((((p >> 1) & 3) << 4) + (i & 15)) * 2 + (p & 1)];
}

// The matrix operand of TI tiles from tile t0: packed, or (RAW) read as it is
// given, column-major n x n, for a matrix that is used once: 16 lanes read 128
// contiguous bytes of a column.  Tiles and rows past the last are clamped.
template <bool RAW, int TI>
struct MatrixTiles {
  const double* at[TI];   // packed: the lane's pair of the tile's first chunk
  uint32_t off[TI];       // RAW: byte offset of the lane's entry in columns 0, 8, ..
  const double* M;
  int n, g;

  __device__ __forceinline__ MatrixTiles(const void* P, int n_, int t0, int lane) : M((const double*)P), n(n_), g(lane >> 4) {
    const int nt = (n + 15) >> 4, nch = chunks_of(n);
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      if constexpr (RAW) off[i] = (uint32_t)((min(16 * (t0 + i) + (lane & 15), n - 1) + (int64_t)n * (2 * g)) * 8);
      else at[i] = M + (int64_t)min(t0 + i, nt - 1) * nch * 128 + 2 * lane;
    }
  }
  // chunk c: entries of p = 8 c + 2 g + j; RAW: c < n / 8
  __device__ __forceinline__ void load(int c, d2 (&p)[TI]) const {
    if constexpr (RAW) {
      const char* c0 = (const char*)(M + (int64_t)n * (8 * c));
      const char* c1 = (const char*)(M + (int64_t)n * (8 * c + 1));
#pragma unroll
      for (int i = 0; i < TI; ++i) p[i] = d2{*(const double*)(c0 + off[i]), *(const double*)(c1 + off[i])};
    } else {
#pragma unroll
      for (int i = 0; i < TI; ++i) p[i] = *(const d2*)(at[i] + (int64_t)c * 128);
    }
  }
  // the last chunk, of n % 8: zero past n
  __device__ __forceinline__ void load_tail(d2 (&p)[TI]) const {
    if constexpr (RAW) {
      const int c = n >> 3;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int q = 8 * c + 2 * g + j;
        const char* cq = (const char*)(M + (int64_t)n * (min(q, n - 1) - 2 * g));
#pragma unroll
        for (int i = 0; i < TI; ++i) p[i][j] = *(const double*)(cq + off[i]);
#pragma unroll
        for (int i = 0; i < TI; ++i) p[i][j] = q < n ? p[i][j] : 0.0;
      }
    } else {
      load(n >> 3, p);
    }
  }
};

// Adds sum_p S[i, p] X[.., p, ..] of one term to the accumulators, for p of
// the chunks lo .. hi - 1.  x0 is the tile's first element, xo[o] the byte
// offset of the lane's first element of column (row) block o from it; M1:
// consecutive p are adjacent, else `na` elements apart.
template <bool M1, bool RAW, int TI, int TO, int D, typename Off, bool V = false>
__device__ __forceinline__ void add_term(d4 (&acc)[TI][TO], const double* __restrict__ x0,
                                         const Off (&xo)[V ? 1 : TO],
                                         int64_t na, const MatrixTiles<RAW, TI>& mat, int n, int lane, int lo,
                                         int hi) {
  const int g = lane >> 4;
  const int nfull = n >> 3;
  auto load = [&](int c, d2 (&xr)[TO], d2 (&pr)[TI]) {
    mat.load(c, pr);
    if constexpr (M1) {
      const char* xb = (const char*)(x0 + 8 * c);
#pragma unroll
      for (int o = 0; o < TO; ++o) xr[o] = *(const d2u*)(xb + xo[o]);
    } else {
      const char* xb0 = (const char*)(x0 + na * (8 * (int64_t)c));
      const char* xb1 = (const char*)(x0 + na * (8 * (int64_t)c + 1));
      if constexpr (V) {
        typedef double dv __attribute__((ext_vector_type(TO), aligned(8)));
        const dv v0 = *(const dv*)(xb0 + xo[0]), v1 = *(const dv*)(xb1 + xo[0]);
#pragma unroll
        for (int o = 0; o < TO; ++o) xr[o] = d2{v0[o], v1[o]};
      } else {
#pragma unroll
        for (int o = 0; o < TO; ++o) xr[o][0] = *(const double*)(xb0 + xo[o]);
#pragma unroll
        for (int o = 0; o < TO; ++o) xr[o][1] = *(const double*)(xb1 + xo[o]);
      }
    }
  };
  auto mma = [&](const d2 (&xr)[TO], const d2 (&pr)[TI]) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int o = 0; o < TO; ++o)
          acc[i][o] = M1 ? mfma(xr[o][j], pr[i][j], acc[i][o]) : mfma(pr[i][j], xr[o][j], acc[i][o]);
  };
  const int c0 = lo, c1 = min(hi, nfull);
  const bool tail = hi > nfull;   // the last chunk, of n % 8
  d2 xr[D][TO], pr[D][TI];
  if (tail) {
    // the last n % 8 values of p: clamped loads, zero past n
    mat.load_tail(pr[D - 1]);
    const int64_t ps = M1 ? 1 : na;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int p = 8 * nfull + 2 * g + j;
      const char* xp = (const char*)(x0 + ps * (min(p, n - 1) - 2 * g));   // xo holds the lane's 2 g
      if constexpr (V) {
        typedef double dv __attribute__((ext_vector_type(TO), aligned(8)));
        const dv v = *(const dv*)(xp + xo[0]);
#pragma unroll
        for (int o = 0; o < TO; ++o) xr[D - 1][o][j] = v[o];
      } else {
#pragma unroll
        for (int o = 0; o < TO; ++o) xr[D - 1][o][j] = *(const double*)(xp + xo[o]);
      }
#pragma unroll
      for (int o = 0; o < TO; ++o) xr[D - 1][o][j] = p < n ? xr[D - 1][o][j] : 0.0;
    }
  }
  if (c0 < c1) {
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(min(c0 + d, c1 - 1), xr[d], pr[d]);
  }
  if (tail) mma(xr[D - 1], pr[D - 1]);
  if (c0 >= c1) return;
  load(min(c0 + D - 1, c1 - 1), xr[D - 1], pr[D - 1]);
  int c = c0;
  for (; c + D <= c1; c += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      mma(xr[d], pr[d]);
      load(min(c + d + D, c1 - 1), xr[d], pr[d]);   // the last ones re-read a valid chunk: no branch
    }
  }
#pragma unroll
  for (int d = 0; d < D - 1; ++d)
    if (c + d < c1) mma(xr[d], pr[d]);
}

// One wave computes tile `lt` of job `jb` (part kw of ks of its contraction;
// `red` is the LDS the waves of one tile add up in when ks > 1).
template <bool M1, bool RAW, int TI, int TO, int D, int KS, typename Off, bool V = false>
__device__ __forceinline__ void mode_tile(const ModeJob& jb, uint32_t lt, int lane, int kw, d4* red) {
  const int g = lane >> 4, l = lane & 15;
  const int n = jb.n;
  const uint32_t ti = (uint32_t)jb.tiles_i;
  const uint32_t ot = lt / ti;
  const int t0 = (int)(lt - ot * ti) * TI;
  // The other tiled index: b in mode 1; else a and b together, q = a + na b,
  // so that only the last tile is ragged whatever na is.
  const int64_t na = M1 ? 1 : jb.na;
  const int64_t ext = M1 ? jb.nb : na * jb.nb;
  const int64_t q0 = (int64_t)ot * (16 * TO);
  const uint32_t una = (uint32_t)na;
  const uint32_t b0 = M1 ? 0 : jb.nb == 1 ? 0 : (uint32_t)((uint64_t)q0 / una);
  const int64_t r0 = q0 - (int64_t)b0 * na;   // a of the tile's first column
  const int64_t origin_x = M1 ? q0 * n : (int64_t)b0 * na * n + r0;
  // element offset of the lane's column in block o of the tile (clamped to
  // the extent) from the tile's first
  auto column = [&](int k) -> Off {
    const int64_t rel = min(q0 + k, ext - 1) - q0;
    if (M1) return (Off)(rel * n);
    if (jb.nb == 1) return (Off)rel;
    const Off q = (Off)(r0 + rel);
    const Off bb = q / (Off)na;
    return (Off)(bb * (Off)(na * n) + (q - bb * (Off)na) - (Off)r0);
  };
  // columns of the lane: 16 o + l, or with V the TO consecutive ones from TO l
  // on (the last lanes move back to end with the last column; they keep the
  // first `skip` of theirs to themselves).  The moved lanes of a tile with
  // fewer than TO columns begin before it: with V offsets count from TO
  // elements before the tile's first.
  constexpr int NX = V ? 1 : TO, kBack = V ? TO : 0;
  const int k0 = V ? (int)(min(q0 + TO * l, ext - TO) - q0) : 0, skip = TO * l - k0;
  Off xo[NX];
#pragma unroll
  for (int o = 0; o < NX; ++o)
    xo[o] = (column(V ? k0 : 16 * o + l) + (Off)kBack + (M1 ? (Off)(2 * g) : (Off)na * (Off)(2 * g))) * 8;
  d4 acc[TI][TO];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int o = 0; o < TO; ++o) acc[i][o] = d4{0.0, 0.0, 0.0, 0.0};
  __builtin_amdgcn_s_setprio(1);   // products ahead of another wave's epilogue on the SIMD
  // the chunks of all terms in a row, in KS equal parts
  const int nterms = M1 ? 1 : jb.nterms, nch = chunks_of(n);
  const int first = KS > 1 ? nterms * nch * kw / KS : 0, last = KS > 1 ? nterms * nch * (kw + 1) / KS : nterms * nch;
  for (int term = 0; term < nterms; ++term) {
    if (term > 0 && jb.scale[term] != jb.scale[term - 1]) {   // the sum is kept in units of the term's scale
      const double ratio = jb.scale[term - 1] / jb.scale[term];
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int o = 0; o < TO; ++o) acc[i][o] *= ratio;
    }
    const int lo = max(first - term * nch, 0), hi = min(last - term * nch, nch);
    if (lo < hi)
      add_term<M1, RAW, TI, TO, D, Off, V>(acc, (const double*)jb.X[term] + (origin_x - kBack), xo, na,
                                        MatrixTiles<RAW, TI>(jb.P[term], n, t0, lane), n, lane, lo, hi);
  }
  const double sc = jb.scale[nterms - 1];
  __builtin_amdgcn_s_setprio(0);
  // Epilogue.  The FP64 16x16 accumulator holds tile row 4 r + g in register
  // r of lane (g, l), column l: mode 1, row b and column i; else row i and
  // column a.  16 lanes write 128 contiguous bytes.  The base values of a
  // block of rows are read together, from clamped indices, so that they are
  // one wait and not one each.
  constexpr int TR = M1 ? TO : TI, TC = M1 ? TI : TO;
  const int64_t origin = M1 ? q0 * n + 16 * t0 : origin_x + na * 16 * t0;
  const int imax = n - 16 * t0;                                     // i of the tile below it
  const int omax = (int)min(ext - q0, (int64_t)(16 * TO));          // columns of the tile
  double* __restrict__ Y = (double*)jb.Y + origin;
  const double* __restrict__ bs = (const double*)jb.base + origin;
  const bool has_base = jb.base != nullptr;
  const int64_t ld = M1 ? n : na;
  if constexpr (V) {
    typedef double dv __attribute__((ext_vector_type(TO), aligned(8)));
    const Off y0 = column(k0) + (Off)kBack;
#pragma unroll
    for (int m = 0; m < TI; ++m) {
      dv bv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (has_base) bv[r] = *(const dv*)(bs - kBack + min(16 * m + 4 * r + g, imax - 1) * ld + y0);
        else bv[r] = dv(-0.0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * m + 4 * r + g;
        if (row >= imax) continue;
        dv v;
#pragma unroll
        for (int u = 0; u < TO; ++u) v[u] = acc[m][u][r] * sc + bv[r][u];
        double* y = Y - kBack + row * ld + y0;
        if (skip == 0) {
          *(dv*)y = v;
        } else {
#pragma unroll
          for (int u = 0; u < TO; ++u)
            if (u >= skip) y[u] = v[u];
        }
      }
    }
    return;
  }
  Off yo[TC];   // column of each block
#pragma unroll
  for (int u = 0; u < TC; ++u) yo[u] = M1 ? (Off)min(16 * u + l, imax - 1) : column(16 * u + l);
  if constexpr (KS > 1) {
    // the parts meet in LDS; each wave adds up and stores its share of the blocks
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int o = 0; o < TO; ++o) red[(kw * TI * TO + (M1 ? o * TI + i : i * TO + o)) * 64 + lane] = acc[i][o];
    __syncthreads();
#pragma unroll 1
    for (int k = kw; k < TR * TC; k += KS) {
      const int m = k / TC, u = k % TC;
      const Off y = M1 ? (Off)min(16 * u + l, imax - 1) : column(16 * u + l);
      double bv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        bv[r] = has_base ? bs[min(16 * m + 4 * r + g, (M1 ? omax : imax) - 1) * ld + y] : -0.0;
      d4 v = red[k * 64 + lane];
#pragma unroll
      for (int w = 1; w < KS; ++w) v += red[(w * TI * TO + k) * 64 + lane];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * m + 4 * r + g;
        if (row < (M1 ? omax : imax) && 16 * u + l < (M1 ? imax : omax)) Y[row * ld + y] = v[r] * sc + bv[r];
      }
    }
    return;
  }
#pragma unroll
  for (int m = 0; m < TR; ++m) {
    double bv[4][TC];
    if (has_base) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < TC; ++u) bv[r][u] = bs[min(16 * m + 4 * r + g, (M1 ? omax : imax) - 1) * ld + yo[u]];
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < TC; ++u) bv[r][u] = -0.0;   // the sum is then the product itself
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * m + 4 * r + g;
#pragma unroll
      for (int u = 0; u < TC; ++u)
        if (row < (M1 ? omax : imax) && 16 * u + l < (M1 ? imax : omax))
          Y[row * ld + yo[u]] = (M1 ? acc[u][m][r] : acc[m][u][r]) * sc + bv[r][u];
    }
  }
}

// Ring depth: more chunks in flight where a chunk is only a few products; 1 x 4
// tiles have two chunks at most and hide their latency with waves.
constexpr int ring_depth(int ti, int to) {
  return ti == 1 && to == 4 ? 1 : ti * to <= 2 ? 4 : ti * to <= 4 ? 3 : 2;
}
// LDS of a workgroup whose waves split contractions: 4 / KS tiles, KS parts each.
constexpr int red_size(int ti, int to, int ks) { return ks > 1 ? 4 * ti * to * 64 : 1; }

// Job table in the kernel arguments (up to kMaxJobs outputs per launch).
// Two waves per SIMD is the target occupancy of the larger tiles: with that
// register budget the accumulators stay in place through the k loop (a
// tighter default made the compiler copy all of them between register files
// every iteration).
template <bool M1, bool RAW, int TI, int TO, int KS, typename Off, bool V>
__global__ void __launch_bounds__(256, 2) mode_f64_kernel(const ModeJobs J, int64_t per_xcd) {
  __shared__ d4 red[red_size(TI, TO, KS)];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t t = (uint32_t)remap_xcd(blockIdx.x, per_xcd) * (4 / KS) + wave / KS;
  if (t >= (uint32_t)J.total_tiles) {
    if constexpr (KS > 1) __syncthreads();   // the barrier of the waves with a tile
    return;
  }
  const ModeJob& jb = J.job[find_job(J, t)];
  mode_tile<M1, RAW, TI, TO, ring_depth(TI, TO), KS, Off, V>(jb, t - (uint32_t)jb.tile_begin, lane, wave % KS,
                                                          red + (wave / KS) * KS * TI * TO * 64);
}

// Work list in device memory (any number of jobs, e.g. many independent
// instances), walked by a persistent grid of 4-wave workgroups.  The tiles of
// a list differ in length (they are sorted longest first), so an XCD takes
// runs of kListRun workgroups in turn rather than one contiguous range.
constexpr int kListRun = 8;
template <bool M1, int TI, int TO, int KS>
__global__ void __launch_bounds__(256, 2) mode_f64_list_kernel(const ModeJob* __restrict__ jobs,
                                                               const int64_t* __restrict__ begins, int njobs,
                                                               int64_t total, int64_t ngroups) {
  __shared__ d4 red[red_size(TI, TO, KS)];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  for (int64_t raw = blockIdx.x; raw < ngroups; raw += gridDim.x) {
    const int64_t run = raw / (8 * kListRun), in = raw % (8 * kListRun);
    const int64_t t = (run * 8 * kListRun + (in & 7) * kListRun + (in >> 3)) * (4 / KS) + wave / KS;
    if (t < total) {
      const int j = find_job_list(begins, njobs, t);
      mode_tile<M1, false, TI, TO, ring_depth(TI, TO), KS, uint32_t>(jobs[j], (uint32_t)(t - begins[j]), lane, wave % KS,
                                                                     red + (wave / KS) * KS * TI * TO * 64);
    } else if (KS > 1) {
      __syncthreads();   // the barrier of the waves with a tile
    }
    if constexpr (KS > 1) __syncthreads();   // the parts have been read
  }
}

// ---------------------------------------------------------------------------
// modes 1 and 2 in one pass
// ---------------------------------------------------------------------------
// Y_b = base_b + sum_t s_t P1_t X_t,b P2_t^T for every slab b (n1 x n2, i_1
// fastest): the mode-1 and the mode-2 product of a Tucker operator without
// the intermediate tensor.  A workgroup of 4 waves owns one slab and up to
// 16 TJ columns j of its result.  Phase 1 forms Z = X_b P2^T for those
// columns (a modes >= 2 product over the whole mode-2 fibres), each wave the
// blocks of 16 i_1 w, w + 4, ..; Z goes to LDS (with the term's scale), where
// phase 2 reads it as the tensor operand of the mode-1 product.  Both
// contractions run over all of Z, so nothing is computed twice; X_b is
// re-read once per column block, from L2.
// Bound by the matrix cores once two or more workgroups share a CU (128^3:
// busy 77% with 18 jobs, 71% with 6).  It saves
// the traffic of the intermediate, which is what the two products were bound
// by for n < 200 (n / 8 flops per byte), and one launch.
// Waves whose share of i_1 blocks or columns is one smaller run their own
// instance of the body (NI - 1, TJ - 1), and the smaller share moves round
// the SIMDs from one workgroup to the next.
constexpr int slab_ring(int tj, int ni) { return tj * ni >= 6 ? 2 : 3; }

// X: the slab, in LDS, of a stage difference; nullptr: the term's tensor.
template <bool RAW, bool SUM, int TJ, int NI, int LD, bool DIFF = false>
__device__ __forceinline__ void slab_body(const SlabJob& jb, uint32_t b, int tj0, int w, int term, int lane,
                                          double* Zall, const double* X = nullptr) {
  const int g = lane >> 4, l = lane & 15;
  const int n1 = jb.n1, n2 = jb.n2, nch1 = chunks_of(n1);
  const int64_t slab = (int64_t)n1 * n2 * b;
  double* Z = Zall + term * (16 * TJ * LD);
  {
    uint32_t xo[NI];
#pragma unroll
    for (int o = 0; o < NI; ++o) xo[o] = (uint32_t)((min(16 * (w + 4 * o) + l, n1 - 1) + n1 * (2 * g)) * 8);
    d4 z[TJ][NI];
#pragma unroll
    for (int m = 0; m < TJ; ++m)
#pragma unroll
      for (int o = 0; o < NI; ++o) z[m][o] = d4{0.0, 0.0, 0.0, 0.0};
    add_term<false, RAW, TJ, NI, slab_ring(TJ, NI), uint32_t>(
        z, DIFF ? X : (const double*)jb.X[term] + slab, xo, n1, MatrixTiles<RAW, TJ>(jb.P2[term], n2, tj0, lane), n2, lane, 0,
        chunks_of(n2));
    const double sc = jb.scale[term];
#pragma unroll
    for (int m = 0; m < TJ; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int o = 0; o < NI; ++o) {
          const int a = 16 * (w + 4 * o) + l;
          Z[(16 * m + 4 * r + g) * LD + a] = a < n1 ? z[m][o][r] * sc : 0.0;
        }
  }
  // phase 2: the wave's tiles w, w + 4, .. of P1, one MatrixTiles each
  const MatrixTiles<RAW, 1> mat0(jb.P1[term], n1, w, lane);
  const uint32_t step = 4u * nch1 * 128 * 8;   // packed: bytes from one of them to the next
  auto load = [&](int c, d2 (&p)[NI]) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if constexpr (RAW) {
        d2 q[1];
        const MatrixTiles<true, 1> mi(jb.P1[term], n1, w + 4 * i, lane);
        if (c < (n1 >> 3)) mi.load(c, q);
        else mi.load_tail(q);
        p[i] = q[0];
      } else {
        p[i] = *(const d2*)((const char*)(mat0.at[0] + (int64_t)c * 128) + (uint32_t)i * step);
      }
    }
  };
  d4 acc[NI][TJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int m = 0; m < TJ; ++m) acc[i][m] = d4{0.0, 0.0, 0.0, 0.0};
  constexpr int D2 = 2;
  d2 p[D2][NI];
#pragma unroll
  for (int d = 0; d < D2; ++d) load(min(d, nch1 - 1), p[d]);   // in flight over the barrier
  __syncthreads();
  const double* zr = Z + l * LD + 2 * g;
  auto mma = [&](int c, const d2 (&pr)[NI]) {
    d2 zz[TJ];
#pragma unroll
    for (int m = 0; m < TJ; ++m) zz[m] = *(const d2*)(zr + 16 * m * LD + 8 * c);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int m = 0; m < TJ; ++m) acc[i][m] = mfma(zz[m][j], pr[i][j], acc[i][m]);
  };
  int c = 0;
  for (; c + D2 <= nch1; c += D2) {
#pragma unroll
    for (int d = 0; d < D2; ++d) {
      mma(c + d, p[d]);
      load(min(c + d + D2, nch1 - 1), p[d]);
    }
  }
#pragma unroll
  for (int d = 0; d < D2 - 1; ++d)
    if (c + d < nch1) mma(c + d, p[d]);
  if constexpr (SUM) {
    // the waves of the first term add up the others', handed over in their Z
    constexpr int share = (LD - 2) / 64 * TJ;   // accumulators of the wave with the most blocks
    __syncthreads();
    d4* red = (d4*)Z + w * share * 64 + lane;
    if (term > 0) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int m = 0; m < TJ; ++m) red[(i * TJ + m) * 64] = acc[i][m];
    }
    __syncthreads();
    if (term > 0) return;
    for (int t = 1; t < jb.nterms; ++t) {
      red = (d4*)(Zall + t * (16 * TJ * LD)) + w * share * 64 + lane;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int m = 0; m < TJ; ++m) acc[i][m] += red[(i * TJ + m) * 64];
    }
  }
  double* __restrict__ Y = (double*)jb.Y + slab;
  const bool has_base = jb.base != nullptr;
  const double* __restrict__ bs = (const double*)jb.base + slab;
#pragma unroll
  for (int m = 0; m < TJ; ++m) {
    double bv[4][NI];
    if (has_base) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < NI; ++i)
          bv[r][i] = bs[min(16 * (tj0 + m) + 4 * r + g, n2 - 1) * n1 + min(16 * (w + 4 * i) + l, n1 - 1)];
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < NI; ++i) bv[r][i] = -0.0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = 16 * (tj0 + m) + 4 * r + g;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int a = 16 * (w + 4 * i) + l;
        if (j < n2 && a < n1) Y[j * n1 + a] = acc[i][m][r] + bv[r][i];
      }
    }
  }
}

// SUM: jobs of kSlabTerms terms, each term on four waves of its own; else one.
constexpr int kSlabTerms = 2;
template <bool RAW, bool SUM, int TJ, int NI>
__global__ void __launch_bounds__(SUM ? 256 * kSlabTerms : 256, 2) slab_f64_kernel(const SlabJobs J, int64_t per_xcd) {
  // rows of Z two doubles apart from a multiple of 64: the 16 lanes of a
  // phase-2 read start 16 bytes apart in the banks
  constexpr int LD = 64 * NI + 2;
  __shared__ double Z[(SUM ? kSlabTerms : 1) * 16 * TJ * LD];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t t = (uint32_t)remap_xcd(blockIdx.x, per_xcd);
  if (t >= (uint32_t)J.total) return;   // uniform over the workgroup
  const uint32_t jj = t / (uint32_t)J.tiles_per_job;
  const SlabJob& jb = J.job[jj];
  const uint32_t lt = t - jj * (uint32_t)J.tiles_per_job;
  const uint32_t b = lt / (uint32_t)J.nblk;
  const int blk = (int)(lt - b * (uint32_t)J.nblk);
  const int nt1 = (jb.n1 + 15) >> 4, nt2 = (jb.n2 + 15) >> 4;
  // column blocks: nt2 / nblk tiles each, the first nt2 % nblk one more
  const int q = nt2 / J.nblk, rem = nt2 % J.nblk;
  const int tj0 = blk * q + min(blk, rem), tj = q + (blk < rem);
  const int w = ((wave & 3) + (int)(lt & 3)) & 3, term = SUM ? wave >> 2 : 0;
  const int ni = (nt1 - w + 3) >> 2;   // tiles w, w + 4, .. below nt1
  if (ni == 0) {   // a wave without i_1 blocks only keeps the barriers
    for (int k = 0; k < (SUM ? 3 : 1); ++k) __syncthreads();
    return;
  }
  if (tj == TJ) {
    if (ni == NI) slab_body<RAW, SUM, TJ, NI, LD>(jb, b, tj0, w, term, lane, Z);
    else if constexpr (NI > 1) slab_body<RAW, SUM, TJ, NI - 1, LD>(jb, b, tj0, w, term, lane, Z);
  } else if constexpr (TJ > 1) {
    if (ni == NI) slab_body<RAW, SUM, TJ - 1, NI, LD>(jb, b, tj0, w, term, lane, Z);
    else if constexpr (NI > 1) slab_body<RAW, SUM, TJ - 1, NI - 1, LD>(jb, b, tj0, w, term, lane, Z);
  }
}

// The two-term pass over one slab of up to kSlabSumN x kSlabSumN whose tensor
// is a component of a stage difference, or (FIRST) of F = K u + g(u): every
// workgroup forms all of it in LDS (it reads all of it anyway), which saves the
// kernels that formed them before: three of the six of a 64^2 step, 43.0 -> 36.2
// us.  FIRST: the stencil reads u from LDS, its sums in the order of
// gf_stencil_kernel; the first column block of the component's first job writes
// G.  Bound by latency (cold first loads, the barriers between the phases).
template <bool FIRST>
__global__ void __launch_bounds__(256 * kSlabTerms, 2) slab_diff_f64_kernel(const SlabJobs J, const StageDiff sd,
                                                                            int64_t per_xcd) {
  constexpr int LD = 66, kThreads = 256 * kSlabTerms, kPer = kSlabSumN * kSlabSumN / kThreads;
  __shared__ double Z[kSlabTerms * 16 * LD];
  __shared__ double X[kSlabSumN * kSlabSumN];
  __shared__ double U[FIRST ? kSlabSumN * kSlabSumN : 1];
  __shared__ double K[FIRST ? 6 * kSlabSumN : 1];   // lo, di, up of both directions
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t t = (uint32_t)remap_xcd(blockIdx.x, per_xcd);
  if (t >= (uint32_t)J.total) return;   // uniform over the workgroup
  const uint32_t jj = t / (uint32_t)J.tiles_per_job;
  const SlabJob& jb = J.job[jj];
  const uint32_t lt = t - jj * (uint32_t)J.tiles_per_job;   // its column block: one slab
  const int n1 = jb.n1, n2 = jb.n2, nn = n1 * n2, comp = jb.comp;
  double u[kPer], v[kPer], g[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = min((int)threadIdx.x + kThreads * k, nn - 1);
    u[k] = sd.Us[i];
    v[k] = sd.Us[(sd.ncomp > 1 ? sd.N : 0) + i];
    if (!FIRST) g[k] = sd.G[comp * sd.N + i];
  }
  if constexpr (FIRST) {
    if (threadIdx.x < 6 * kSlabSumN) {
      const int q = threadIdx.x / kSlabSumN, i = threadIdx.x % kSlabSumN, dir = q / 3, n = dir ? n2 : n1;
      const int at = comp * 3 + dir, ic = min(i, n - 1);
      const double* c = q % 3 == 0 ? sd.st.lo[at] : q % 3 == 1 ? sd.st.di[at] : sd.st.up[at];
      const bool out = (q % 3 == 0 && i == 0) || (q % 3 == 2 && i + 1 >= n);   // zero past the boundary
      const double x = c[ic];
      K[threadIdx.x] = out ? 0.0 : x;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = (int)threadIdx.x + kThreads * k;
      if (i < nn) U[i] = comp == 0 ? u[k] : v[k];
    }
    __syncthreads();
  }
  const bool write_g = FIRST && lt == 0 && (jj == 0 || J.job[jj - 1].comp != comp);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = (int)threadIdx.x + kThreads * k;
    double r[2];
    reaction(sd.gp, u[k], sd.ncomp > 1 ? v[k] : 0.0, r[0], r[1]);
    const double gc = comp == 0 ? r[0] : r[1];
    if (i >= nn) continue;
    if constexpr (FIRST) {
      const int i2 = i / n1, i1 = i - i2 * n1;
      const double* k1 = K + i1;
      const double* k2 = K + 3 * kSlabSumN + i2;
      const double x = U[i];
      // rounded as in gf_stencil_kernel
      const double s1 = fma(k1[2 * kSlabSumN], U[i1 + 1 < n1 ? i + 1 : i],
                            fma(k1[kSlabSumN], x, k1[0] * U[i1 > 0 ? i - 1 : i]));
      const double s2 = fma(k2[2 * kSlabSumN], U[i2 + 1 < n2 ? i + n1 : i],
                            fma(k2[0], U[i2 > 0 ? i - n1 : i], k2[kSlabSumN] * x));
      X[i] = s1 + s2 + gc;
      if (write_g) sd.G[comp * sd.N + i] = gc;
    } else {
      X[i] = gc - g[k];
    }
  }
  __syncthreads();
  const int nt1 = (n1 + 15) >> 4;
  const int w = ((wave & 3) + (int)(lt & 3)) & 3, term = wave >> 2;
  if (w >= nt1) {   // a wave without i_1 blocks only keeps the barriers
    for (int k = 0; k < 3; ++k) __syncthreads();
    return;
  }
  slab_body<false, true, 1, 1, LD, true>(jb, 0, (int)lt, w, term, lane, Z, X);
}

// ---------------------------------------------------------------------------
// 192 <= n <= 256: the matrix panel in LDS
// ---------------------------------------------------------------------------
// Mode 1 with the matrix panel in LDS (interior jobs, 192 <= n <= 256,
// 4 x 4 tiles).  A workgroup of 8 waves shares one 64-row panel of P, stored
// in LDS in the order the MFMA reads it (chunk of 16 p, row m, lane: 4 p),
// so no wave holds P in registers; each wave then computes `reps` 64 x 64
// tiles of the workgroup's column group (8 * reps column tiles), reading X
// in 32-byte runs per lane (whole cache lines) through a two-deep ring that
// runs on from one tile into the next (FHN 256^3, 18 jobs: 2.31 ms when each
// tile started its own, 2.29 now; bound by the matrix cores, 67.5 TFLOP/s).
// Workgroup w of a job: panel w % tiles_i, column group w / tiles_i.
constexpr int kLdsWaves = 8;
constexpr int kLdsMinN = 192, kLdsMaxN = 256;
// Tiles per wave: 4 measured best at FHN 256^3 (mode 1 at 64.8 TFLOP/s
// against 63.0 with 2, 52.3 with 6 and 58.2 for the register-only kernel);
// below n = 192 the register-only kernel is faster (the panel fill weighs
// more against a shorter contraction).
constexpr int kLdsReps = 4;

__global__ void __launch_bounds__(512, 1) mode1_lds_kernel(const ModeJobs J, int64_t per_xcd, int reps) {
  __shared__ d4 panel[(kLdsMaxN / 16) * 4 * 64];   // 128 KB
  const int64_t w = remap_xcd(blockIdx.x, per_xcd);
  if (w >= J.total_tiles) return;   // uniform over the workgroup
  const int j = find_job(J, w);
  const ModeJob& jb = J.job[j];
  const int64_t lw = w - jb.tile_begin;
  const int it = (int)(lw % jb.tiles_i);
  const int64_t bg = lw / jb.tiles_i;
  const int n = jb.n;
  const int nchunk = n / 16;
  const int i0 = it * 64;
  const double* __restrict__ PT = (const double*)jb.P[0];
  // fill: entry q = (c * 4 + m) * 64 + lane holds P[i0 + 4 l + m][16 c + 4 g + 0..3]
  for (int q = threadIdx.x; q < nchunk * 256; q += 512) {
    const int ln = q & 63, m = (q >> 6) & 3, c = q >> 8;
    const int l = ln & 15, g = ln >> 4;
    const int i = i0 + 4 * l + m, p = 16 * c + 4 * g;   // p % 4 == 0: two neighbouring pairs of the packed matrix
    const double* e = PT + ((int64_t)(i >> 4) * chunks_of(n) + (p >> 3)) * 128 + (((p >> 1) & 3) * 16 + (i & 15)) * 2;
    const d2 lo = *(const d2*)e, hi = *(const d2*)(e + 32);
    panel[q] = d4{lo[0], lo[1], hi[0], hi[1]};
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, l = lane & 15;
  const double* __restrict__ X = (const double*)jb.X[0];
  // b-block of repetition r (past the job's blocks: not run), and the lane's
  // first X element of it
  auto block_of = [&](int r) { return (bg * reps + r) * kLdsWaves + wave; };
  auto xbase = [&](int64_t bt) { return X + (bt * 64 + l) * (int64_t)n + 4 * g; };
  auto load = [&](const double* xb, d4* xr) {
#pragma unroll
    for (int u = 0; u < 4; ++u) xr[u] = *(const d4*)(xb + 16 * u * (int64_t)n);
  };
  if (block_of(0) >= jb.tiles_a) return;   // no barrier follows
  const double* xb = xbase(block_of(0));
  d4 x0[4], x1[4];
  load(xb, x0);
  for (int rep = 0; rep < reps; ++rep) {
    const int64_t b0 = block_of(rep) * 64;
    // the next block's first chunk is loaded during this block's last one
    const bool next = rep + 1 < reps && block_of(rep + 1) < jb.tiles_a;
    const double* xn = next ? xbase(block_of(rep + 1)) : xb;
    __builtin_amdgcn_s_setprio(1);   // products ahead of another wave's epilogue on the SIMD
    d4 acc[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[m][u] = d4{0.0, 0.0, 0.0, 0.0};
    auto mma = [&](int c, const d4* xr) {
      d4 a[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) a[m] = panel[(c * 4 + m) * 64 + lane];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[m][u] = mfma(a[m][jj], xr[u][jj], acc[m][u]);
    };
    for (int c = 0; c < nchunk; c += 2) {   // nchunk is even (n % 32 == 0)
      load(xb + 16 * (c + 1), x1);
      mma(c, x0);
      load(c + 2 < nchunk ? xb + 16 * (c + 2) : xn, x0);   // unconditional: no branch
      mma(c + 1, x1);
    }
    __builtin_amdgcn_s_setprio(0);
    // epilogue: lane (g, l) owns rows i0 + 4 g + 16 r + (0..3) of column
    // b0 + 16 u + l
    const double sc = jb.scale[0];
    double* __restrict__ Y = (double*)jb.Y;
    const double* __restrict__ base = (const double*)jb.base;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t col = (b0 + 16 * u + l) * (int64_t)n;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ir = i0 + 4 * g + 16 * r;
        if (ir < n) {   // n % 32 == 0: all four or none
#pragma unroll
          for (int m = 0; m < 4; m += 2) {
            d2 v = d2{acc[m][u][r], acc[m + 1][u][r]} * sc;
            if (base) v += *(const d2*)(base + col + ir + m);
            *(d2*)(Y + col + ir + m) = v;
          }
        }
      }
    }
    if (!next) return;
    xb = xn;
  }
}

// Modes >= 2 with the matrix panel in LDS (interior single-term jobs,
// 192 <= n <= 256, n % 64 == 0, 4 x 4 tiles).  A workgroup of 8 waves shares
// one 64-column panel of P (times the job's scale), stored in LDS in the
// order the MFMA reads it (k-step, lane: 4 columns); each wave computes
// `reps` 64 a x 64 i tiles of the workgroup's group of (a-block, slab) pairs,
// reading X in 32-byte runs per lane through a two-deep ring of 4-k-step
// blocks.  (Multi-term jobs stay on the register kernel: refilling the panel
// for every term cost more than it saved.)
// Workgroup w of a job: panel w % tiles_i, group w / tiles_i of 8 * reps
// (a-block, slab) pairs, pair q = a-block q % tiles_a, slab q / tiles_a.
__global__ void __launch_bounds__(512, 1) modeB_lds_kernel(const ModeJobs J, int64_t per_xcd, int reps) {
  __shared__ d4 panel[(kLdsMaxN / 4) * 64];   // 128 KB
  const int64_t w = remap_xcd(blockIdx.x, per_xcd);
  if (w >= J.total_tiles) return;   // uniform over the workgroup
  const ModeJob& jb = J.job[find_job(J, w)];
  const int64_t lw = w - jb.tile_begin;
  const int it = (int)(lw % jb.tiles_i);
  const int64_t grp = lw / jb.tiles_i;
  const int n = jb.n;
  const int64_t na = jb.na;
  const int64_t npairs = (int64_t)jb.tiles_a * jb.nb;
  const int i0 = it * 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, l = lane & 15;
  // fill: entry q = kk * 64 + lane' holds sc * P[i0 + 4 l' + 0..3][4 kk + g']
  {
    const double* __restrict__ P = (const double*)jb.P[0];
    const double sc = jb.scale[0];
    for (int q = threadIdx.x; q < (n / 4) * 64; q += 512) {
      const int ln = q & 63, kk = q >> 6;
      const int i = i0 + 4 * (ln & 15), p = 4 * kk + (ln >> 4);
      panel[q] = d4{packed_at(P, n, i, p), packed_at(P, n, i + 1, p), packed_at(P, n, i + 2, p),
                    packed_at(P, n, i + 3, p)} * sc;
    }
  }
  __syncthreads();
  constexpr int KB = 4;
  const double* __restrict__ X = (const double*)jb.X[0];
  // (a-block, slab) pair of repetition r (past the job's pairs: not run), and
  // the lane's first X element of it
  auto pair_of = [&](int r) { return (grp * reps + r) * kLdsWaves + wave; };
  auto xbase = [&](int64_t q) {
    const int64_t at = q % jb.tiles_a, b = q / jb.tiles_a;
    return X + na * (int64_t)n * b + at * 64 + 4 * l + na * g;
  };
  auto loadblk = [&](const double* xb, int p0, d4* xr) {
#pragma unroll
    for (int k = 0; k < KB; ++k) xr[k] = *(const d4*)(xb + na * (int64_t)(p0 + 4 * k));
  };
  d4 xa[KB], xq[KB];
  if (pair_of(0) >= npairs) return;   // no barrier follows
  const double* xb = xbase(pair_of(0));
  loadblk(xb, 0, xa);
  for (int rep = 0; rep < reps; ++rep) {
    const int64_t q = pair_of(rep);
    // the next pair's first block is loaded during this pair's last one
    const bool next = rep + 1 < reps && pair_of(rep + 1) < npairs;
    const double* xn = next ? xbase(pair_of(rep + 1)) : xb;
    __builtin_amdgcn_s_setprio(1);   // products ahead of another wave's epilogue on the SIMD
    const int64_t at = q % jb.tiles_a, b = q / jb.tiles_a;
    const int64_t a0 = at * 64;
    const int64_t slab = na * (int64_t)n * b;
    d4 acc[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[m][u] = d4{0.0, 0.0, 0.0, 0.0};
    {
      auto mmablk = [&](int p0, const d4* xr) {
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          const d4 pv = panel[(p0 / 4 + k) * 64 + lane];
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int m = 0; m < 4; ++m) acc[m][u] = mfma(xr[k][m], pv[u], acc[m][u]);
        }
      };
      for (int p0 = 0; p0 < n; p0 += 8 * KB) {   // n % 32 == 0
        loadblk(xb, p0 + 4 * KB, xq);
        mmablk(p0, xa);
        const bool last = p0 + 8 * KB >= n;
        loadblk(last ? xn : xb + na * (int64_t)(p0 + 8 * KB), 0, xa);   // unconditional: no branch
        mmablk(p0 + 4 * KB, xq);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    // epilogue: lane (g, l) owns a = a0 + 4 g + 16 r + (0..3) of the columns
    // i0 + 4 l + u, every row and column in range
    double* __restrict__ Y = (double*)jb.Y;
    const double* __restrict__ base = (const double*)jb.base;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t off = slab + na * (int64_t)(i0 + 4 * l + u);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t ar = a0 + 4 * g + 16 * r;
#pragma unroll
        for (int m = 0; m < 4; m += 2) {
          d2 v = d2{acc[m][u][r], acc[m + 1][u][r]};
          if (base) v += *(const d2*)(base + off + ar + m);
          *(d2*)(Y + off + ar + m) = v;
        }
      }
    }
    if (!next) return;
    xb = xn;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int64_t assign_tiles_f64(ModeJob* jobs, int njobs, bool mode1, int ti, int to) {
  int64_t tot = 0;
  for (int j = 0; j < njobs; ++j) {
    ModeJob& jb = jobs[j];
    jb.tiles_i = (int)ceil_div(jb.n, 16 * ti);
    jb.tiles_a = 0;   // not used
    jb.tile_begin = tot;
    tot += jb.tiles_i * ceil_div(mode1 ? jb.nb : jb.na * jb.nb, 16 * to);
  }
  return tot;
}

namespace {

bool aligned(const void* p, uintptr_t a) { return ((uintptr_t)p % a) == 0; }

// Tile of one launch: ti x to blocks of 16 (i x the other index) per wave, ks
// waves per tile (1 x 4: modes >= 2 of up to kShortN, bound by memory: few
// registers, so that six waves share a SIMD; 1024 x 2 x 3200, mode 2, 46 us
// against 82 with 2 x 2, 1024 x 16 x 400 18.4 against 23.4).  rate: share of the matrix rate that the products of its
// waves reach (1 x 1 tiles wait for their operands); rate_long: the same for n >
// kLongN, where the matrix (8 n^2 bytes) is past the 4 MB of an XCD's L2 and
// every tile reads it from further away, the smaller the tile the oftener (2048
// x 4096, mode 1: 2 x 2 tiles with 4 waves 732 us, 4 x 4 483); block: cycles per
// block that loading and storing it adds to a wave (fitted to sweeps of all
// tiles at 64^2 .. 600^2, 64^3 .. 256^3 and up to 4096 in one direction).
struct TileCfg {
  int ti, to, ks;
  double rate, rate_long, block;
};
constexpr int kLongN = 640, kShortN = 16;
constexpr TileCfg kTiles[] = {{1, 1, 4, .50, .36, 550}, {1, 4, 1, .84, .70, 700}, {2, 2, 4, .92, .66, 550},
                              {2, 2, 2, .86, .68, 600}, {2, 2, 1, .84, .70, 700}, {4, 2, 4, .92, .80, 550},
                              {4, 2, 2, .92, .84, 600}, {4, 2, 1, .90, .85, 700}, {5, 2, 4, .92, .80, 550},
                              {5, 2, 1, .92, .75, 700}, {7, 1, 4, .92, .60, 550}, {7, 2, 1, .92, .72, 700},
                              {4, 4, 1, .94, .94, 700}};

TileCfg env_tile(const char* name, TileCfg def) {
  const char* s = std::getenv(name);
  if (!s) return def;
  int a = 0, b = 0, c = 1;
  if (std::sscanf(s, "%dx%dx%d", &a, &b, &c) >= 2)
    for (const TileCfg& t : kTiles)
      if (t.ti == a && t.to == b && t.ks == c) return t;
  return def;
}

int64_t tile_count(const ModeJobs& J, bool mode1, const TileCfg& t) {
  int64_t w = 0;
  for (int j = 0; j < J.njobs; ++j) {
    const ModeJob& jb = J.job[j];
    w += ceil_div(jb.n, 16 * t.ti) * ceil_div(mode1 ? jb.nb : jb.na * jb.nb, 16 * t.to);
  }
  return w;
}

// The tile whose launch should take least time: rounds of 1024 SIMDs (a
// partial one counts whole while there are few), each as long as one wave, 64
// cycles per MFMA, and the part of a wave that the launch begins and ends with.
// A launch with a round of 4 x 4 tiles fills the chip: that part is small, and
// waves that split a contraction add only its parts (128 x 65536, mode 1: 4 x 4
// 43 us, 4 x 2 53; 64 x 99328: 4 x 4 26, 4 x 2 of two waves 35).  Mode 1 with n a
// multiple of 16: every row of X starts at a line, so that the half lines of a
// load fall into the same half of the L1's banks, which tiles with little of i to
// reuse them for feel (224 x 27648: 2 x 2 70 us, 7 x 2 55; modes >= 2 of that size
// 51 and 59).  4 x 4 tiles, two waves to a SIMD, run in pairs of rounds (230 x
// 46200, mode 1, 2.8 rounds: 124 us, as long as 4; 2 x 2 97).  Measured against each other at the two ends: 300^2, 4 jobs of mode
// 1: 2 x 2 tiles with 4 waves each 9.2 us, 4 x 4 41.9; 256^3, 6 jobs of 3 terms: 4
// x 4 2.17 ms, 4 x 2 2.27, 2 x 2 with 4 waves 3.4.
TileCfg choose_tile(const ModeJobs& J, bool mode1) {
  const bool full = tile_count(J, mode1, TileCfg{4, 4, 1, 0, 0, 0}) >= 1024;
  bool wide = !mode1;   // 1 x 4
  for (int j = 0; j < J.njobs; ++j) wide = wide && J.job[j].n <= kShortN;
  TileCfg best{4, 4, 1, 0, 0, 0};
  double bt = 1e300;
  for (const TileCfg& t : kTiles) {
    if ((t.ti == 1 && t.to == 4 && !wide) || (full && t.ks > 1)) continue;
    const int64_t tiles = tile_count(J, mode1, t);
    if (!fits_grid(tiles, t.ks)) continue;
    const double w = (double)tiles * t.ks / 1024.0;
    double wave = 0.0;
    for (int j = 0; j < J.njobs; ++j) {
      const ModeJob& jb = J.job[j];
      const double chunks = (double)jb.nterms * ceil_div(jb.n, 8) / t.ks;
      const double banks = mode1 && t.ti <= 2 && jb.n > 32 && jb.n % 16 == 0 ? 0.7 : 1.0;
      const double rate = banks * (jb.n > kLongN ? t.rate_long : t.rate);
      wave = std::max(wave, t.ti * t.to * (chunks * 128.0 / rate + t.block * (jb.base ? 1.6 : 1.0)));
    }
    const bool pairs = t.ti * t.to == 16 && w > 1.0;
    const double rounds = w >= 6.0 ? w : pairs ? 2.0 * std::ceil(w / 2.0) : std::ceil(w);
    const double time = (rounds + (full ? 0.1 : 0.3)) * wave;
    if (time < bt) {
      bt = time;
      best = t;
    }
  }
  return best;
}

int finish_tiles(ModeJobs& J, bool mode1, const TileCfg& t) {
  J.total_tiles = assign_tiles_f64(J.job, J.njobs, mode1, t.ti, t.to);
  J.tiles_per_job = J.njobs > 0 ? J.total_tiles / J.njobs : 0;
  for (int j = 0; j < J.njobs; ++j)
    if (J.job[j].tile_begin != (int64_t)j * J.tiles_per_job) J.tiles_per_job = 0;
  return SETD_OK;
}

template <bool M1, bool RAW, int TI, int TO, int KS, typename Off, bool V = false>
int launch_tile(const ModeJobs& J, hipStream_t s) {
  const int64_t per = ceil_div(ceil_div(J.total_tiles, 4 / KS), 8);
  hipLaunchKernelGGL((mode_f64_kernel<M1, RAW, TI, TO, KS, Off, V>), dim3((unsigned)(per * 8)), dim3(256), 0, s, J, per);
  SETD_LAUNCHED();
  return SETD_OK;
}

// Modes >= 2 whose contraction is not split load and store a lane's TO columns
// together where no slab ends between them: at 256^3 (6 jobs of 3 terms) 4 x 4
// tiles take 2.17 ms and not 2.29, 4 x 2 2.27 and not 2.38; 200^3 2 x 2 1.02 and
// not 1.08; but 7 x 2, whose matrix loads are most of it, 1.007 and not 0.996.
template <bool M1, bool RAW>
int launch_cfg(const ModeJobs& J, const TileCfg& t, hipStream_t s) {
#define SETD_TILE(TI_, TO_, KS_) \
  if (t.ti == TI_ && t.to == TO_ && t.ks == KS_) {                                              \
    if constexpr (!M1 && KS_ == 1 && TI_ <= 5)                                                  \
      if (vector_columns(J, TO_)) return launch_tile<M1, RAW, TI_, TO_, KS_, uint32_t, true>(J, s); \
    return launch_tile<M1, RAW, TI_, TO_, KS_, uint32_t>(J, s);                                \
  }
  SETD_TILE(1, 1, 4)
  SETD_TILE(1, 4, 1)
  SETD_TILE(2, 2, 4)
  SETD_TILE(2, 2, 2)
  SETD_TILE(2, 2, 1)
  SETD_TILE(4, 2, 4)
  SETD_TILE(4, 2, 2)
  SETD_TILE(4, 2, 1)
  SETD_TILE(5, 2, 4)
  SETD_TILE(5, 2, 1)
  SETD_TILE(7, 1, 4)
  SETD_TILE(7, 2, 1)
  SETD_TILE(4, 4, 1)
#undef SETD_TILE
  set_error("unsupported tile %dx%d", t.ti, t.to);
  return SETD_EUNSUPPORTED;
}

// The panel kernels' job records: workgroups instead of tiles.
void finish_panels(ModeJobs& J, bool mode1) {
  int64_t tot = 0;
  for (int j = 0; j < J.njobs; ++j) {
    ModeJob& jb = J.job[j];
    jb.tiles_i = (int)ceil_div(jb.n, 64);
    jb.tiles_a = (int)((mode1 ? jb.nb : jb.na) / 64);
    jb.tile_begin = tot;
    tot += (int64_t)jb.tiles_i * ceil_div((int64_t)jb.tiles_a * (mode1 ? 1 : jb.nb), (int64_t)kLdsWaves * kLdsReps);
  }
  J.total_tiles = tot;
  J.tiles_per_job = J.njobs > 0 ? tot / J.njobs : 0;
  for (int j = 0; j < J.njobs; ++j)
    if (J.job[j].tile_begin != (int64_t)j * J.tiles_per_job) J.tiles_per_job = 0;
}

// Whether the LDS panel kernels take a job: one term, 192 <= n <= 256, whole
// panels and tiles, aligned vector accesses.
bool panel_job(const ModeJob& jb, bool mode1) {
  if (jb.nterms != 1 || jb.n < kLdsMinN || jb.n > kLdsMaxN) return false;
  if (!aligned(jb.X[0], 32) || !aligned(jb.Y, 16) || !aligned(jb.base, 16)) return false;
  return mode1 ? jb.n % 32 == 0 && jb.nb % 64 == 0 : jb.n % 64 == 0 && jb.na % 64 == 0;
}

}  // namespace

void job_work(const ModeJobs& J, int es_in, int es_out, int es_mat, double& flops, double& bytes) {
  flops = 0.0;
  bytes = 0.0;
  for (int j = 0; j < J.njobs; ++j) {
    const ModeJob& jb = J.job[j];
    const double N = (double)jb.na * jb.n * jb.nb;
    flops += jb.nterms * 2.0 * N * jb.n;
    bytes += jb.nterms * (N * es_in + (double)jb.n * jb.n * es_mat) + N * es_out * (jb.base ? 2.0 : 1.0);
  }
}

int launch_mode1_f64(ModeJobs& J, hipStream_t s, bool raw) {
  double fl = 0.0, by = 0.0;
  if (prof_on()) job_work(J, 8, 8, 8, fl, by);
  bool lds = J.njobs > 0 && !raw;
  for (int j = 0; j < J.njobs; ++j) lds = lds && panel_job(J.job[j], true);
  const TileCfg cfg = env_tile("SETD_TILE_MODE1", choose_tile(J, true));
  if (lds) finish_panels(J, true);
  else finish_tiles(J, true, cfg);
  if (J.total_tiles == 0) return SETD_OK;
  ProfScope prof(s, kProfMode1F64, fl, by);
  if (!lds) return raw ? launch_cfg<true, true>(J, cfg, s) : launch_cfg<true, false>(J, cfg, s);
  const int64_t per = ceil_div(J.total_tiles, 8);
  hipLaunchKernelGGL(mode1_lds_kernel, dim3((unsigned)(per * 8)), dim3(64 * kLdsWaves), 0, s, J, per, kLdsReps);
  SETD_LAUNCHED();
  return SETD_OK;
}

int launch_modeB_f64(ModeJobs& J, hipStream_t s, bool raw) {
  double fl = 0.0, by = 0.0;
  if (prof_on()) job_work(J, 8, 8, 8, fl, by);
  bool lds = J.njobs > 0 && !raw, big = false;
  for (int j = 0; j < J.njobs; ++j) {
    lds = lds && panel_job(J.job[j], false);
    // a tile's offsets span more than 32 bits: 8 rows of X, or (with several
    // slabs) the slabs of one tile's columns
    const ModeJob& jb = J.job[j];
    big = big || jb.na > (int64_t(1) << 26) ||
          (jb.nb > 1 && (ceil_div(128, jb.na) + 1) * jb.na * jb.n > (int64_t(1) << 28));
  }
  TileCfg cfg = big ? TileCfg{4, 2, 1, 0, 0, 0} : env_tile("SETD_TILE_MODEB", choose_tile(J, false));
  if (big && !fits_grid(tile_count(J, false, cfg), 1)) cfg = TileCfg{4, 4, 1, 0, 0, 0};
  if (lds) finish_panels(J, false);
  else finish_tiles(J, false, cfg);
  if (J.total_tiles == 0) return SETD_OK;
  // the two kernels are timed as separate classes
  ProfScope prof(s, lds ? kProfModeBPanelF64 : kProfModeBF64, fl, by);
  if (big && !lds) {
    if (cfg.to == 4) return launch_tile<false, false, 4, 4, 1, uint64_t>(J, s);   // raw tensors are not that large
    return raw ? launch_tile<false, true, 4, 2, 1, uint64_t>(J, s) : launch_tile<false, false, 4, 2, 1, uint64_t>(J, s);
  }
  if (!lds) return raw ? launch_cfg<false, true>(J, cfg, s) : launch_cfg<false, false>(J, cfg, s);
  const int64_t per = ceil_div(J.total_tiles, 8);
  hipLaunchKernelGGL(modeB_lds_kernel, dim3((unsigned)(per * 8)), dim3(64 * kLdsWaves), 0, s, J, per, kLdsReps);
  SETD_LAUNCHED();
  return SETD_OK;
}

namespace {
template <bool RAW, bool SUM, int TJ, int NI>
int launch_slab_tile(SlabJobs& J, hipStream_t s) {
  J.nblk = (int)ceil_div(ceil_div(J.job[0].n2, 16), TJ);
  J.tiles_per_job = J.nblk * J.job[0].nb;
  J.total = J.tiles_per_job * J.njobs;
  const int64_t per = ceil_div(J.total, 8);
  hipLaunchKernelGGL((slab_f64_kernel<RAW, SUM, TJ, NI>), dim3((unsigned)(per * 8)),
                     dim3(SUM ? 256 * kSlabTerms : 256), 0, s, J, per);
  SETD_LAUNCHED();
  return SETD_OK;
}

template <bool RAW, bool SUM>
int launch_slab_ni(SlabJobs& J, hipStream_t s) {
  // one column tile per workgroup while that leaves a workgroup per CU or less
  const bool wide = ceil_div(J.job[0].n2, 16) * J.job[0].nb * J.njobs > 256;
  if constexpr (SUM) return launch_slab_tile<RAW, SUM, 1, 1>(J, s);   // n1 <= kSlabSumN
  switch (ceil_div(J.job[0].n1, 64)) {
    case 1: return wide ? launch_slab_tile<RAW, SUM, 2, 1>(J, s) : launch_slab_tile<RAW, SUM, 1, 1>(J, s);
    case 2: return wide ? launch_slab_tile<RAW, SUM, 2, 2>(J, s) : launch_slab_tile<RAW, SUM, 1, 2>(J, s);
    case 3: return wide ? launch_slab_tile<RAW, SUM, 2, 3>(J, s) : launch_slab_tile<RAW, SUM, 1, 3>(J, s);
    case 4: return wide ? launch_slab_tile<RAW, SUM, 2, 4>(J, s) : launch_slab_tile<RAW, SUM, 1, 4>(J, s);
  }
  set_error("slab product: n1 = %d", J.job[0].n1);
  return SETD_EUNSUPPORTED;
}
}  // namespace

int launch_slab_f64(SlabJobs& J, hipStream_t s, bool raw) {
  if (J.njobs == 0) return SETD_OK;
  double fl = 0.0, by = 0.0;
  bool sum = false;
  for (int j = 0; j < J.njobs; ++j) {
    const SlabJob& q = J.job[j];
    const double N = (double)q.n1 * q.n2 * q.nb;
    fl += q.nterms * 2.0 * N * (q.n1 + q.n2);
    by += q.nterms * (8.0 * N + 8.0 * q.n1 * q.n1 + 8.0 * q.n2 * q.n2) + N * (q.base ? 16.0 : 8.0);
    sum = sum || q.nterms > 1;
  }
  ProfScope prof(s, kProfMode1F64, fl, by);
  if (raw && !sum) return launch_slab_ni<true, false>(J, s);
  if (sum && (raw || J.job[0].n1 > kSlabSumN)) {
    set_error("slab product: sums need packed matrices and n1 <= %d", kSlabSumN);
    return SETD_EUNSUPPORTED;
  }
  return sum ? launch_slab_ni<false, true>(J, s) : launch_slab_ni<false, false>(J, s);
}

int launch_slab_diff_f64(SlabJobs& J, const StageDiff& diff, hipStream_t s) {
  if (J.njobs == 0) return SETD_OK;
  double fl = 0.0, by = 0.0;
  for (int j = 0; j < J.njobs; ++j) {
    const SlabJob& q = J.job[j];
    if (q.nterms != kSlabTerms || q.nb != 1 || q.n1 > kSlabSumN || q.n2 > kSlabSumN || q.n1 != J.job[0].n1 ||
        q.n2 != J.job[0].n2 || (int64_t)q.n1 * q.n2 != diff.N || q.comp < 0 || q.comp >= diff.ncomp) {
      set_error("slab product of a stage difference: two terms on one slab of up to %d x %d", kSlabSumN, kSlabSumN);
      return SETD_EUNSUPPORTED;
    }
    const double N = (double)q.n1 * q.n2;
    fl += q.nterms * 2.0 * N * (q.n1 + q.n2);
    by += 24.0 * N + q.nterms * (8.0 * q.n1 * q.n1 + 8.0 * q.n2 * q.n2) + N * (q.base ? 16.0 : 8.0);
  }
  ProfScope prof(s, kProfMode1F64, fl, by);
  J.nblk = (int)ceil_div(J.job[0].n2, 16);
  J.tiles_per_job = J.nblk;
  J.total = J.tiles_per_job * J.njobs;
  const int64_t per = ceil_div(J.total, 8);
  hipLaunchKernelGGL(diff.first ? slab_diff_f64_kernel<true> : slab_diff_f64_kernel<false>, dim3((unsigned)(per * 8)),
                     dim3(256 * kSlabTerms), 0, s, J, diff, per);
  SETD_LAUNCHED();
  return SETD_OK;
}

namespace {
template <int TI, int TO, int KS>
void launch_list_tile(const ModeList& L, dim3 grid, int64_t groups, hipStream_t s) {
  if (L.mode1)
    hipLaunchKernelGGL((mode_f64_list_kernel<true, TI, TO, KS>), grid, dim3(256), 0, s, L.jobs, L.begins, L.njobs,
                       L.total, groups);
  else
    hipLaunchKernelGGL((mode_f64_list_kernel<false, TI, TO, KS>), grid, dim3(256), 0, s, L.jobs, L.begins, L.njobs,
                       L.total, groups);
}
}  // namespace

int launch_list_f64(const ModeList& L, hipStream_t s) {
  if (L.total == 0) return SETD_OK;
  const int64_t groups = round_up(ceil_div(L.total, 4 / L.ks), 8 * kListRun);
  // a multiple of 8 blocks, so that block b stays on XCD b % 8 through the
  // whole loop; at most `grid_cap` of them, rounded up (0: all)
  int64_t nblk = groups;
  if (L.grid_cap > 0 && nblk > L.grid_cap) nblk = round_up(L.grid_cap, 8);
  const dim3 grid((unsigned)nblk);
  ProfScope prof(s, L.mode1 ? kProfMode1F64 : kProfModeBF64, L.flops, L.bytes);
  const int key = 100 * L.ti + 10 * L.to + L.ks;
  switch (key) {
    case 224: launch_list_tile<2, 2, 4>(L, grid, groups, s); break;
    case 222: launch_list_tile<2, 2, 2>(L, grid, groups, s); break;
    case 221: launch_list_tile<2, 2, 1>(L, grid, groups, s); break;
    case 241: launch_list_tile<2, 4, 1>(L, grid, groups, s); break;
    case 424: launch_list_tile<4, 2, 4>(L, grid, groups, s); break;
    case 422: launch_list_tile<4, 2, 2>(L, grid, groups, s); break;
    case 421: launch_list_tile<4, 2, 1>(L, grid, groups, s); break;
    case 441: launch_list_tile<4, 4, 1>(L, grid, groups, s); break;
    default:
      set_error("unsupported tile %dx%dx%d", L.ti, L.to, L.ks);
      return SETD_EUNSUPPORTED;
  }
  SETD_LAUNCHED();
  return SETD_OK;
}

}  // namespace setd
