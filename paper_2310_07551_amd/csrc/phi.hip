// phi-functions of small dense matrices on the GPU, computed in double-double
// arithmetic and rounded once to FP64.
//
// Section 2.4 computes the phi matrices once, before time stepping, with
// scaling and "modified squaring" (Skaflestad and Wright, 2009).  This file
// does all of it on the device:
//
//  1. X = c A (the FP64 product of the scalar and each entry);
//     s = max(0, ceil(log2 ||X||_1)),  Y = X / 2^s  (exact).
//  2. The Taylor polynomials of degree 21 of every order at Y (||Y||_1 <= 1).
//  3. s modified squarings
//       phi_0(2Y) = phi_0(Y)^2,
//       phi_k(2Y) = 2^{-k} [ phi_0(Y) phi_k(Y) + sum_{j=1}^{k} phi_j(Y)/(k-j)! ].
//
// Accuracy.  A squaring maps an error E in phi_0(Y) to about phi_0 E + E
// phi_0; on an eigenvector whose eigenvalue is near zero (the constant vector
// of a Neumann Laplacian, where phi_0 = 1) that doubles it.  s squarings thus
// turn a rounding error of u into 2^s u ~ u ||X||: 2e-11 for the stiffest
// matrix of a 256-point direction of the 3D FitzHugh-Nagumo workload (||X||
// ~ 2e5), enough to move a time step's result by ~1e-12.  Here every matrix
// entry is a pair of FP64 numbers (hi, lo) and every product and sum is done in
// double-double arithmetic (error ~ u^2 per operation), so 2^s u^2 stays far
// below an FP64 ulp, and the result is rounded once.
//
// Deviations.  All stages carry psi_k = phi_k - I/k! instead of phi_k:
//   psi_k(Y)  = sum_{i>=1} Y^i / (k+i)!;
//   psi_0(2Y) = psi_0^2 + 2 psi_0;
//   psi_k(2Y) = 2^{-k} [ psi_0 psi_k + psi_0/k! + 2 psi_k + sum_{j=1}^{k-1} psi_j/(k-j)! ]   (k >= 1),
// which follow from the formulas above with phi_j = I/j! + psi_j (the identity
// parts sum to I/k!).  On an eigenvector with eigenvalue 0 every psi is
// exactly 0, and a small relative error of the polynomial (the terms left out
// are below 1/22! ~ 9e-22 of psi) stays a small relative error of psi through
// the squarings instead of being doubled s times.
//
// Work.  The polynomials share the powers Y .. Y^7 (three levels of products)
// and take two more products each (Paterson-Stockmeyer, blocks of seven
// terms): five levels of batched products where a diagonal Pade quotient by
// an iterated inverse took 22 in a row.  Everything linear that follows a
// product (the next block of terms, the sums of a squaring, the final I/k! and
// rounding) is done where its result is stored.
//
// A batch shares A and n; every entry has its own scalar c_j and the batch
// uses the largest scaling exponent of its entries (extra squarings of a
// smaller argument only shrink the truncation error).
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "common.hpp"
#include "pointwise.hpp"

// Double-double arithmetic relies on every sum and product being rounded on
// its own; explicit fma() calls are the only fused operations in this file.
#pragma clang fp contract(off)

namespace setd {
namespace {

constexpr int kMaxOrder = 6;
constexpr int kPowers = 7;               // Y .. Y^7
constexpr int kBlocks = 3;               // blocks of seven terms: degree 21
constexpr int kMaxEntries = 64;          // scalars of one launch

// ---- double-double helpers (device and host) ----
struct DD {
  double hi, lo;
};

__host__ __device__ inline DD dd_two_sum(double a, double b) {
  const double s = a + b;
  const double v = s - a;
  return {s, (a - (s - v)) + (b - v)};
}

__host__ __device__ inline DD dd_add(DD a, DD b) {
  const DD s = dd_two_sum(a.hi, b.hi);
  const double e = s.lo + (a.lo + b.lo);
  return dd_two_sum(s.hi, e);
}

__device__ inline DD dd_mul(DD a, DD b) {
  const double p = a.hi * b.hi;
  double e = fma(a.hi, b.hi, -p);
  e = fma(a.hi, b.lo, e);
  e = fma(a.lo, b.hi, e);
  return dd_two_sum(p, e);
}

// a / b for a double-double a and an FP64 b (host).
inline DD hdd_div(DD a, double b) {
  const double q1 = a.hi / b;
  const double r = std::fma(-q1, b, a.hi) + a.lo;   // fma(-q1, b, a.hi) is exact
  return dd_two_sum(q1, r / b);
}

// ---- matrices: n^2 (hi, lo) pairs, column-major; entry j of a batch holds its
// blocks (powers, then two sets of psi_0 .. psi_p) one after another ----

// C = 2^-shift (A B + sum_q coef_q M_q) for blocks of one entry; final_k >= 0:
// phi_k = I/k! + C rounded to FP64 into the caller's matrix instead.
constexpr int kMaxAdd = kPowers + 1;
struct Product {
  int a, b, c;
  int nadd, shift, final_k;
  int add[kMaxAdd];
  DD coef[kMaxAdd];
};
struct Level {
  Product prod[kMaxOrder + 1];
  int count;          // products per entry
  int n, orders;      // orders = p + 1
  int64_t stride;     // pairs per entry
  d2* ws;
  double* out;        // phi_k of entry j at (j * orders + k) n^2
  DD unit[kMaxOrder + 1];   // 1/k!
};

// One 16 x 16 tile per workgroup: its four waves take every fourth chunk of 16
// contraction indices and their sums meet in LDS, so that even one matrix
// (256 tiles at n = 256, three orders) fills the chip three times over; a
// 64 x 64 tile per workgroup ran on 48 of 256 compute units, 112 us a launch.
// Bound by the FP64 vector units: 12 operations per product (its rounding
// error by fma, the cross terms, a two-sum), 2 x 2 results per lane so that
// four operand reads from LDS serve four of them.
constexpr int kTile = 16;
__global__ void __launch_bounds__(256, 3) product_dd_kernel(const Level L) {
  const int z = blockIdx.z, e = z / L.count, q = z - e * L.count;
  const Product& P = L.prod[q];
  const int n = L.n;
  const int64_t nn = (int64_t)n * n;
  d2* const base = L.ws + L.stride * e;
  const d2* __restrict__ A = base + nn * P.a;
  const d2* __restrict__ B = base + nn * P.b;
  __shared__ d2 As[4][kTile][kTile];         // [wave][k][row]
  __shared__ d2 Bs[4][kTile][kTile + 1];     // [wave][k][column]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int tx = lane & 7, ty = lane >> 3;
  const int m0 = blockIdx.x * kTile, n0 = blockIdx.y * kTile;
  const int r16 = lane & 15, r4 = lane >> 4;
  double ch[2][2] = {{0.0, 0.0}, {0.0, 0.0}}, cl[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
  d2 ra[4], rb[4];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int ka = k0 + r4 + 4 * t, row = m0 + r16, kb = k0 + r16, col = n0 + r4 + 4 * t;
      ra[t] = (row < n && ka < n) ? A[row + (int64_t)n * ka] : d2{0.0, 0.0};
      rb[t] = (kb < n && col < n) ? B[kb + (int64_t)n * col] : d2{0.0, 0.0};
    }
  };
  int k0 = wave * kTile;
  if (k0 < n) fetch(k0);
  for (; k0 < n; k0 += 4 * kTile) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      As[wave][r4 + 4 * t][r16] = ra[t];
      Bs[wave][r16][r4 + 4 * t] = rb[t];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // each wave reads only what it wrote
    __builtin_amdgcn_wave_barrier();
    if (k0 + 4 * kTile < n) fetch(k0 + 4 * kTile);
#pragma unroll 4
    for (int k = 0; k < kTile; ++k) {
      d2 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = As[wave][k][tx + 8 * i];
        b[i] = Bs[wave][k][ty + 8 * i];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const double p = a[i][0] * b[j][0];
          double er = fma(a[i][0], b[j][0], -p);
          er = fma(a[i][0], b[j][1], er);
          er = fma(a[i][1], b[j][0], er);
          const double s = ch[i][j] + p;
          const double v = s - ch[i][j];
          const double t = (ch[i][j] - (s - v)) + (p - v);
          ch[i][j] = s;
          cl[i][j] = cl[i][j] + (t + er);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  // the four parts of a result meet in the waves' own A tiles
  d2* const part = &As[wave][0][0];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) part[(tx + 8 * i) + kTile * (ty + 8 * j)] = d2{ch[i][j], cl[i][j]};
  __syncthreads();
  const int r = m0 + (threadIdx.x & 15), c = n0 + (threadIdx.x >> 4);
  if (r >= n || c >= n) return;
  DD v{0.0, 0.0};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const d2 x = (&As[w][0][0])[threadIdx.x];
    v = dd_add(v, dd_two_sum(x[0], x[1]));
  }
  const int64_t idx = r + (int64_t)n * c;
  for (int t = 0; t < P.nadd; ++t) {
    const d2 m = base[nn * P.add[t] + idx];
    v = dd_add(v, dd_mul(P.coef[t], DD{m[0], m[1]}));
  }
  v.hi = ldexp(v.hi, -P.shift);
  v.lo = ldexp(v.lo, -P.shift);
  if (P.final_k >= 0) {
    if (r == c) v = dd_add(v, L.unit[P.final_k]);
    L.out[((int64_t)e * L.orders + P.final_k) * nn + idx] = v.hi + v.lo;
  } else {
    base[nn * P.c + idx] = d2{v.hi, v.lo};
  }
}

// Column sums of |A| (their maximum is ||A||_1; not finite if an entry is
// not): one wave per column.
__global__ void norm1_kernel(const double* __restrict__ A, int n, double* __restrict__ out) {
  const int j = (int)(blockIdx.x * (blockDim.x >> 6)) + (threadIdx.x >> 6);
  if (j >= n) return;
  double s = 0.0;
  for (int i = threadIdx.x & 63; i < n; i += 64) s += fabs(A[i + (int64_t)n * j]);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) out[j] = s;
}

// Y_j = (c_j A) 2^-s for every entry: hi = the FP64 product (scal_j = c_j 2^-s,
// an exact power-of-two scaling of c_j), lo = 0.
struct Scalars {
  double c[kMaxEntries];
};
__global__ void scale_batch_kernel(const double* __restrict__ A, int64_t nn, Scalars scal, d2* __restrict__ W,
                                   int64_t stride) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nn) return;
  W[stride * blockIdx.y + idx] = d2{scal.c[blockIdx.y] * A[idx], 0.0};
}

// The highest block of terms of every order: block dst + k of each entry =
// sum_i coef[k + i] Y^(i+1), i < kPowers.
struct TopCoefs {
  DD c[kMaxOrder + kPowers];
};
__global__ void top_block_kernel(d2* __restrict__ W, int64_t nn, int64_t stride, int orders, int dst, TopCoefs cf) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nn) return;
  d2* w = W + stride * blockIdx.y;
  d2 y[kPowers];
#pragma unroll
  for (int i = 0; i < kPowers; ++i) y[i] = w[nn * i + idx];
  for (int k = 0; k < orders; ++k) {
    DD v{0.0, 0.0};
#pragma unroll
    for (int i = kPowers - 1; i >= 0; --i) v = dd_add(v, dd_mul(cf.c[k + i], DD{y[i][0], y[i][1]}));
    w[nn * (dst + k) + idx] = d2{v.hi, v.lo};
  }
}

// Workspace of the builds: one buffer per device of at most kPoolBytes, kept
// between calls (allocating and freeing it cost more than a small build) until
// setd_release_workspace or a failing allocation.  A call owns it from its first launch to its final
// synchronisation; a call that finds it taken, or needs more, allocates its own.
constexpr size_t kPoolBytes = (size_t)256 << 20;
constexpr int kMaxDevices = 64;
struct Pool {
  std::mutex mu;
  void* p = nullptr;
  size_t bytes = 0;
};
Pool g_pool[kMaxDevices];

class Workspace {
 public:
  ~Workspace() {
    if (own_) (void)hipFree(own_);
  }
  int get(size_t bytes) {
    int dev = 0;
    SETD_HIP(hipGetDevice(&dev));
    if (bytes <= kPoolBytes && dev >= 0 && dev < kMaxDevices) {
      lock_ = std::unique_lock<std::mutex>(g_pool[dev].mu, std::try_to_lock);
      if (lock_.owns_lock()) {
        Pool& pool = g_pool[dev];
        if (pool.bytes < bytes) {
          if (pool.p) (void)hipFree(pool.p);
          pool.p = nullptr;
          pool.bytes = 0;
          SETD_TRY(device_malloc(&pool.p, bytes, false));
          pool.bytes = bytes;
        }
        p = (char*)pool.p;
        return SETD_OK;
      }
    }
    SETD_TRY(device_malloc(&own_, bytes));
    p = (char*)own_;
    return SETD_OK;
  }
  char* p = nullptr;

 private:
  void* own_ = nullptr;
  std::unique_lock<std::mutex> lock_;
};

int launch_level(const Level& L, int E, hipStream_t s) {
  const unsigned t = (unsigned)ceil_div(L.n, kTile);
  hipLaunchKernelGGL(product_dd_kernel, dim3(t, t, (unsigned)(E * L.count)), dim3(256), 0, s, L);
  SETD_LAUNCHED();
  return SETD_OK;
}

// phi_0 .. phi_p of c_j A for the entries of one chunk; anorm = ||A||_1.
int build_chunk(const double* A, int n, const double* c, int E, int p, double anorm, double* out, d2* ws,
                int64_t stride, hipStream_t s) {
  const int64_t nn = (int64_t)n * n;
  double cmax = 0.0;
  for (int j = 0; j < E; ++j) cmax = std::max(cmax, std::fabs(c[j]));
  const double xnorm = cmax * anorm;
  int sq = 0;
  if (xnorm > 1.0) sq = (int)std::ceil(std::log2(xnorm));
  if (sq > 1000) {
    set_error("phi: argument norm too large");
    return SETD_EUNSUPPORTED;
  }
  DD fact[kMaxOrder + kBlocks * kPowers + 1];   // 1/k!
  fact[0] = DD{1.0, 0.0};
  for (int k = 1; k <= kMaxOrder + kBlocks * kPowers; ++k) fact[k] = hdd_div(fact[k - 1], (double)k);

  // blocks of an entry: Y .. Y^7 | bufA[0..p] | bufB[0..p]
  const int offA = kPowers, offB = kPowers + p + 1;
  Level L{};
  L.n = n;
  L.orders = p + 1;
  L.stride = stride;
  L.ws = ws;
  L.out = out;
  for (int k = 0; k <= p; ++k) L.unit[k] = fact[k];
  auto product = [&](int a, int b, int dst) {
    Product& P = L.prod[L.count++];
    P = Product{};
    P.a = a;
    P.b = b;
    P.c = dst;
    P.final_k = -1;
    return &P;
  };
  const dim3 ew((unsigned)ceil_div(nn, 256), (unsigned)E);
  Scalars scal{};
  for (int j = 0; j < E; ++j) scal.c[j] = std::ldexp(c[j], -sq);
  hipLaunchKernelGGL(scale_batch_kernel, ew, dim3(256), 0, s, A, nn, scal, ws, stride);
  SETD_LAUNCHED();
  // powers (block i holds Y^(i+1))
  product(0, 0, 1);
  SETD_TRY(launch_level(L, E, s));
  L.count = 0;
  product(1, 0, 2);
  product(1, 1, 3);
  SETD_TRY(launch_level(L, E, s));
  L.count = 0;
  product(3, 0, 4);
  product(3, 1, 5);
  product(3, 2, 6);
  SETD_TRY(launch_level(L, E, s));
  // psi_k = sum_{b} Y^(7b) sum_{i=1..7} Y^i / (k + 7b + i)!, highest block first
  TopCoefs top{};
  for (int i = 0; i < p + kPowers; ++i) top.c[i] = fact[(kBlocks - 1) * kPowers + 1 + i];
  hipLaunchKernelGGL(top_block_kernel, ew, dim3(256), 0, s, ws, nn, stride, p + 1, offA, top);
  SETD_LAUNCHED();
  int cur = offA, nxt = offB;
  for (int b = kBlocks - 2; b >= 0; --b) {
    L.count = 0;
    for (int k = 0; k <= p; ++k) {
      Product* P = product(kPowers - 1, cur + k, nxt + k);
      P->nadd = kPowers;
      for (int i = 0; i < kPowers; ++i) {   // small terms first
        P->add[i] = kPowers - 1 - i;
        P->coef[i] = fact[k + b * kPowers + kPowers - i];
      }
      if (b == 0 && sq == 0) P->final_k = k;
    }
    SETD_TRY(launch_level(L, E, s));
    std::swap(cur, nxt);
  }
  // modified squarings
  for (int it = 0; it < sq; ++it) {
    L.count = 0;
    for (int k = 0; k <= p; ++k) {
      Product* P = product(cur, cur + k, nxt + k);
      auto add = [&](int block, DD coef) {
        P->add[P->nadd] = block;
        P->coef[P->nadd++] = coef;
      };
      add(cur + k, DD{2.0, 0.0});
      if (k >= 1) add(cur, fact[k]);
      for (int j = 1; j < k; ++j) add(cur + j, fact[k - j]);
      P->shift = k;
      if (it == sq - 1) P->final_k = k;
    }
    SETD_TRY(launch_level(L, E, s));
    std::swap(cur, nxt);
  }
  return SETD_OK;
}

}  // namespace

int phi_release_workspace(int dev, bool wait) {
  if (dev < 0 || dev >= kMaxDevices) return SETD_OK;
  std::unique_lock<std::mutex> lk(g_pool[dev].mu, std::defer_lock);
  if (wait) lk.lock();
  else if (!lk.try_lock()) return SETD_OK;
  if (g_pool[dev].p) SETD_HIP(hipFree(g_pool[dev].p));
  g_pool[dev].p = nullptr;
  g_pool[dev].bytes = 0;
  return SETD_OK;
}

int phi_batch(const double* A, int n, const double* c, int nentries, int p, double* out, hipStream_t s) {
  if (nentries <= 0) return SETD_OK;
  if (p < 0 || p > kMaxOrder) {
    set_error("phi order %d outside 0..%d", p, kMaxOrder);
    return SETD_EINVAL;
  }
  const int64_t nn = (int64_t)n * n;
  const int64_t stride = nn * (kPowers + 2 * (p + 1));   // pairs of one entry
  // entries are processed in chunks that keep the workspace below ~1 GiB
  int chunk = (int)std::max<int64_t>(1, (int64_t)(1ll << 26) / stride);
  chunk = std::min({chunk, nentries, kMaxEntries});
  const size_t nb = (size_t)round_up((int64_t)n * 8, 256);

  Workspace ws;
  SETD_TRY(ws.get(nb + (size_t)chunk * stride * sizeof(d2)));
  std::vector<double> sums(n);
  hipLaunchKernelGGL(norm1_kernel, dim3((unsigned)ceil_div(n, 4)), dim3(256), 0, s, A, n, (double*)ws.p);
  SETD_LAUNCHED();
  SETD_HIP(hipMemcpyAsync(sums.data(), ws.p, (size_t)n * sizeof(double), hipMemcpyDeviceToHost, s));
  SETD_HIP(hipStreamSynchronize(s));
  double anorm = 0.0;
  bool finite = true;
  for (double v : sums) {
    finite = finite && std::isfinite(v);
    anorm = std::max(anorm, v);
  }
  if (!finite) {
    set_error("phi: matrix has non-finite entries");
    return SETD_ENONFINITE;
  }
  for (int j = 0; j < nentries; ++j)
    if (!std::isfinite(c[j])) {
      set_error("phi: non-finite scalar argument");
      return SETD_ENONFINITE;
    }
  int rc = SETD_OK;
  for (int e0 = 0; e0 < nentries && rc == SETD_OK; e0 += chunk)
    rc = build_chunk(A, n, c + e0, std::min(chunk, nentries - e0), p, anorm, out + (int64_t)e0 * (p + 1) * nn,
                     (d2*)(ws.p + nb), stride, s);
  const hipError_t e = hipStreamSynchronize(s);   // the workspace goes back
  if (rc == SETD_OK && e != hipSuccess) {
    set_error("phi build failed: %s", hipGetErrorString(e));
    rc = SETD_EHIP;
  }
  return rc;
}

}  // namespace setd
