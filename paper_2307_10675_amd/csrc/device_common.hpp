// Device helpers shared by the libifci kernels: MFMA wrappers, wavefront and
// workgroup reductions, packed-index arithmetic and the small symmetric
// eigensolver of the Davidson subspace.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ifci_internal.h"

namespace ifci {

// f(std::integral_constant<int, i>) for i = B .. E-1, unrolled at compile time
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// C(k, k/2): the most strings a k-orbital increment can have
__host__ __device__ constexpr int max_strings(int k) {
  int c = 1;
  for (int i = 1; i <= k / 2; ++i) c = c * (k - k / 2 + i) / i;
  return c;
}

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Mfma;
// 16x16x4 tiles.  Lane L holds A[L % 16][L / 16] and B[L / 16][L % 16];
// accumulator register r of lane L holds column L % 16 and row row(L / 16, r):
// 4 r + L / 16 for FP64 (v_mfma_f64_16x16x4f64), 4 (L / 16) + r for FP32
// (v_mfma_f32_16x16x4f32), as measured on gfx950.
template <>
struct Mfma<double> {
  typedef d4 acc;
  static constexpr __host__ __device__ int row(int lane_hi, int r) { return 4 * r + lane_hi; }
  static __device__ __forceinline__ acc zero() { return acc{0.0, 0.0, 0.0, 0.0}; }
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<float> {
  typedef f4 acc;
  static constexpr __host__ __device__ int row(int lane_hi, int r) { return 4 * lane_hi + r; }
  static __device__ __forceinline__ acc zero() { return acc{0.f, 0.f, 0.f, 0.f}; }
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Lane movement of a double by DPP (two 32-bit moves, no LDS traffic).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Sum over the four rows of 16 lanes (lanes equal mod 16), in each of them.
__device__ __forceinline__ double rows_sum(double v) {
#pragma clang fp contract(off)
  {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  }
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// Sum over the wavefront, the total in every lane.  Inside a row of 16 lanes
// by DPP (neighbour, pair, half-row and row mirrors), across rows by the
// gfx950 lane-row swaps: both operands of each add are the same in every
// lane of a group, so all lanes hold the same bits.  (Through __shfl_xor a
// step is two ds_bpermute and a wait on LDS: in the on-chip Davidson the
// wave sums of its overlaps took 18k of an iteration's 108k cycles at 6
// orbitals.)
__device__ __forceinline__ double wave_sum(double v) {
  // no contraction with a product passed in: fma(x, y, moved x y) is not the
  // same number in the two lanes of a pair
#pragma clang fp contract(off)
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);  // row_half_mirror: the other quad of the half row
  v += dpp_f64<0x140>(v);  // row_mirror: the other half row
  return rows_sum(v);
}

// Sum NV values over the workgroup; every thread gets the totals in out[].
// Deterministic: fixed butterfly inside each wave, waves added in order.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* red, double* out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int j = 0; j < NV; ++j) v[j] = wave_sum(v[j]);
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < NV; ++j) red[wave * NV + j] = v[j];
  __syncthreads();
  if (threadIdx.x < NV) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w * NV + threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

// Same sums with one barrier: every thread adds the per-wave partials itself
// (in the same fixed order) and gets the totals back in v[].  `red` holds two
// buffers of 128 doubles (8 waves x NV <= 16) used alternately (`parity`
// flips each call), so a call never overwrites partials that a slower
// thread may still be reading from the call before.
template <int NV>
__device__ __forceinline__ void block_sum_1b(double (&v)[NV], double* red, int& parity) {
  static_assert(NV <= 16, "two buffers of 8 waves x 16 values");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  double* buf = red + parity * 128;
  parity ^= 1;
#pragma unroll
  for (int j = 0; j < NV; ++j) v[j] = wave_sum(v[j]);
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < NV; ++j) buf[wave * NV + j] = v[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += buf[w * NV + j];
    v[j] = s;
  }
}

// Packed upper-triangle index: entry (a, b), a <= b, lives at b (b + 1) / 2 + a.
__device__ __forceinline__ int64_t packed(int64_t a, int64_t b) {
  return a <= b ? tri(b) + a : tri(a) + b;
}
// 32-bit variant for indices below 2^24 (single-precision square root, then
// an exact integer correction).
__device__ __forceinline__ void unpack32(int i, int* a, int* b) {
  int c = (int)((__builtin_sqrtf(8.0f * (float)i + 1.0f) - 1.0f) * 0.5f);
  if (((c + 1) * (c + 2)) / 2 <= i) ++c;
  if ((c * (c + 1)) / 2 > i) --c;
  *b = c;
  *a = i - (c * (c + 1)) / 2;
}
__device__ __forceinline__ void unpack(int64_t i, int* a, int* b) {
  int64_t c = (int64_t)((sqrt(8.0 * (double)i + 1.0) - 1.0) * 0.5);
  while (tri(c + 1) <= i) ++c;
  while (tri(c) > i) --c;
  *b = (int)c;
  *a = (int)(i - tri(c));
}

// Atomic add into LDS (ds_add_f64).  The pointer must point into LDS.
typedef __attribute__((address_space(3))) double lds_double;
__device__ __forceinline__ void lds_add(double* p, double v) {
  __atomic_fetch_add((lds_double*)p, v, __ATOMIC_RELAXED);
}

constexpr double kSqrt2 = 1.4142135623730950488;
constexpr double kRSqrt2 = 0.70710678118654752440;

// Value v of lane `k` (a constant) in every lane, as scalars.
__device__ __forceinline__ double lane_f64(double v, int k) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k),
                          __builtin_amdgcn_readlane(__double2loint(v), k));
}

// 1 / x to rounding for normal x: the hardware reciprocal and two Newton steps.
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// Largest value over the wavefront, in every lane (steps as in wave_sum).
__device__ __forceinline__ float wave_max(float v) {
  auto dpp = [](float x, auto c) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(c)::value, 0xf, 0xf, true));
  };
  v = fmaxf(v, dpp(v, std::integral_constant<int, 0xB1>{}));
  v = fmaxf(v, dpp(v, std::integral_constant<int, 0x4E>{}));
  v = fmaxf(v, dpp(v, std::integral_constant<int, 0x141>{}));
  v = fmaxf(v, dpp(v, std::integral_constant<int, 0x140>{}));
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
  v = fmaxf(__int_as_float(a[0]), __int_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
  return fmaxf(__int_as_float(b[0]), __int_as_float(b[1]));
}

// Lowest eigenpair of the symmetric n x n matrix G (row stride 16, n <= 16)
// of a Davidson subspace, from the secular function of one taken-out index.
// With index p taken out, G = [[g, b^T], [b, B]]; below the lowest eigenvalue
// of B,
//   s(x) = g - x - b^T (B - x)^-1 b
// is decreasing and concave and its one root is the lowest eigenvalue of G,
// with eigenvector (1, -w), w = (B - x)^-1 b.  B - x0 is eliminated once
// (Gauss-Jordan in registers, lane i holding row i, pivot rows passed as
// scalars, the multipliers kept), w_0 = (B - x0)^-1 b, w_1 = (B - x0)^-1 w_0
// and w_2 give s to fifth order and w to second order around x0; the root is
// taken from that expansion, and where the step is too long for it (more than
// 2e-5 of the distance to the spectrum of B) the expansion is repeated about
// the new x0.  The first x0 is the lowest eigenvalue of G between the
// previous subspace's eigenvector (yp, eigenvalue tp, over the first n - 1
// indices) and the new basis vector: an upper bound that is close once the
// iteration converges, so that most calls eliminate once.  p is the largest
// component of yp, which keeps B - x0 far from singular.  There is no
// pivoting; a pivot that is not clearly positive means x0 is not (safely)
// below the spectrum of B, and the call returns -1 with nothing written.
// Otherwise it returns the index of the largest component of y (the p of the
// next call).  Executed by one full wavefront, with LDS arguments; y may be
// yp.  NN >= n is the compile-time size the elimination is unrolled to (the
// padding rows are decoupled): a test of every index against n costs as much
// again as the arithmetic.  (In place of a full Jacobi decomposition per iteration, warm started
// from the previous subspace, which took 56k cycles of an on-chip iteration's
// 108k at 6 orbitals.)
template <int NN>
__device__ __forceinline__ int lowest_pair_n(const double* G, int n, int p, double tp, const double* yp, double* theta,
                                             double* y) {
  const int lane = threadIdx.x & 63;
  auto at = [&](int i) { return i == 0 ? p : (i == p ? 0 : i); };
  double row[NN];
  const int ri = at(lane < n ? lane : 0);
#pragma unroll
  for (int j = 0; j < NN; ++j) {
    const double v = G[ri * 16 + at(j < n ? j : 0)];
    row[j] = lane < n && j < n ? v : 0.0;
  }
  const double gl = lane < n - 1 ? G[lane * 16 + n - 1] * yp[lane] : 0.0;
  const double gam = G[(n - 1) * 17];
  const double g = lane_f64(row[0], 0);
  const double b = lane > 0 && lane < n ? row[0] : 0.0;
  const double dg = lane < n ? G[ri * 17] : 0.0;
  // size of the diagonal and the border: the scale rounding is measured in
  const double scale = wave_sum(fabs(dg) + fabs(b));
  const double beta = wave_sum(gl);
  const double h = 0.5 * (gam - tp);
  const double q = sqrt(h * h + beta * beta);
  double x = h >= 0.0 ? (q > 0.0 ? tp - beta * beta / (h + q) : tp) : 0.5 * (tp + gam) - q;
  const double floor_p = 1e-7 * scale;
  double w = 0.0, ww = 0.0;
  for (int it = 0;; ++it) {
    if (it == 12) return -1;
    double a[NN], f[NN], w0 = b, own = 0.0, low = scale;
#pragma unroll
    for (int j = 1; j < NN; ++j) a[j] = lane == j ? (j < n ? row[j] - x : scale) : row[j];
#pragma unroll
    for (int k = 1; k < NN; ++k) {
      const double pk = lane_f64(a[k], k);
      low = pk > low ? low : pk;  // a NaN stays
      const double inv = fast_rcp(pk);
      f[k] = lane == k ? 0.0 : a[k] * inv;
      own = lane == k ? inv : own;
      w0 = __builtin_fma(-f[k], lane_f64(w0, k), w0);
#pragma unroll
      for (int j = k + 1; j < NN; ++j) a[j] = __builtin_fma(-f[k], lane_f64(a[j], k), a[j]);
    }
    if (!(low > floor_p)) return -1;
    auto solve = [&](double r) -> double {
#pragma unroll
      for (int k = 1; k < NN; ++k) r = __builtin_fma(-f[k], lane_f64(r, k), r);
      return r * own;
    };
    w0 *= own;
    const double w1 = solve(w0), w2 = solve(w1);
    const double c0 = wave_sum(b * w0), c1 = wave_sum(w0 * w0), c2 = wave_sum(w0 * w1), c3 = wave_sum(w1 * w1),
                 c4 = wave_sum(w1 * w2), c5 = wave_sum(w2 * w2);
    const double s0 = g - x - c0;
    // the root of s0 - d - c1 d - c2 d^2 - ... by Newton's method from d = 0
    double d = s0 * fast_rcp(1.0 + c1);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const double v = s0 - d * (1.0 + c1 + d * (c2 + d * (c3 + d * (c4 + d * c5))));
      const double dv = 1.0 + c1 + d * (2.0 * c2 + d * (3.0 * c3 + d * (4.0 * c4 + d * 5.0 * c5)));
      d = dv > 0.0 ? d + v * fast_rcp(dv) : d;
    }
    // |d| over the distance to the spectrum of B that b sees
    const double rho = fabs(d) * c5;
    if (rho <= 2e-5 * c4 || fabs(d) <= 1e-15 * scale) {
      w = __builtin_fma(d, __builtin_fma(d, w2, w1), w0);
      ww = wave_sum(w * w);
      x += d;
      break;
    }
    // too long a step: the first-order one stays right of the root
    const double d1 = s0 * fast_rcp(1.0 + c1);
    x += rho <= 0.3 * c4 ? d : d1;
  }
  const double inv = 1.0 / sqrt(1.0 + ww);
  const double yl = lane == 0 ? inv : (lane < n ? -w * inv : 0.0);
  if (lane < n) y[at(lane)] = yl;
  if (lane == 0) *theta = x;
  const float m = fabsf((float)yl);
  const int big = __ffsll((unsigned long long)__ballot(m == wave_max(m))) - 1;
  __builtin_amdgcn_wave_barrier();
  return at(big);
}

__device__ inline int lowest_pair(const double* G, int n, int p, double tp, const double* yp, double* theta,
                                  double* y) {
  if (n == 1) {
    if ((threadIdx.x & 63) == 0) {
      y[0] = 1.0;
      *theta = G[0];
    }
    __builtin_amdgcn_wave_barrier();
    return 0;
  }
  if (n <= 4) return lowest_pair_n<4>(G, n, p, tp, yp, theta, y);
  if (n <= 8) return lowest_pair_n<8>(G, n, p, tp, yp, theta, y);
  if (n <= 12) return lowest_pair_n<12>(G, n, p, tp, yp, theta, y);
  return lowest_pair_n<16>(G, n, p, tp, yp, theta, y);
}

// Eigen-decomposition of the symmetric n x n matrix A (row stride 16,
// n <= 16) by parallel cyclic Jacobi (Golub & Van Loan, symmetric Schur
// rotations in the Brent-Luk circle ordering), accumulating the rotations
// into Q (stride 16), which the caller initialises (identity, or
// eigenvectors of a previous nearby matrix to warm start).  An odd n is
// padded with a decoupled index whose diagonal entry lies far above the
// spectrum (its row and column of A and Q are overwritten).  Each round
// rotates N / 2 disjoint planes at once: lane L updates the 2 x 2 block
// (L / 8, L % 8) of A and rows L / 8 and L / 8 + 8 of Q in plane L % 8, with
// the rotations of its two planes formed by itself.
// Pivots below 1e-15 ||A||_F are not rotated (FP64 rounding keeps
// regenerating off-diagonal noise near 1e-16 ||A||); sweeps stop after one
// whose pivots times angles (the sizes of both sums of squares) are below 1e-17
// ||A||_F: a sweep leaves no more than that of the off-diagonal part.  (The
// pivots alone do not tell: where eigenvalues lie as close to each other as the
// pivots are large, the angles are not small and what is left is of the
// pivots' own size.)  Executed by one
// full wavefront, which orders its own LDS accesses, so no workgroup
// barrier is needed.  Returns the sorted eigenvalues in evals, their
// columns of Q in perm, and the lowest pair in theta / y.
__device__ inline void jacobi_warm(double* A, double* Q, int n, double* theta, double* y, double* evals,
                                   int* perm) {
  const int lane = threadIdx.x & 63;
  const int N = n + (n & 1), H = N >> 1, m = N - 1;
  __builtin_amdgcn_wave_barrier();
  double f2 = 0.0;
  if (lane < n)
    for (int j = 0; j < n; ++j) f2 += A[lane * 16 + j] * A[lane * 16 + j];
  f2 = wave_sum(f2);
  if (n & 1) {
    // decoupled padding index n
    const double big = 1e3 * (1.0 + sqrt(f2));
    if (lane < 16) {
      A[lane * 16 + n] = (lane == n) ? big : 0.0;
      A[n * 16 + lane] = (lane == n) ? big : 0.0;
      Q[lane * 16 + n] = (lane == n) ? 1.0 : 0.0;
      Q[n * 16 + lane] = (lane == n) ? 1.0 : 0.0;
    }
  }
  __builtin_amdgcn_wave_barrier();
  const double tol = 1e-15 * sqrt(f2);
  const int kr = lane >> 3, kc = lane & 7;
  const bool blk = kr < H && kc < H;
  // plane k of round s holds (m, s) for k = 0, else (s + k, s - k) mod m
  auto first = [&](int k) { return k == 0 ? m : k; };
  auto other = [&](int k) { return k == 0 ? 0 : m - k; };
  auto next = [&](int v) { return v + 1 == m ? 0 : v + 1; };
  for (int sweep = 0; sweep < 12 && N > 1; ++sweep) {
    double piv2 = 0.0, ang2 = 0.0;
    int x1 = first(kr < H ? kr : 0), y1 = other(kr < H ? kr : 0);
    int x2 = first(kc < H ? kc : 0), y2 = other(kc < H ? kc : 0);
    for (int s = 0; s < m; ++s) {
      // every lane forms the rotations of its own row and column plane: one
      // round of loads, no lane exchange
      const int p1 = x1 < y1 ? x1 : y1, q1 = x1 < y1 ? y1 : x1;
      const int p2 = x2 < y2 ? x2 : y2, q2 = x2 < y2 ? y2 : x2;
      const double pp1 = A[p1 * 17], qq1 = A[q1 * 17], pq1 = A[p1 * 16 + q1];
      const double pp2 = A[p2 * 17], qq2 = A[q2 * 17], pq2 = A[p2 * 16 + q2];
      const double a = A[p1 * 16 + p2], b = A[p1 * 16 + q2], e = A[q1 * 16 + p2], f = A[q1 * 16 + q2];
      const int i0 = kr < N ? kr : 0, i1 = kr + 8 < N ? kr + 8 : 0;
      const double u0 = Q[i0 * 16 + p2], v0 = Q[i0 * 16 + q2], u1 = Q[i1 * 16 + p2], v1 = Q[i1 * 16 + q2];
      auto rotation = [&](double app, double aqq, double apq, double& c, double& sn) {
        // tangent of the angle in single precision, then one Newton step on
        // apq (t^2 - 1) + (aqq - app) t = 0, whose slope is 2 apq (t + tau) =
        // +-2 apq sqrt(tau^2 + 1): 1e-14 of the pivot is left; c and s are
        // normalised to FP64 rounding, which keeps Q orthogonal
        const double d = aqq - app, ra = __builtin_amdgcn_rcp(apq);
        const float tau = (float)(d * 0.5 * ra);
        const float u = fmaf(tau, tau, 1.0f), ru = __builtin_amdgcn_rsqf(u);
        double t = (double)copysignf(__builtin_amdgcn_rcpf(fmaf(u, ru, fabsf(tau))), tau);
        t -= fma(apq, fma(t, t, -1.0), d * t) * (0.5 * ra * (double)copysignf(ru, tau));
        t = fabs(apq) > tol ? t : 0.0;
        const double h = fma(t, t, 1.0);
        c = __builtin_amdgcn_rsq(h);
        c = fma(0.5 * c, fma(-h * c, c, 1.0), c);
        c = fma(0.5 * c, fma(-h * c, c, 1.0), c);
        sn = t * c;
      };
      double c1, s1, c2, s2;
      rotation(pp1, qq1, pq1, c1, s1);
      rotation(pp2, qq2, pq2, c2, s2);
      if (kr == 0 && kc < H) {
        piv2 += pq2 * pq2;
        ang2 += s2 * s2;
      }
      if (kr > 0) x1 = next(x1);
      y1 = next(y1);
      if (kc > 0) x2 = next(x2);
      y2 = next(y2);
      __builtin_amdgcn_wave_barrier();
      if (blk) {
        const double a1 = c2 * a - s2 * b, b1 = s2 * a + c2 * b;
        const double e1 = c2 * e - s2 * f, f1 = s2 * e + c2 * f;
        A[p1 * 16 + p2] = c1 * a1 - s1 * e1;
        A[q1 * 16 + p2] = s1 * a1 + c1 * e1;
        A[p1 * 16 + q2] = c1 * b1 - s1 * f1;
        A[q1 * 16 + q2] = s1 * b1 + c1 * f1;
      }
      if (kc < H) {
        if (kr < N) {
          Q[i0 * 16 + p2] = c2 * u0 - s2 * v0;
          Q[i0 * 16 + q2] = s2 * u0 + c2 * v0;
        }
        if (kr + 8 < N) {
          Q[i1 * 16 + p2] = c2 * u1 - s2 * v1;
          Q[i1 * 16 + q2] = s2 * u1 + c2 * v1;
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
    if (!(wave_sum(piv2) * wave_sum(ang2) > 1e-34 * f2)) break;
  }
  __builtin_amdgcn_wave_barrier();
  // eigenvalues in increasing order (ties by index): perm[i] is the column
  // of Q holding the i-th lowest; lane j finds the rank of eigenvalue j
  if (lane < n) {
    const double vj = A[lane * 16 + lane];
    int rank = 0;
    for (int i = 0; i < n; ++i) {
      const double vi = A[i * 16 + i];
      rank += (vi < vj || (vi == vj && i < lane)) ? 1 : 0;
    }
    perm[rank] = lane;
    evals[rank] = vj;
    if (rank == 0) *theta = vj;
  }
  __builtin_amdgcn_wave_barrier();
  if (lane < n) y[lane] = Q[lane * 16 + perm[0]];
  __builtin_amdgcn_wave_barrier();
}

// Cold-start variant: Q = I, then jacobi_warm.
__device__ inline void jacobi_lowest(double* A, double* Q, int n, double* theta, double* y, double* evals,
                                     int* perm) {
  const int lane = threadIdx.x & 63;
  if (lane < 16)
    for (int j = 0; j < 16; ++j) Q[lane * 16 + j] = (lane == j) ? 1.0 : 0.0;
  jacobi_warm(A, Q, n, theta, y, evals, perm);
}

}  // namespace ifci
