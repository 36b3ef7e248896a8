// Cholesky factor, its inverse and the product with a factor before it, of a small Gram matrix by one wave (device code).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace sceig {
namespace {

// Cholesky of the b x b Gram matrix in the registers of one wave: lane t owns column t of G, R and R^-1;
// values of other columns travel by lane reads.  Same dropping rule as documented in kernels.h.
// Value of lane `l` (a compile-time constant after unrolling) for the whole wave: a scalar lane read, not a trip
// through the LDS crossbar.
__device__ __forceinline__ double bcast_lane(double v, int l) {
  const long long bits = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)bits, l);
  const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// sqrt(p) and its inverse, and quotients by it, for the factorizations below: one approximate inverse root (v_rsq_f64),
// two Newton steps, then root, inverse and quotients each corrected by their own remainder, as a division does.  Half the
// dependent operations of a square root and a division, and the inverse serves the whole row and the triangular inverse
// (a launch for b = 16: 9.2 -> 7.7 us; for b = 32, bound by the fetch of its code, 38.7 -> 36.6 us).  p > 0 and normal: it has passed the drop test.
__device__ __forceinline__ void root_and_inverse(double p, double* root, double* inv) {
  double y = __builtin_amdgcn_rsq(p);
  const double h = 0.5 * p;
  y = fma(y, fma(-h * y, y, 0.5), y);
  y = fma(y, fma(-h * y, y, 0.5), y);
  double r = p * y;
  r = fma(fma(-r, r, p), 0.5 * y, r);
  *inv = fma(fma(-r, y, 1.0), y, y);
  *root = r;
}
__device__ __forceinline__ double quotient(double a, double root, double inv) {
  const double q = a * inv;
  return fma(fma(-q, root, a), inv, q);
}

// Cholesky with column drop, inverse and product with the factor before it, by one wave, lane t = column t (see
// launch_gram_cholesky): b <= 16.  g: b x b, row stride gs.  A finished row of R is taken out of all remaining rows at
// once, a finished entry of the inverse's column goes into all sums that wait for it, so that the multiply-adds of a step
// do not wait for one another.
template <int B>
__device__ __forceinline__ void chol_wave(const double* g, int gs, double* __restrict__ g_out,
                                          double* __restrict__ rinv_out, double* __restrict__ r_out,
                                          const double* __restrict__ rprev, double abs_tol2, double rel_tol) {
  const int t = threadIdx.x & 63;
  const bool act = t < B;
  const int tc = act ? t : 0;
  double gcol[B], rcol[B], ricol[B], root[B], inv[B];
  double gdiag = 0.0;  // own diagonal entry of g
#pragma unroll
  for (int q = 0; q < B; ++q) {
    const int lo = q < tc ? q : tc, hi = q < tc ? tc : q;
    gcol[q] = g[lo * gs + hi];  // upper triangle, mirrored
    gdiag = q == tc ? gcol[q] : gdiag;
    ricol[q] = 0.0;
  }
  if (g_out && act) {
#pragma unroll
    for (int q = 0; q < B; ++q) g_out[q * kPartialPad + t] = gcol[q];
  }
#pragma unroll
  for (int k = 0; k < B; ++k) {
    const double gkk = bcast_lane(gdiag, k), pk = bcast_lane(gcol[k], k);
    const bool drop = !(gkk > abs_tol2) || !(pk > rel_tol * gkk);
    root_and_inverse(drop ? 1.0 : pk, &root[k], &inv[k]);
    rcol[k] = drop || t < k ? 0.0 : (t == k ? root[k] : quotient(gcol[k], root[k], inv[k]));
#pragma unroll
    for (int q = k + 1; q < B; ++q) gcol[q] -= bcast_lane(rcol[k], q) * rcol[k];
  }
  double rcc = 0.0;  // own diagonal entry
#pragma unroll
  for (int q = 0; q < B; ++q) rcc = (q == t) ? rcol[q] : rcc;
  // ricol[r] holds the sum over the finished entries x > r of R[r][x] Rinv[x][t] until it is its turn
#pragma unroll
  for (int r = B - 1; r >= 0; --r) {
    const double rrr = bcast_lane(rcol[r], r);
    double v = 0.0;
    if (rrr != 0.0 && rcc != 0.0) v = (t == r) ? inv[r] : (t > r ? -quotient(ricol[r], root[r], inv[r]) : 0.0);
    ricol[r] = v;
#pragma unroll
    for (int x = 0; x < r; ++x) ricol[x] += bcast_lane(rcol[x], r) * v;
  }
  if (rinv_out && act) {
#pragma unroll
    for (int q = 0; q < B; ++q) rinv_out[q * kPartialPad + t] = ricol[q];
  }
  if (r_out) {
    if (rprev) {
      double v[B];
#pragma unroll
      for (int q = 0; q < B; ++q) v[q] = 0.0;
#pragma unroll
      for (int x = 0; x < B; ++x) {
        const double p = rprev[x * kPartialPad + tc];
#pragma unroll
        for (int q = 0; q <= x; ++q) v[q] += bcast_lane(rcol[q], x) * p;
      }
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (act) r_out[q * kPartialPad + t] = v[q];
    } else {
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (act) r_out[q * kPartialPad + t] = rcol[q];
    }
  }
}

}  // namespace
}  // namespace sceig
