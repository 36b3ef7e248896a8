// Cholesky factor, its inverse and the product with a factor before it, of a small Gram matrix by one wave (device code).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace sceig {
namespace {

// Value of lane `l` (the same for the whole wave) for all lanes: a scalar lane read, not a trip through the LDS crossbar.
__device__ __forceinline__ double bcast_lane(double v, int l) {
  const long long bits = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)bits, l);
  const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// sqrt(p) and its inverse, and quotients by it, for the factorization below: one approximate inverse root (v_rsq_f64),
// two Newton steps, then root, inverse and quotients each corrected by their own remainder, as a division does.  Half the
// dependent operations of a square root and a division, and the inverse serves the whole row of R and of the inverse (in
// a factorization whose rows were straight-line code, a launch for b = 16: 9.2 -> 7.7 us).  p > 0 and normal: it has
// passed the drop test.
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

// Cholesky with column drop (the rule stands at launch_gram_cholesky in kernels.h) and inverse by one wave: b <= 32.  g: b x b,
// row stride gs.  Lane t < b holds column t of what is left of G, lane b + c column c of what elimination makes of the identity:
// the same operations leave R and, row by row, the inverse of its transpose, so that the inverse takes no chain of its own.  Row k
// of both goes to LDS, rows[k][0 .. b) = R[k], rows[k][b + c] = R^-1[c][k], from where all lanes read the entries of R[k] that
// they multiply by. The columns move up by one a step, so that the loop is not unrolled: with a step per row in registers, entries by lane
// reads, the code (40 KB for b = 32) ran once and took as long as its fetch, and the inverse took as many steps again.
// A launch for b = 32: 34 us, now 17; b = 16: 7.5, now 5.8; inside the one-launch QR, b = 16: 4.6, now 2.9.
template <int B>
constexpr int kCholPitch = 2 * B + 1;  // odd: no bank conflicts along columns
template <int B>
__device__ __forceinline__ void chol_rows(const double* g, int gs, double* rows, double abs_tol2, double rel_tol) {
  const int t = threadIdx.x & 63;
  const int tc = t < B ? t : 0;
  double col[B];
  double gdiag = 0.0;  // own diagonal entry of g
#pragma unroll
  for (int q = 0; q < B; ++q) {
    const int lo = q < tc ? q : tc, hi = q < tc ? tc : q;
    const double v = g[lo * gs + hi];  // upper triangle, mirrored
    gdiag = q == tc ? v : gdiag;
    col[q] = t < B ? v : (q == t - B ? 1.0 : 0.0);
  }
  // row k of R and of the inverse, from what is left of row k of G
  auto finish = [&](double left, int k) __attribute__((always_inline)) {
    double gkk = bcast_lane(gdiag, k), pk = bcast_lane(left, k);
    asm("" : "+v"(gkk), "+v"(pk));  // vector registers: a scalar condition makes a longer chain (b = 16: 3.4 us instead of 2.9)
    const bool drop = !(gkk > abs_tol2) || !(pk > rel_tol * gkk);
    double root, inv;
    root_and_inverse(drop ? 1.0 : pk, &root, &inv);
    return drop || t < k ? 0.0 : (t == k ? root : quotient(left, root, inv));
  };
  double r = finish(col[0], 0);
#pragma unroll 1
  for (int k = 0;; ++k) {
    double* const row = rows + k * kCholPitch<B>;
    if (t < 2 * B) row[t] = r;
    if (k + 1 == B) break;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the wave's own LDS operations complete in order
    __builtin_amdgcn_wave_barrier();
    if constexpr (B > 1) {
      // the next row first, by a lane read: its root is on its way while the others wait for their factors
      double by[B];
#pragma unroll
      for (int q = 1; q < B; ++q) by[q] = row[k + q];  // from q = B - k on nothing that is used
      const double next = finish(col[1] - bcast_lane(r, k + 1) * r, k + 1);
#pragma unroll
      for (int q = 1; q < B; ++q) col[q - 1] = col[q] - by[q] * r;
      r = next;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ... and what launch_gram_cholesky gives back.  rprev's columns are read before the factorization.
template <int B>
__device__ __forceinline__ void chol_wave(const double* g, int gs, double* rows, double* __restrict__ g_out,
                                          double* __restrict__ rinv_out, double* __restrict__ r_out,
                                          const double* __restrict__ rprev, double abs_tol2, double rel_tol) {
  constexpr int LANES = B < 64 / B ? B : 64 / B;  // rows at a time
  const int t = threadIdx.x & 63, c = t % B, q0 = t / B;
  double prev[B];
  if (r_out && rprev) {
#pragma unroll
    for (int x = 0; x < B; ++x) prev[x] = rprev[x * kPartialPad + c];
  }
  if (g_out && q0 < LANES) {
    for (int q = q0; q < B; q += LANES) g_out[q * kPartialPad + c] = q < c ? g[q * gs + c] : g[c * gs + q];
  }
  chol_rows<B>(g, gs, rows, abs_tol2, rel_tol);
  if (q0 >= LANES) return;
#pragma unroll 1
  for (int q = q0; q < B; q += LANES) {
    const double* const row = rows + q * kCholPitch<B>;
    if (rinv_out) rinv_out[q * kPartialPad + c] = rows[c * kCholPitch<B> + B + q];
    if (r_out) {
      double v = row[c];
      if (rprev) {
        constexpr int CHAINS = B < 4 ? B : 4;
        double part[CHAINS] = {};
#pragma unroll
        for (int x = 0; x < B; ++x) part[x % CHAINS] += row[x] * prev[x];  // x < q: zeros
        v = part[0];
#pragma unroll
        for (int x = 1; x < CHAINS; ++x) v += part[x];
      }
      r_out[q * kPartialPad + c] = v;
    }
  }
}

}  // namespace
}  // namespace sceig
