// k-nearest-neighbour similarity graph (paper Section III-A: two points are connected if either is among the k most
// similar points of the other), device kernels: exact brute-force search by Euclidean distance and the list of the
// graph's undirected edges.
//
// Search.  The distance that ranks the neighbours is the plain sum of squared coordinate differences in coordinate
// order (the |x|^2 + |y|^2 - 2xy expansion loses digits to cancellation), and equal distances are ranked by index,
// so the result is unique.  Up to 128 coordinates the expansion is still used, on the matrix cores, but only to screen
// the candidates: in bf16 parts with a bound of the error (screen_kernel), in fp64 for what that cannot settle and for
// small sets (knn_mfma_kernel); beyond, a vector kernel computes every distance directly (knn_search_kernel: one
// thread per query, the query's coordinates in LDS, the candidates' read with wave-uniform addresses from a
// zero-padded copy, four candidates in flight).  Either way a query keeps its k best so far in LDS together with the
// worst of them; a candidate that beats the worst replaces it and the worst is found again by a scan of the k slots,
// which after the first few hundred candidates happens rarely.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/device/device_select.hpp>
#include <rocprim/functional.hpp>
#include <rocprim/iterator/counting_iterator.hpp>

#include <cstdint>

#include "exchange.h"
#include "kernels.h"

typedef double d4 __attribute__((ext_vector_type(4)));
#define MFMA_F64(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64((a), (b), (c), 0, 0, 0)

namespace sceig {
namespace {

constexpr int kT = 256;
constexpr int kQ = 128;  // queries per workgroup of the search
constexpr int kJU = 4;   // candidates in flight (the asm statements that pin the order name four sums)
constexpr int kDC = 8;   // coordinates per piece (rows are padded to a multiple of it)
inline unsigned blocks(int64_t n) { return (unsigned)((n + kT - 1) / kT); }

__global__ __launch_bounds__(kT) void pad_rows_kernel(const double* __restrict__ x, int64_t ldx, int64_t n, int d,
                                                      int dp, double* __restrict__ xp) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (e >= n * dp) return;
  const int64_t i = e / dp;
  const int t = (int)(e - i * dp);
  xp[e] = t < d ? x[i * ldx + t] : 0.0;
}

__global__ __launch_bounds__(kQ) void knn_search_kernel(const double* __restrict__ xp, int64_t n, int dp, int k,
                                                        int32_t* __restrict__ idx_out,
                                                        double* __restrict__ dist_out) {
  extern __shared__ double lds[];
  double* qs = lds;                                              // [dp][kQ]  the queries, one column per thread
  double* bd = qs + (size_t)dp * kQ;                             // [k][kQ]   squared distances of the best so far
  int32_t* bi = reinterpret_cast<int32_t*>(bd + (size_t)k * kQ); // [k][kQ]   their indices
  const int tid = threadIdx.x;
  const int64_t i = (int64_t)blockIdx.x * kQ + tid;
  const bool live = i < n;
  // every thread touches only its own column of the three arrays: no barrier anywhere in this kernel
  for (int t = 0; t < dp; ++t) qs[t * kQ + tid] = live ? xp[i * dp + t] : 0.0;
  for (int s = 0; s < k; ++s) {
    bd[s * kQ + tid] = INFINITY;
    bi[s * kQ + tid] = INT32_MAX;
  }
  // the worst of the kept candidates: (thr, thr_idx) in slot thr_slot; a dead lane accepts nothing
  double thr = live ? INFINITY : -1.0;
  int32_t thr_idx = INT32_MAX;
  int thr_slot = 0;
  for (int64_t j0 = 0; j0 < n; j0 += kJU) {
    const double* __restrict__ y[kJU];
#pragma unroll
    for (int u = 0; u < kJU; ++u) y[u] = xp + (j0 + u < n ? j0 + u : n - 1) * dp;  // uniform over the workgroup
    double acc[kJU];
#pragma unroll
    for (int u = 0; u < kJU; ++u) acc[u] = 0.0;
    for (int c = 0; c < dp; c += kDC) {
#pragma unroll
      for (int t = 0; t < kDC; ++t) {
        const double qv = qs[(c + t) * kQ + tid];
#pragma unroll
        for (int u = 0; u < kJU; ++u) {
          const double df = qv - y[u][c + t];
          acc[u] = fma(df, df, acc[u]);
        }
        asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));  // the four sums advance together
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // the sums stay in front of the tests
#pragma unroll
    for (int u = 0; u < kJU; ++u) {
      const int64_t j = j0 + u;
      const bool pass = (j < n) & (j != i) & ((acc[u] < thr) | ((acc[u] == thr) & ((int32_t)j < thr_idx)));
      if (pass) {  // bitwise, not short-circuit: the sums must not be moved behind a test of j
        bd[thr_slot * kQ + tid] = acc[u];
        bi[thr_slot * kQ + tid] = (int32_t)j;
        thr = -1.0;
        for (int s = 0; s < k; ++s) {
          const double v = bd[s * kQ + tid];
          const int32_t id = bi[s * kQ + tid];
          if (v > thr || (v == thr && id > thr_idx)) {
            thr = v;
            thr_idx = id;
            thr_slot = s;
          }
        }
      }
    }
  }
  if (!live) return;
  // nearest first (ties: lower index first): selection sort of the k slots
  for (int a = 0; a < k; ++a) {
    int best = a;
    double bv = bd[a * kQ + tid];
    int32_t bid = bi[a * kQ + tid];
    for (int s = a + 1; s < k; ++s) {
      const double v = bd[s * kQ + tid];
      const int32_t id = bi[s * kQ + tid];
      if (v < bv || (v == bv && id < bid)) {
        best = s;
        bv = v;
        bid = id;
      }
    }
    bd[best * kQ + tid] = bd[a * kQ + tid];
    bi[best * kQ + tid] = bi[a * kQ + tid];
    bd[a * kQ + tid] = bv;
    bi[a * kQ + tid] = bid;
    idx_out[i * k + a] = bid == INT32_MAX ? -1 : bid;
    dist_out[i * k + a] = sqrt(bv);
  }
}

// xn[i] = sum_t xp[i][t]^2 in coordinate order
__global__ __launch_bounds__(kT) void row_norms_kernel(const double* __restrict__ xp, int64_t n, int dp,
                                                       double* __restrict__ xn) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  double acc = 0.0;
  for (int t = 0; t < dp; ++t) acc = fma(xp[i * dp + t], xp[i * dp + t], acc);
  xn[i] = acc;
}

// The search with the cross term on the matrix cores.  |q - y|^2 = |q|^2 + |y|^2 - 2 q.y, and q.y over 64 queries x
// 64 candidates is a dense contraction: a workgroup of four waves owns 64 queries, wave w the 16 x 64 block of its 16
// queries, as 16x16x4 fp64 MFMAs with the queries' coordinates resident in registers and the candidates' loaded with
// 16-byte loads one step ahead.  The expanded form loses digits to cancellation, so it only screens: a candidate
// whose approximate squared distance lies below the query's threshold (the k-th best exact distance so far) plus a
// bound of the rounding error, kMarginUlps * 2^-53 * (|q|^2 + |y|^2), gets a bit in an LDS mask, and every kRound
// steps one thread per query walks its bits, computes the exact distance as the plain sum of squared differences in
// coordinate order and keeps the k best by (distance, index) exactly as the other kernels do.  The thresholds the
// screen uses are those of the last walk: they only ever shrink, so a lagging threshold lets more candidates
// through, never fewer; the result is the exact one.
// Error bound: both norms carry a relative error of dp * u (u = 2^-53), the dot product an absolute error of
// dp * u * |q||y| <= dp * u * (|q|^2 + |y|^2) / 2, the two final additions 2u more of the terms' size: together
// below (2 dp + 3) u (|q|^2 + |y|^2); the margin is twice that and more.
constexpr int kMq = 64;      // queries per workgroup
constexpr int kMt = 256;     // threads
constexpr int kRound = 2;    // steps of 64 candidates between two walks of the masks
template <int DP>
__global__ __launch_bounds__(kMt) __attribute__((amdgpu_waves_per_eu(DP <= 32 ? 3 : 2))) void knn_mfma_kernel(
    const double* __restrict__ xp, const double* __restrict__ xn, int64_t n, int k, const int32_t* __restrict__ tiles,
    const double* __restrict__ bound, int32_t* __restrict__ idx_out, double* __restrict__ dist_out) {
  constexpr int NS = DP / 4;            // MFMAs per 16 x 16 block
  // coordinates per piece of a step (the B operands of one piece are in flight).  Up to 32 coordinates the pieces are
  // 16 wide, which fits three waves per SIMD without spills (28 instead of 30 ms on 100,000 points of 32 coordinates:
  // three rounds of workgroups instead of four); at 128 coordinates three waves spill and lose (2.08 against 1.93 s
  // on 500,000 points), so the wider kernels keep 32-wide pieces and two waves.
  constexpr int KC = DP <= 32 ? (DP < 16 ? DP : 16) : 32;
  constexpr int NCH = DP / KC;           // pieces per step: 1, 2 or 4
  constexpr int NSC = KC / 4;            // MFMAs per block and piece
  constexpr double kMargin = (4.0 * DP + 16.0) * 1.1102230246251565e-16;
  extern __shared__ double lds[];
  double* bd = lds;                                   // [k][kMq]
  double* thrq = bd + (size_t)k * kMq;                // [kMq]      thresholds of the last walk
  unsigned long long* mask = reinterpret_cast<unsigned long long*>(thrq + kMq);  // [kRound][kMq]
  int32_t* bi = reinterpret_cast<int32_t*>(mask + kRound * kMq);                 // [k][kMq]
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63, i = lane & 15, g = lane >> 4;
  const int64_t q0 = (int64_t)(tiles ? tiles[blockIdx.x] : (int32_t)blockIdx.x) * kMq;
  const double2* __restrict__ xp2 = reinterpret_cast<const double2*>(xp);

  // setup: lists, thresholds, masks
  for (int e = tid; e < k * kMq; e += kMt) {
    bd[e] = INFINITY;
    bi[e] = INT32_MAX;
  }
  for (int e = tid; e < kRound * kMq; e += kMt) mask[e] = 0ull;
  // bound (may be null): per query a squared distance that at least k others do not exceed; a query past the end lets
  // nothing through
  if (tid < kMq) thrq[tid] = q0 + tid < n ? (bound ? bound[q0 + tid] : INFINITY) : -INFINITY;
  // this lane's part of the A operand: query 16 wave + i, coordinates 8m + 2g, 8m + 2g + 1
  double a[NS];
  {
    const int64_t qrow = q0 + 16 * wave + i < n ? q0 + 16 * wave + i : n - 1;
#pragma unroll
    for (int m = 0; m < NS / 2; ++m) {
      const double2 v = xp2[(qrow * DP + 8 * m + 2 * g) / 2];
      a[2 * m] = v.x;
      a[2 * m + 1] = v.y;
    }
  }
  // the queries whose results this lane holds after an MFMA: 16 wave + 4 rr + g
  double qn[4];
  int64_t qidx[4];
#pragma unroll
  for (int rr = 0; rr < 4; ++rr) {
    qidx[rr] = q0 + 16 * wave + 4 * rr + g;
    qn[rr] = qidx[rr] < n ? xn[qidx[rr]] : 0.0;
  }
  // the walking lanes' state: lanes 0..15 of every wave, one of the wave's queries each.  A wave screens and walks
  // on its own: after the setup no barrier joins the four waves, so one wave's walk does not hold up the others.
  const int myql = 16 * wave + lane;  // meaningful for lane < 16
  const int64_t myq = q0 + myql;
  const double cut = bound && lane < 16 && myq < n ? bound[myq] : INFINITY;
  double thr = cut;
  int32_t thr_idx = INT32_MAX;
  int thr_slot = 0;
  __syncthreads();

  const int64_t nstep = (n + 63) / 64;
  double2 b0[4][NSC / 2], b1[4][NSC / 2];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    const int64_t c = 16 * cb + i < n ? 16 * cb + i : n - 1;
#pragma unroll
    for (int m = 0; m < NSC / 2; ++m) b0[cb][m] = xp2[(c * DP + 8 * m + 2 * g) / 2];
  }
  d4 acc[4];
  double yn[4];
  // one piece (KC coordinates) of a step of 64 candidates: operands in bcur, the next piece's are fetched into bnxt
  auto do_piece = [&](double2 (&bcur)[4][NSC / 2], double2 (&bnxt)[4][NSC / 2], int64_t step, int kc)
                      __attribute__((always_inline)) {
    const int64_t c0 = step * 64;
    {  // the next piece: the next coordinates of this step, or the first of the next step.  Rows are clamped to the
       // last one: straight-line loads, masked out by the index test of the screen.
      const int kcn = kc + 1 < NCH ? kc + 1 : 0;
      const int64_t cn = kc + 1 < NCH ? c0 : c0 + 64;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        int64_t c = cn + 16 * cb + i;
        c = c < n ? c : n - 1;
#pragma unroll
        for (int m = 0; m < NSC / 2; ++m) bnxt[cb][m] = xp2[(c * DP + kcn * KC + 8 * m + 2 * g) / 2];
      }
    }
    if (kc == 0) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        acc[cb] = (d4){0.0, 0.0, 0.0, 0.0};
        const int64_t c = c0 + 16 * cb + i;
        yn[cb] = xn[c < n ? c : n - 1];  // used after the step's MFMAs
      }
    }
    // four independent accumulators between two MFMAs on the same one
#pragma unroll
    for (int m = 0; m < NSC / 2; ++m) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[cb] = MFMA_F64(a[kc * NSC + 2 * m], bcur[cb][m].x, acc[cb]);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[cb] = MFMA_F64(a[kc * NSC + 2 * m + 1], bcur[cb][m].y, acc[cb]);
    }
    if (kc != NCH - 1) return;
    const int sr = (int)(step % kRound);
    // only the last step has candidates past the end, only the step with the workgroup's own rows a query's self
    const bool edge = (c0 + 64 > n) | ((c0 < q0 + kMq) & (c0 + 64 > q0));  // uniform
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int ql = 16 * wave + 4 * rr + g;
      const double tq = thrq[ql];
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const double sum = qn[rr] + yn[cb];
        const double d2 = fma(-2.0, acc[cb][rr], sum);
        bool pass = d2 < fma(kMargin, sum, tq);
        if (edge) {
          const int64_t c = c0 + 16 * cb + i;
          pass = pass & (c < n) & (c != qidx[rr]);
        }
        if (pass) atomicOr(&mask[sr * kMq + ql], 1ull << (16 * cb + i));
      }
    }
    if (sr == kRound - 1 || step == nstep - 1) {  // uniform
      // the wave's own LDS operations complete in order; the fence keeps the compiler from moving them
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (lane < 16 && myq < n) {
        const int cq = myql;   // this lane's column of the per-query arrays
        const int64_t cbase = (step - sr) * 64;
        for (int st = 0; st <= sr; ++st) {
          unsigned long long mbits = mask[st * kMq + cq];
          mask[st * kMq + cq] = 0ull;
          while (mbits) {
            const int bit = __ffsll((long long)mbits) - 1;
            mbits &= mbits - 1;
            const int64_t j = cbase + st * 64 + bit;
            double ex = 0.0;
            const double2* __restrict__ qr = xp2 + myq * (DP / 2);
            const double2* __restrict__ yr = xp2 + j * (DP / 2);
#pragma unroll 8
            for (int t = 0; t < DP / 2; ++t) {  // rarely run: kept small, the registers belong to the MFMA loop
              const double2 qv = qr[t], yv = yr[t];
              const double d0 = qv.x - yv.x;
              ex = fma(d0, d0, ex);
              const double d1 = qv.y - yv.y;
              ex = fma(d1, d1, ex);
            }
            if (ex < thr || (ex == thr && (int32_t)j < thr_idx)) {
              bd[thr_slot * kMq + cq] = ex;
              bi[thr_slot * kMq + cq] = (int32_t)j;
              double w = -1.0;
              int32_t wid = INT32_MAX;
              int ws = 0;
              for (int s = 0; s < k; ++s) {
                const double x = bd[s * kMq + cq];
                const int32_t id = bi[s * kMq + cq];
                if (x > w || (x == w && id > wid)) {
                  w = x;
                  wid = id;
                  ws = s;
                }
              }
              thr = w < cut ? w : cut;
              thr_idx = w < cut ? wid : INT32_MAX;
              thr_slot = ws;
            }
          }
        }
        thrq[cq] = thr;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };
  if constexpr (NCH == 1) {
    for (int64_t step = 0; step < nstep; step += 2) {
      do_piece(b0, b1, step, 0);
      if (step + 1 < nstep) do_piece(b1, b0, step + 1, 0);
    }
  } else {  // an even number of pieces per step: every step starts on b0
    for (int64_t step = 0; step < nstep; ++step) {
#pragma unroll
      for (int kc = 0; kc < NCH; kc += 2) {
        do_piece(b0, b1, step, kc);
        do_piece(b1, b0, step, kc + 1);
      }
    }
  }
  if (lane >= 16 || myq >= n) return;
  const int tidq = myql;
  for (int aidx = 0; aidx < k; ++aidx) {  // nearest first (ties: lower index first): selection sort of the k slots
    int best = aidx;
    double bv = bd[aidx * kMq + tidq];
    int32_t bid = bi[aidx * kMq + tidq];
    for (int s = aidx + 1; s < k; ++s) {
      const double x = bd[s * kMq + tidq];
      const int32_t id = bi[s * kMq + tidq];
      if (x < bv || (x == bv && id < bid)) {
        best = s;
        bv = x;
        bid = id;
      }
    }
    bd[best * kMq + tidq] = bd[aidx * kMq + tidq];
    bi[best * kMq + tidq] = bi[aidx * kMq + tidq];
    bd[aidx * kMq + tidq] = bv;
    bi[aidx * kMq + tidq] = bid;
    idx_out[myq * k + aidx] = bid == INT32_MAX ? -1 : bid;
    dist_out[myq * k + aidx] = sqrt(bv);
  }
}

// ---- the bf16 screen ---------------------------------------------------------------------------------------------
// Up to 128 coordinates and from kScreenMinN points on, the candidates are screened twice on the bf16 matrix cores,
// which are 32 times as fast as the fp64 ones, and only what survives is looked at in fp64.  With
//   v(q, y) = q.y - |y|^2 / 2      ( |q - y|^2 = |q|^2 - 2 v, so the nearest are the candidates of largest v )
// the first pass (screen_kernel<., ., false>) leaves for every query the largest v of each of `groups` classes of
// candidates (class = index mod 16 and number of the candidate's tile mod `slices`, so that neighbours that follow one
// another in memory fall into different classes).  The (k+1)-th largest of these maxima, v*, is reached by at least k
// candidates besides the query itself, so the k nearest all have v >= v* up to rounding.  The second pass forms the
// same v again and lists the candidates with v >= v* - 2 e (screen_threshold_kernel), about 1.1 to 1.7 k of them, and
// screen_rank_kernel ranks those by (distance, index) with the distances of the other kernels: the same sums in the
// same order, so the result is the same to the last bit.  A query whose list overflows or comes out short (data with
// many equal points, a spread so large that e exceeds the distances, non-finite coordinates) goes to knn_mfma_kernel
// with the 64 queries around it.
//
// e bounds the error of v.  Points are centred and scaled by a power of two (M = the largest norm, in [1, 2)); a
// coordinate is split into two bf16 parts, x = h + m + r with |m| <= 2^-9 |x| and |r| <= 1.02 * 2^-18 |x|, and
// q.y ~ h.h + (h.m + m.h): what is left out is at most 3.1 * 2^-18 |q||y| (Cauchy-Schwarz).  The cross terms are summed
// first, then the DP terms of h.h: taking every one of those additions to be off by 2^-23 of the sum of the moduli gives
// DP 2^-23 (1 + 2^-6) |q||y|, the subtraction of |y|^2 / 2, rounded to float, 2^-23 M^2 more.  The rounding of the
// centred coordinates (2^-52 of the largest original one, A) moves v by less than 3 M sqrt(DP) 2^-52 A, and 2^-40 M^2
// covers the rounding of the fp64 distances that decide in the end.
//
// 100,000 points of 32 coordinates, k = 20: 28.2 ms for the fp64 screen alone (22.7 TFLOP/s), 3.75 ms with
// this one (two passes of 1.5 and 2.1 ms; 64 coordinates, k = 32: 61 -> 7.2 ms).  Data that it cannot settle pay for what
// it did before that showed: 28.0 -> 29.1 ms for tight clusters far apart, 48.5 -> 53.2 ms with every 20th point the same
// one, which leaves each tile of 64 queries to the fp64 kernel.  Bound by the matrix cores and, up to 32 coordinates, the vector
// work on the 16 results that a lane gets from each tile (subtract, running maximum).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int kScreenMinN = 512;
constexpr int kMomentBlocks = 256;
constexpr int kQueue = 256;        // survivors a wave gathers in LDS before it hands them on
constexpr float kNoValue = -3.0e38f;

struct ScreenScale {  // device: what the passes need to know of the whole point set
  double max_abs;            // A, of the original coordinates
  unsigned long long m2;     // bits of the largest centred squared norm
};

// part[b][c] = sum, part[b][DP + c] = largest modulus of coordinate c over the rows of block b
__global__ __launch_bounds__(kT) void screen_moments_kernel(const double* __restrict__ xp, int64_t n, int dp,
                                                            double* __restrict__ part) {
  __shared__ double sums[kT], tops[kT];
  const int c = threadIdx.x % dp, r = threadIdx.x / dp, nr = kT / dp;
  double sum = 0.0, top = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * nr + r; i < n; i += (int64_t)gridDim.x * nr) {
    const double v = xp[i * dp + c];
    sum += v;
    top = fmax(top, fabs(v));
  }
  sums[threadIdx.x] = sum;
  tops[threadIdx.x] = top;
  __syncthreads();
  if (r) return;
  for (int q = 1; q < nr; ++q) {
    sum += sums[q * dp + c];
    top = fmax(top, tops[q * dp + c]);
  }
  part[(int64_t)blockIdx.x * 2 * dp + c] = sum;
  part[(int64_t)blockIdx.x * 2 * dp + dp + c] = top;
}

// 8 threads per coordinate take every 8th block's part; their sums are added in thread order
__global__ __launch_bounds__(1024) void screen_mean_kernel(const double* __restrict__ part, int nparts, int64_t n, int dp,
                                                           double* __restrict__ mean, ScreenScale* __restrict__ scale) {
  __shared__ double sums[8][128], tops[8][128];
  const int c = threadIdx.x & 127, r = threadIdx.x >> 7;
  double sum = 0.0, top = 0.0;
  if (c < dp) {
#pragma unroll 4
    for (int b = r; b < nparts; b += 8) {
      sum += part[(int64_t)b * 2 * dp + c];
      top = fmax(top, part[(int64_t)b * 2 * dp + dp + c]);
    }
  }
  sums[r][c] = sum;
  tops[r][c] = top;
  __syncthreads();
  if (r == 0) {
    for (int q = 1; q < 8; ++q) {
      sum += sums[q][c];
      top = fmax(top, tops[q][c]);
    }
    if (c < dp) mean[c] = sum / (double)n;
    tops[0][c] = top;
  }
  __syncthreads();
  if (threadIdx.x) return;
  for (int q = 1; q < 128; ++q) top = fmax(top, tops[0][q]);
  scale->max_abs = top;
  scale->m2 = 0ull;
}

// nrm2[i] = |x_i - mean|^2, scale->m2 = the largest (as bits: a NaN counts as larger than everything)
__global__ __launch_bounds__(kT) void screen_norms_kernel(const double* __restrict__ xp, const double* __restrict__ mean,
                                                          int64_t n, int dp, double* __restrict__ nrm2,
                                                          ScreenScale* __restrict__ scale) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  double acc = 0.0;
  if (i < n) {
    for (int t = 0; t < dp; ++t) {
      const double v = xp[i * dp + t] - mean[t];
      acc = fma(v, v, acc);
    }
    nrm2[i] = acc;
  }
  unsigned long long bits = (unsigned long long)__double_as_longlong(acc);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(bits, o, 64);
    bits = other > bits ? other : bits;
  }
  if ((threadIdx.x & 63) == 0 && bits > scale->m2) atomicMax(&scale->m2, bits);
}

__device__ __forceinline__ bool screen_usable(const ScreenScale& s) {
  const double m2 = __longlong_as_double((long long)s.m2);
  return m2 > 1e-200 && m2 < 1e200 && s.max_abs < 1e100;
}
__device__ __forceinline__ double screen_factor(const ScreenScale& s) {  // power of two that takes M into [1, 2)
  return screen_usable(s) ? ldexp(1.0, -ilogb(sqrt(__longlong_as_double((long long)s.m2)))) : 0.0;
}

// parts that a list of candidate tiles is taken in: about kPartTiles tiles each, at least `least` while there are tiles
constexpr int kPartTiles = 24;
__host__ __device__ __forceinline__ int group_parts(int tiles, int least) {
  const int by_size = (tiles + kPartTiles - 1) / kPartTiles, some = tiles < least ? tiles : least;
  return by_size > some ? by_size : some;
}

__device__ __forceinline__ uint32_t ordered(float v) {  // order-preserving image of a float
  const uint32_t b = __float_as_uint(v);
  return b & 0x80000000u ? ~b : b | 0x80000000u;
}

// The operands in the order in which a wave reads them.  Tile t = points 32 t .. 32 t + 31; piece (t, s, part) = 64
// lanes x 8 bf16, lane l = coordinates 16 s + 8 (l / 32) + 0..7 of point 32 t + l % 32, part 0 = h, part 1 = m.  Points
// past the end are zeros with half[.] = +3e38, which no query ever prefers.  One thread per lane of a piece pair.
// src (may be null): place i holds point src[i], or nothing where that is negative.
__global__ __launch_bounds__(kT) void screen_split_kernel(const double* __restrict__ xp, const double* __restrict__ mean,
                                                          const double* __restrict__ nrm2, int64_t n, int dp, int ks,
                                                          const ScreenScale* __restrict__ scale, int64_t tiles,
                                                          const int32_t* __restrict__ src, u4* __restrict__ xb, float* __restrict__ half,
                                                          float* __restrict__ norm) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (e >= tiles * ks * 64) return;
  const int l = (int)(e & 63);
  const int64_t ts = e >> 6;
  const int s = (int)(ts % ks);
  const int64_t t = ts / ks, place = 32 * t + (l & 31);
  const int64_t i = src ? (int64_t)src[place] : (place < n ? place : -1);
  const double f = screen_factor(*scale);
  union { __bf16 b[8]; u4 v; } h, m;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int c = 16 * s + 8 * (l >> 5) + q;
    const float x = i >= 0 && c < dp ? (float)((xp[i * dp + c] - mean[c]) * f) : 0.0f;
    h.b[q] = (__bf16)x;
    m.b[q] = (__bf16)(x - (float)h.b[q]);
  }
  xb[(ts * 2) * 64 + l] = h.v;
  xb[(ts * 2 + 1) * 64 + l] = m.v;
  if (s == 0 && l < 32) {
    const double q = i >= 0 ? nrm2[i] * f * f : 0.0;
    half[place] = i >= 0 ? (float)(0.5 * q) : 3.0e38f;
    norm[place] = (float)(sqrt(q) * 1.000001);  // rounded up
  }
}

// One pass over all candidates for the queries of tiles qtile0 ...  A workgroup's four waves own NQ tiles of 32 queries
// each (B operands, in registers) and go through the candidate tiles slice, slice + slices, ... (A operands), staged
// through LDS in 16 KB chunks that all four read; the next chunk is in flight while this one is multiplied.  A lane
// then holds 16 candidates of one query: register r = candidate 8 (r / 4) + 4 (lane / 32) + r % 4 of the tile.
//   COLLECT false: maxima[(query - first query) * groups + slice * 16 + 8 (lane / 32) + r % 8]
//   COLLECT true:  candidates with v >= tau[query - first query] are appended to the query's list (count, list)
// Where the point set has no usable scale (a NaN among the coordinates, all points equal) there is nothing to screen.
// LISTED: the points are grouped (see below): tiles of places, point of place p = src[p] (negative: none).  A workgroup takes
// a part of a query block's list of candidate tiles, parts[blockIdx.x] = (block, part, number of parts of the block, -):
// entries part, part + number, ... of near[near_stride block ...].  The maxima are kept as order-preserving integers; parts
// share the `slices` sets of classes where there are more of them (the list kernel has then cleared the block's maxima).
template <int DP, int NQ, bool COLLECT, bool LISTED>
__global__ __launch_bounds__(kMt) __attribute__((amdgpu_waves_per_eu(2))) void screen_kernel(
    const u4* __restrict__ xb, const float* __restrict__ half, int64_t n, int64_t tiles, int64_t qtile0, int64_t qtiles,
    int slices, const ScreenScale* __restrict__ scale, const int32_t* __restrict__ src, const int32_t* __restrict__ near,
    const int32_t* __restrict__ near_count, int64_t near_stride, const int4* __restrict__ parts,
    const int32_t* __restrict__ nparts, float* __restrict__ maxima, const float* __restrict__ tau, int cap,
    int32_t* __restrict__ count, int32_t* __restrict__ list) {
  if (!screen_usable(*scale)) return;  // uniform over the grid
  int4 part = make_int4((int)blockIdx.x, (int)blockIdx.y, slices, 0);
  if constexpr (LISTED) {
    if ((int)blockIdx.x >= *nparts) return;
    part = parts[blockIdx.x];
  }
  constexpr int KS = DP / 16;
  constexpr int CT = 8 / KS;             // candidate tiles per chunk: 16 KB
  constexpr int PT = KS * 2 * 64;        // 16-byte pieces per tile
  constexpr int NL = CT * PT / kMt;      // pieces a thread stages: 4
  __shared__ u4 stage[2][CT * PT];
  __shared__ float hstage[2][CT * 32];
  __shared__ int2 queue[COLLECT ? 4 : 1][COLLECT ? kQueue : 1];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int slice = part.y, step = part.z;
  const int64_t qt0 = ((int64_t)part.x * 4 + wave) * NQ;  // relative to qtile0
  // at least one: slices <= tiles, and a list has no more parts than entries
  const int64_t nj = ((LISTED ? (int64_t)near_count[part.x] : tiles) - slice + step - 1) / step;
  const int64_t nchunk = (nj + CT - 1) / CT;
  const int32_t* __restrict__ mine = LISTED ? near + (int64_t)part.x * near_stride + slice : nullptr;
  // the j-th candidate tile
  auto tile_of = [&](int64_t j) __attribute__((always_inline)) -> int64_t {
    return LISTED ? (int64_t)mine[j * step] : slice + j * step;
  };

  bf16x8 bh[NQ][KS], bm[NQ][KS];
  float thr[NQ];
  float best[COLLECT ? 1 : NQ][8];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    int64_t t = qtile0 + qt0 + q;
    t = t < tiles ? t : tiles - 1;  // past the end: computed, never stored
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      bh[q][s] = __builtin_bit_cast(bf16x8, xb[((t * KS + s) * 2) * 64 + lane]);
      bm[q][s] = __builtin_bit_cast(bf16x8, xb[((t * KS + s) * 2 + 1) * 64 + lane]);
    }
    if constexpr (COLLECT)
      thr[q] = qt0 + q < qtiles && (LISTED || t * 32 + (lane & 31) < n) ? tau[(qt0 + q) * 32 + (lane & 31)] : INFINITY;
    else
#pragma unroll
      for (int r = 0; r < 8; ++r) best[q][r] = kNoValue;
  }

  u4 next[NL];
  float hnext = 0.0f;
  // LISTED: the tiles of the chunk after the next one are looked up a chunk ahead (kept in registers without a list, too, they
  // cost 3 to 6 % of a pass at 128 coordinates)
  int64_t at[NL], hat = 0;
  auto nth = [&](int64_t chunk, int of) __attribute__((always_inline)) -> int64_t {
    const int64_t j = chunk * CT + of;
    return tile_of(j < nj ? j : nj - 1);  // the last tile again: skipped below
  };
  auto look_up = [&](int64_t chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NL; ++u) at[u] = nth(chunk, (tid + u * kMt) / PT);
    if (tid < CT * 32) hat = nth(chunk, tid / 32);
  };
  auto request = [&](int64_t chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NL; ++u) next[u] = xb[(LISTED ? at[u] : nth(chunk, (tid + u * kMt) / PT)) * PT + (tid + u * kMt) % PT];
    if (tid < CT * 32) hnext = half[(LISTED ? hat : nth(chunk, tid / 32)) * 32 + tid % 32];
    if (LISTED && chunk + 1 < nchunk) look_up(chunk + 1);
  };
  auto park = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NL; ++u) stage[buf][tid + u * kMt] = next[u];
    if (tid < CT * 32) hstage[buf][tid] = hnext;
  };

  int queued = 0;  // wave-uniform
  auto hand_on = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // the wave's own LDS operations complete in order
    __builtin_amdgcn_wave_barrier();
    for (int e = lane; e < queued; e += 64) {
      const int2 entry = queue[wave][e];
      const int32_t point = LISTED ? src[entry.y] : entry.y;
      const int slot = atomicAdd(&count[entry.x], 1);
      if (slot < cap) list[(int64_t)entry.x * cap + slot] = point;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    queued = 0;
  };

  if (LISTED) look_up(0);
  request(0);
  park(0);
  __syncthreads();
  for (int64_t chunk = 0; chunk < nchunk; ++chunk) {
    const int buf = (int)(chunk & 1);
    if (chunk + 1 < nchunk) request(chunk + 1);
#pragma unroll 1
    for (int ct = 0; ct < CT; ++ct) {
      const int64_t j = chunk * CT + ct;
      if (j >= nj) break;  // uniform
      const u4* __restrict__ a = &stage[buf][ct * PT];
      f16v acc[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0.0f;
#pragma unroll
      for (int s = 0; s < KS; ++s) {  // the small cross terms first
        const bf16x8 ah = __builtin_bit_cast(bf16x8, a[(s * 2) * 64 + lane]);
        const bf16x8 am = __builtin_bit_cast(bf16x8, a[(s * 2 + 1) * 64 + lane]);
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bh[q][s], acc[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bm[q][s], acc[q], 0, 0, 0);
      }
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const bf16x8 ah = __builtin_bit_cast(bf16x8, a[(s * 2) * 64 + lane]);
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh[q][s], acc[q], 0, 0, 0);
      }
      float y[16];
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f4 v = *reinterpret_cast<const f4*>(&hstage[buf][ct * 32 + 8 * r4 + 4 * (lane >> 5)]);
#pragma unroll
        for (int r = 0; r < 4; ++r) y[4 * r4 + r] = v[r];
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = acc[q][r] - y[r];
        if constexpr (!COLLECT) {
#pragma unroll
          for (int r = 0; r < 8; ++r) best[q][r] = fmaxf(fmaxf(best[q][r], v[r]), v[r + 8]);
        } else {
          float top = v[0];
#pragma unroll
          for (int r = 1; r < 16; ++r) top = fmaxf(top, v[r]);
          if (__any(top >= thr[q])) {  // uniform
            // places past the end and empty ones have v of -3e38, below every threshold; a query's own place is left out
            const int64_t tile = tile_of(j);
            uint32_t hits = 0u;
#pragma unroll
            for (int r = 0; r < 16; ++r) hits |= v[r] >= thr[q] ? 1u << r : 0u;
            if (tile == qtile0 + qt0 + q && (((lane & 31) >> 2) & 1) == (lane >> 5))  // uniform; the lane that holds it
              hits &= ~(1u << (4 * ((lane & 31) >> 3) + (lane & 3)));
            const int c0 = (int)tile * 32 + 4 * (lane >> 5);
            const int ql = (int)(qt0 + q) * 32 + (lane & 31);  // relative to the first query
            // a lane's hits one by one: as many turns as the fullest lane has
            for (;;) {
              const unsigned long long mask = __ballot(hits != 0u);
              if (!mask) break;
              if (hits) {
                const int r = __ffs(hits) - 1;
                queue[wave][queued + __popcll(mask & ((1ull << lane) - 1ull))] = make_int2(ql, c0 + 8 * (r >> 2) + (r & 3));
                hits &= hits - 1u;
              }
              queued += __popcll(mask);
              if (queued > kQueue - 64) hand_on();
            }
          }
        }
      }
    }
    if (chunk + 1 < nchunk) park(buf ^ 1);  // nobody reads that buffer before the barrier
    __syncthreads();
  }
  if constexpr (COLLECT) {
    hand_on();
  } else {
    const int groups = slices * 16;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (qt0 + q >= qtiles) continue;
      const int set = LISTED ? slice % slices : slice;
      float* __restrict__ out = maxima + ((qt0 + q) * 32 + (lane & 31)) * groups + set * 16 + 8 * (lane >> 5);
      if constexpr (LISTED) {
        if (step > slices) {  // uniform
#pragma unroll
          for (int r = 0; r < 8; ++r) atomicMax(reinterpret_cast<uint32_t*>(out) + r, ordered(best[q][r]));
          continue;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) best[q][r] = __uint_as_float(ordered(best[q][r]));
      }
#pragma unroll
      for (int r = 0; r < 8; r += 4) *reinterpret_cast<f4*>(out + r) = (f4){best[q][r], best[q][r + 1], best[q][r + 2], best[q][r + 3]};
    }
  }
}

// tau[q] = v* - 2 e, v* = the (k+1)-th largest maximum of query q0 + q, found bit by bit; clears the query's list.
// bound[i] = a squared distance that at least k others do not exceed, from the query's point i: what the fp64 kernel starts from
// if it comes to that.  i = q0 + q, or src[q0 + q] where the points are grouped; there only the classes that the parts of the
// query block's list fill are looked at (group_parts).
// A query is lost (tau = +inf: nothing is listed, the fp64 kernel takes it) in a point set without a usable scale and where
// more than most_classes classes reach the cut, far too many for its list; the kLostSlots counters at `lost_count` count the
// lost ones between them (one counter for all of 100,000 took 1 ms).
// What depends on the point set alone is formed once a wave, which then takes `run` queries, up to kThresholdRun where there
// are enough for every place of a wave on the chip (a wave a query, with the square roots and the logarithm of the estimate in
// each, took 110 instead of 74 us for 100,000 queries and 208 classes).
constexpr int kThresholdRun = 8;
template <int NP>  // keys per lane: groups <= 64 NP
__global__ __launch_bounds__(kT) void screen_threshold_kernel(const float* __restrict__ maxima, int groups, int k, int dp,
                                                              const float* __restrict__ norm, int64_t q0, int64_t nq,
                                                              int run, const int32_t* __restrict__ src,
                                                              const int32_t* __restrict__ near_count, int qt, int least_parts,
                                                              const double* __restrict__ nrm2, int most_classes,
                                                              const ScreenScale* __restrict__ scale,
                                                              float* __restrict__ tau, int32_t* __restrict__ count,
                                                              double* __restrict__ bound,
                                                              int32_t* __restrict__ lost_count) {
  const int lane = threadIdx.x & 63;
  const int64_t first = ((int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6)) * run;
  const int64_t end = first + run < nq ? first + run : nq;
  const ScreenScale s = *scale;
  const bool usable = screen_usable(s);
  const double f = screen_factor(s), m = sqrt(__longlong_as_double((long long)s.m2)) * f * 1.000001;
  const double u23 = 1.1920928955078125e-07;  // 2^-23
  const double e_norm = m * (3.1 / 262144.0 + 1.02 * dp * u23);
  const double e_rest = u23 * m * m + 3.0 * m * sqrt((double)dp) * 2.220446049250313e-16 * s.max_abs * f + 9.1e-13 * m * m;
  const double f2 = f * f, per_f2 = 1.0 / f2;  // a power of two: exact
  for (int64_t q = first; q < end; ++q) {
    const int64_t i = src ? (int64_t)src[q0 + q] : q0 + q;  // the point in that place
    if (i < 0) {
      if (lane == 0) {
        count[q] = 0;
        tau[q] = INFINITY;
      }
      continue;
    }
    // classes that have been looked at: all, or those of the parts of the query block's list
    const int filled = src ? min(groups, 16 * group_parts(near_count[q / (32 * qt)], least_parts)) : groups;
    uint32_t key[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      key[u] = 0u;
      if (64 * u + lane < filled) {
        const float v = maxima[q * groups + 64 * u + lane];
        key[u] = src ? __float_as_uint(v) : ordered(v);
      }
    }
    uint32_t low = 0u;  // the largest value that at least k + 1 keys reach
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t probe = low | (1u << bit);
      int reach = 0;
#pragma unroll
      for (int u = 0; u < NP; ++u) reach += __popcll(__ballot(key[u] >= probe));
      if (reach > k) low = probe;
      if (reach == k + 1) {  // uniform: it is the smallest of those
        uint32_t least = 0xffffffffu;
#pragma unroll
        for (int u = 0; u < NP; ++u) least = key[u] >= probe && key[u] < least ? key[u] : least;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          const uint32_t other = __shfl_xor(least, o, 64);
          least = other < least ? other : least;
        }
        low = least;
        break;
      }
    }
    const float vstar = __uint_as_float(low & 0x80000000u ? low & 0x7fffffffu : ~low);
    if (!usable || !(vstar > -1.0e38f)) {  // uniform
      if (lane == 0) {
        count[q] = 0;
        tau[q] = INFINITY;
        bound[i] = INFINITY;
        atomicAdd(&lost_count[blockIdx.x % kLostSlots * kLostStride], 1);
      }
      continue;
    }
    const double e = (double)norm[q0 + q] * e_norm + e_rest;
    const double t = (double)vstar - 2.0 * e;
    const float cut = (float)(t - 1.2e-7 * fabs(t));  // rounded down
    // how many will be listed: the classes that reach the cut say so, were they filled at random
    const uint32_t ck = ordered(cut);
    int reach = 0;
#pragma unroll
    for (int u = 0; u < NP; ++u) reach += __popcll(__ballot(key[u] >= ck));
    if (lane == 0) {
      const bool lost = reach > most_classes;
      count[q] = 0;
      tau[q] = lost ? INFINITY : cut;
      if (lost) atomicAdd(&lost_count[blockIdx.x % kLostSlots * kLostStride], 1);
      const double d2 = nrm2[i] * f2 - 2.0 * ((double)vstar - e);
      bound[i] = (d2 + 1e-6 * fabs(d2)) * per_f2;
    }
  }
}

// grouped points: queries of a round whose lists of candidates did not come out right, for group_exact_kernel
constexpr int kMostLost = 1024;  // more of them in a round go to the fp64 kernel

// The k nearest of the listed candidates, by (exact squared distance, index).  A wave per query: a lane computes a
// candidate's distance as the other kernels do, its rank is the number of listed candidates before it.
// Eight coordinates of 64 rows at a time go through LDS, four lanes a row: a lane that read its own row asked for a line of its
// own in every load, 64 a load, and that was what the launch lasted.  Ranks come from the upper words of the distances, of which
// no two are alike in most queries; where some are, the ranks do not add up to what they then do, and the distances and indices
// themselves are compared.  100,000 queries of 32 coordinates, 20 neighbours: 212 -> 152 us (32
// coordinates of all rows at once: 162); what is left is rows from the L2s, 17 TB/s if all lists are full.
constexpr int kRankPitch = 5;                       // double2s a row: four and one for the banks
constexpr int kRankStage = 64 * kRankPitch + 16;    // ... and the query's
// waves a workgroup: four, or one where lists are so long (171 neighbours) that four take more than 64 KB of LDS
inline int rank_threads(int cap) { return cap <= 576 ? kT : 64; }
inline size_t rank_lds_bytes(int cap) { return (size_t)(rank_threads(cap) / 64) * (kRankStage * 16 + ((size_t)cap + 3) / 4 * 4 * 16); }
typedef double v2d __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(kT) void screen_rank_kernel(const double* __restrict__ xp, int dp, int64_t q0, int64_t nq,
                                                         const int32_t* __restrict__ src, int k, int cap,
                                                         const int32_t* __restrict__ count,
                                                         const int32_t* __restrict__ list,
                                                         int32_t* __restrict__ nlost, int32_t* __restrict__ lost,
                                                         int32_t* __restrict__ tile_flag, int32_t* __restrict__ tiles,
                                                         int32_t* __restrict__ ntiles, int32_t* __restrict__ idx_out,
                                                         double* __restrict__ dist_out) {
  extern __shared__ v2d rank_lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int cap4 = (cap + 3) / 4 * 4;
  v2d* const stage = rank_lds + (size_t)wave * kRankStage;
  v2d* const query = stage + 64 * kRankPitch;
  double* const dist = reinterpret_cast<double*>(rank_lds + (size_t)waves * kRankStage) + (size_t)wave * cap4;
  int32_t* const idx = reinterpret_cast<int32_t*>(dist + (size_t)(waves - wave) * cap4) + (size_t)wave * cap4;
  uint32_t* const upper = reinterpret_cast<uint32_t*>(idx + (size_t)waves * cap4);
  const int64_t q = (int64_t)blockIdx.x * waves + wave;
  if (q >= nq) return;
  const int64_t i = src ? (int64_t)src[q0 + q] : q0 + q;
  if (i < 0) return;
  const int32_t first = list[q * cap + (lane < cap ? lane : 0)];  // before it is known how many there are
  const int found = count[q];
  if (found > cap || found < k) {
    // no further count once there are too many: one counter for 100,000 queries is 1 ms
    if (src && lane == 0 && __hip_atomic_load(nlost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= kMostLost) {
      const int at = atomicAdd(nlost, 1);
      if (at < kMostLost) {
        lost[at] = (int32_t)q;
        return;
      }
    }
    if (lane == 0 && atomicExch(&tile_flag[i / kMq], 1) == 0) tiles[atomicAdd(ntiles, 1)] = (int32_t)(i / kMq);
    return;
  }
  const v2d* __restrict__ qr = reinterpret_cast<const v2d*>(xp + i * dp);
  for (int c0 = 0; c0 < found; c0 += 64) {
    const int here = found - c0 < 64 ? found - c0 : 64;
    const int32_t j = c0 == 0 ? first : list[q * cap + c0 + (lane < here ? lane : 0)];
    int32_t row[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) row[u] = __shfl(j, 16 * u + lane / 4 < here ? 16 * u + lane / 4 : 0, 64);
    double ex = 0.0;
    for (int t0 = 0; t0 < dp; t0 += 16) {  // 16 coordinates of all rows under way at once
      v2d v[2][4], own = {0.0, 0.0};
      if (lane < 8 && t0 + 2 * lane < dp) own = qr[t0 / 2 + lane];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int t = t0 + 8 * h + 2 * (lane & 3);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          v[h][u] = *reinterpret_cast<const v2d*>(xp + (int64_t)row[u] * dp + (t < dp ? t : 0));
      }
      if (lane < 8) query[lane] = own;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int u = 0; u < 4; ++u) stage[(16 * u + lane / 4) * kRankPitch + (lane & 3)] = v[h][u];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the wave's own LDS operations complete in order
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const v2d yv = stage[lane * kRankPitch + p], qv = query[4 * h + p];
          const bool in = t0 + 8 * h + 2 * p < dp;  // uniform; both rows' padding is even
          const double d0 = in ? qv.x - yv.x : 0.0, d1 = in ? qv.y - yv.y : 0.0;
          ex = fma(d0, d0, ex);
          ex = fma(d1, d1, ex);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
    if (lane < here) {
      dist[c0 + lane] = ex;
      idx[c0 + lane] = j;
      upper[c0 + lane] = (uint32_t)__double2hiint(ex);
    }
  }
  if (lane < 3 && found + lane < cap4) upper[found + lane] = 0xffffffffu;  // no distance: up to a whole piece of four
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  auto place = [&](int c, int rank) __attribute__((always_inline)) {
    if (rank < k) {
      idx_out[i * k + rank] = idx[c];
      dist_out[i * k + rank] = sqrt(dist[c]);
    }
  };
  if (found <= 128) {
    const uint32_t own0 = lane < found ? upper[lane] : 0u, own1 = 64 + lane < found ? upper[64 + lane] : 0u;
    int rank0 = 0, rank1 = 0;
    for (int o = 0; o < found; o += 4) {
      const uint4 h = *reinterpret_cast<const uint4*>(upper + o);
      rank0 += (h.x < own0) + (h.y < own0) + (h.z < own0) + (h.w < own0);
      if (found > 64) rank1 += (h.x < own1) + (h.y < own1) + (h.z < own1) + (h.w < own1);
    }
    int sum = rank0 + rank1;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (sum == found * (found - 1) / 2) {  // uniform; less where two are alike
      if (lane < found) place(lane, rank0);
      if (64 + lane < found) place(64 + lane, rank1);
      return;
    }
  }
  for (int c = lane; c < found; c += 64) {
    const double own = dist[c];
    const int32_t id = idx[c];
    int rank = 0;
    for (int o = 0; o < found; ++o) rank += (dist[o] < own || (dist[o] == own && idx[o] < id)) ? 1 : 0;
    place(c, rank);
  }
}

// ---- grouped points ----------------------------------------------------------------------------------------------
// Above kGroupMinWork the points are first put in an order in which tiles of 32 are compact, so that a block of queries
// need not look at most tiles at all.  Points that a spectral clustering is meant for lie in clusters, and then a query's
// neighbours are in the few tiles of its own cluster.
//   * Cells: every (n / cells)-th point is a pivot; a point belongs to the cell of (about) its nearest pivot: the h.h product
//     of the screen, kGroupCell points a cell on average.  Cells are padded to whole tiles and follow one another by nearest
//     pivot among every 64th, of these among every 16th and every 4th, which keeps the tiles of one query block close.
//     A point farther from its pivot than kGroupFar times what pivots have to the nearest of every 4th one (in the mean of
//     the squares) would make its tile's ball useless: such points have kFarCells cells of their own, behind the others.
//   * Whether it will pay is asked of the pivots first: how many of them one has within four times its distance to the nearest
//     other one, in the mean over kWithin of them.  This goes with the share of the points that the lists will keep; where it
//     is above group_within the plain passes are taken at once.  (Finding out by making the lists costs 220 of 980 us for
//     65,000 points, 290 of 2,000 for 100,000.  Lines for 600 sets of 22,500 to 400,000 points in 2 to 128 dimensions: even
//     and normal, curves, sheets, clusters tight and overlapping, heavy tails.)
//   * Reach: the threshold pass over the tiles around the query block alone (kGroupAhead on either side) bounds the distance
//     to the k-th neighbour of every query; reach_t = the largest one of tile t.
//   * Lists: a tile has a centre and a radius (fp64 against the rounded centre, rounded up).  A query block keeps the tiles w
//     at a centre distance c from one of its tiles t with c - r_t - r_w <= reach_t.  Whatever is nearer than the k-th
//     neighbour, or as near, is in them, so both passes over the lists alone leave the same survivors to the fp64 ranking,
//     and the result is the same to the last bit.
//   * Parts: a list is worked on in parts of about kPartTiles tiles, a workgroup each, so that the few blocks that have to
//     look at every tile (the far points') are not what a pass waits for.
// All bounds are in the centred and scaled coordinates of the screen (largest norm in [1, 2)) with a margin of 2e-5 of the
// centre distance (sums of up to 128 rounded squares) and 2e-6 + 8 sqrt(DP) 2^-52 A for the rounding of the coordinates.
// The host reads how much the lists leave (one wait) and takes the plain passes where that is more than group_most: a pair of
// tiles costs four times as much by a list, twice where its products are longer (plain -> grouped, with the lists, which are
// made by then; 100,000 points, 10 neighbours, 4 to 6 dimensions: a share of 0.15 1,995 -> 1,583 us, 0.20 2,017 -> 1,885, 0.22
// 1,941 -> 1,997, 0.26 2,017 -> 2,335, 0.45 2,008 -> 3,526; 32 dimensions: 0.25 3,297 -> 2,629, 0.39 949 -> 1,116 with 45,000,
// 0.47 3,266 -> 4,141; 64 dimensions: 0.38 6,808 -> 4,680, 0.71 6,833 -> 7,737).
//
// What bounded the search before was the number of pairs: 100,000 points of 32 coordinates in 100 clusters took two passes
// of 1.5 and 2.1 ms over 10^10 of them, 3.7 ms in all; 1.09 ms with the lists (3 % of the tile pairs).  400,000 points in 400
// clusters: 49.7 -> 5.2 ms, 100,000 of 3 coordinates in 200: 2.15 -> 0.84 ms, without clusters in 32 dimensions 3.7 ms as
// before.  The line: 30,000 x 32 in 30 clusters (2.9e10) 0.58 -> 0.54 ms, 45,000 x 32 (6.5e10) 1.01 -> 0.60 ms, and the same
// without clusters 1.00 -> 0.98 ms.
constexpr double kGroupMinWork = 6.0e10;  // n^2 (padded coordinates)
constexpr int kGroupCell = 64;
constexpr int kGroupMaxCells = 16384;  // 16 bits in the keys
constexpr int kGroupAhead = 24;
constexpr int kFarCells = 64;
constexpr double kGroupFar = 4.0;
// Share of the pivots within four times the distance to the nearest one up to which the lists are made.  Up to 16 coordinates
// smaller sets have less to save and more neighbours need more tiles (points without clusters; share, plain -> grouped: 62,000
// points, 10 neighbours 0.053 948 -> 778 us, 0.076 920 -> 1,096; 80,000 0.051 1,354 -> 1,326; 100,000 0.093 1,957 -> 1,984;
// 140,000 0.064 3,573 -> 2,838; 50 neighbours, 62,000 0.053 1,265 -> 1,324, 80,000 0.051 1,798 -> 2,087, 100,000 0.047 2,536 ->
// 2,579, 140,000 0.035 4,442 -> 3,517, 0.064 4,457 -> 4,838).
double group_within(int64_t n, int dpb, int k) {
  if (dpb > 16) return 0.25;
  return 0.095 * std::min(1.0, (double)n / 1e5) * std::min(1.0, std::max(0.5, std::pow(10.0 / k, 0.4)));
}
// Share of the plain passes' tile pairs up to which the lists are taken.  A cell's points come in the order of its counter's
// additions, so the share of the same points differs a little from call to call (62,003 points of 2 coordinates, outliers among
// them, 300 calls: 0.240 to 0.256), and calls close to the line may go either way.  They take the same time there: up to 16
// coordinates the lists are the faster way below a share of about 0.2 and the slower one above 0.3, and in between it depends
// on the points (grouped to plain once the lists are made: 0.215 0.87, 0.22 1.03, 0.24 0.87 and 1.12, 0.248 0.94, 0.251 0.92,
// 0.253 1.08, 0.254 1.04, 0.255 0.91, 0.263 1.02, 0.268 1.05, 0.274 1.02, 0.275 0.98, 0.28 0.95, 0.284 1.07, 0.30 1.13, 0.31 1.17;
// 62,003 to 250,000 points of 2 to 16 coordinates, 5 to 50 neighbours).
double group_most(int dpb) { return dpb <= 16 ? 0.265 : dpb <= 32 ? 0.38 : 0.62; }

struct GroupInfo {  // device
  unsigned long long pairs;  // sum of the lists' lengths over the query blocks
  double within;             // share of the pivots within four times a pivot's distance to its nearest other one
  float far;                 // squared distance to the pivot from which a point is a far one, in the screen's scale
  int32_t tiles;             // tiles of the grouped places
  int32_t nparts;            // parts of the lists
  int32_t lost;              // queries that the ranking handed on (may exceed kMostLost: the others went to the fp64 kernel)
};

// entries of `parts` for the list of query block b, and the block's maxima cleared where parts will share them; by the
// `nthreads` threads of which this is number `tid` (all call; one of them reserves and hands the place round through LDS)
__device__ __forceinline__ void group_emit_parts(int b, int listed, int least, int slices, int64_t query_tiles, int qt,
                                                 int tid, int nthreads, int32_t* lds_place, int32_t* __restrict__ nparts,
                                                 int4* __restrict__ parts, uint32_t* __restrict__ maxima) {
  const int np = group_parts(listed, least);
  if (tid == 0) *lds_place = atomicAdd(nparts, np);
  __syncthreads();
  const int at = *lds_place;
  for (int e = tid; e < np; e += nthreads) parts[at + e] = make_int4(b, e, np, 0);
  if (np <= slices) return;
  const int64_t t0 = (int64_t)b * qt, t1 = t0 + qt < query_tiles ? t0 + qt : query_tiles;
  for (int64_t e = t0 * 512 * slices + tid; e < t1 * 512 * slices; e += nthreads) maxima[e] = 0u;  // 32 queries x 16 classes
}

// no point in any place, no point in any cell, the pivots
__global__ __launch_bounds__(kT) void group_init_kernel(int64_t n, int64_t places, int cells, int pivot_places,
                                                        int32_t* __restrict__ src, int32_t* __restrict__ pivot,
                                                        int32_t* __restrict__ size, int32_t* __restrict__ order,
                                                        GroupInfo* __restrict__ info) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (e < places) src[e] = -1;
  if (e < pivot_places) pivot[e] = e < cells ? (int32_t)(e * n / cells) : -1;
  if (e < cells + kFarCells) size[e] = 0;
  if (e >= cells && e < cells + kFarCells) order[e] = (int32_t)e;
  if (e == 0) {
    info->pairs = 0ull;
    info->tiles = 0;
    info->nparts = 0;
    info->lost = 0;
  }
}

// cell[i] = number of the pivot with the largest v(x_i, pivot) by the leading parts, seat[i] = i's place among the cell's
// points.  A wave takes two tiles of points (B operands) and reads the pivots' tiles from the L2.
template <int DP>
__global__ __launch_bounds__(kT) void group_assign_kernel(const u4* __restrict__ xb, int64_t n, int64_t tiles,
                                                          const float* __restrict__ half, const u4* __restrict__ pb,
                                                          const float* __restrict__ phalf, int pivot_tiles, int cells,
                                                          const GroupInfo* __restrict__ info, int32_t* __restrict__ cell,
                                                          int32_t* __restrict__ seat, int32_t* __restrict__ size) {
  constexpr int KS = DP / 16, NQ = 2;
  const int lane = threadIdx.x & 63;
  const int64_t t0 = ((int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6)) * NQ;
  if (t0 >= tiles) return;
  bf16x8 b[NQ][KS];
  float best[NQ];
  int at[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int64_t t = t0 + q < tiles ? t0 + q : tiles - 1;
#pragma unroll
    for (int s = 0; s < KS; ++s) b[q][s] = __builtin_bit_cast(bf16x8, xb[((t * KS + s) * 2) * 64 + lane]);
    best[q] = -INFINITY;
    at[q] = 0;
  }
  for (int pt = 0; pt < pivot_tiles; ++pt) {
    f16v acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[q][r] = 0.0f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, pb[(((int64_t)pt * KS + s) * 2) * 64 + lane]);
#pragma unroll
      for (int q = 0; q < NQ; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[q][s], acc[q], 0, 0, 0);
    }
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int p0 = 32 * pt + 8 * r4 + 4 * (lane >> 5);
      const f4 h = *reinterpret_cast<const f4*>(&phalf[p0]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const float v = acc[q][4 * r4 + r] - h[r];
          at[q] = v > best[q] ? p0 + r : at[q];
          best[q] = fmaxf(best[q], v);
        }
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const float ov = __shfl_xor(best[q], 32, 64);
    const int oa = __shfl_xor(at[q], 32, 64);
    int c = ov > best[q] || (ov == best[q] && oa < at[q]) ? oa : at[q];
    const int64_t i = (t0 + q) * 32 + lane;
    if (lane < 32 && i < n) {
      if (2.0f * (half[i] - fmaxf(ov, best[q])) > info->far) c = cells + (int)(i % kFarCells);
      cell[i] = c;
      seat[i] = atomicAdd(&size[c], 1);
    }
  }
}

constexpr int kKeyPivots = 4;
// d2[p] = squared distance of row q[p] to the row y, of `pairs` pairs of coordinates
__device__ __forceinline__ void pivot_distances(const double2* const (&q)[kKeyPivots], const double2* __restrict__ y, int pairs,
                                                double (&d2)[kKeyPivots]) {
#pragma unroll
  for (int p = 0; p < kKeyPivots; ++p) d2[p] = 0.0;
#pragma unroll 4
  for (int t = 0; t < pairs; ++t) {
    const double2 b = y[t];
#pragma unroll
    for (int p = 0; p < kKeyPivots; ++p) {
      const double2 a = q[p][t];
      d2[p] = fma(a.x - b.x, a.x - b.x, d2[p]);
      d2[p] = fma(a.y - b.y, a.y - b.y, d2[p]);
    }
  }
}

// within[e0 .. e0 + kKeyPivots) = how many pivots are within four times the distance that pivot e cells / kWithin has to its
// nearest other one, the equal ones among them.  A workgroup.
constexpr int kWithin = 256;
__device__ __forceinline__ void count_within(const double2* __restrict__ xp2, int pairs, const int32_t* __restrict__ pivot,
                                             int cells, int e0, int32_t* __restrict__ within) {
  constexpr int W = kT / 64;
  __shared__ double least[kKeyPivots][W];
  __shared__ int counts[kKeyPivots][W];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double2* q[kKeyPivots];
  int from[kKeyPivots], count[kKeyPivots];
  double other[kKeyPivots], d2[kKeyPivots];
#pragma unroll
  for (int p = 0; p < kKeyPivots; ++p) {
    from[p] = (int)((int64_t)(e0 + p) * cells / kWithin);
    q[p] = xp2 + (int64_t)pivot[from[p]] * pairs;
    other[p] = INFINITY;
    count[p] = 0;
  }
  for (int c = threadIdx.x; c < cells; c += kT) {
    pivot_distances(q, xp2 + (int64_t)pivot[c] * pairs, pairs, d2);
#pragma unroll
    for (int p = 0; p < kKeyPivots; ++p)
      if (c != from[p]) other[p] = fmin(other[p], d2[p]);
  }
#pragma unroll
  for (int p = 0; p < kKeyPivots; ++p) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) other[p] = fmin(other[p], __shfl_xor(other[p], o, 64));
    if (lane == 0) least[p][wave] = other[p];
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < kKeyPivots; ++p)
#pragma unroll
    for (int w = 0; w < W; ++w) other[p] = fmin(other[p], least[p][w]);
  for (int c = threadIdx.x; c < cells; c += kT) {
    pivot_distances(q, xp2 + (int64_t)pivot[c] * pairs, pairs, d2);
#pragma unroll
    for (int p = 0; p < kKeyPivots; ++p) count[p] += c != from[p] && d2[p] <= 16.0 * other[p] ? 1 : 0;
  }
#pragma unroll
  for (int p = 0; p < kKeyPivots; ++p) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) count[p] += __shfl_xor(count[p], o, 64);
    if (lane == 0) counts[p][wave] = count[p];
  }
  __syncthreads();
  if (threadIdx.x < kKeyPivots) {
    int all = 0;
    for (int w = 0; w < W; ++w) all += counts[threadIdx.x][w];
    within[e0 + threadIdx.x] = all;
  }
}

// key[f] = (nearest of every 64th pivot, of every 16th, of every 4th, f) of pivot f, each nearest to the one after it;
// near2[f] = squared distance to the nearest other one of every 4th.  A wave takes kKeyPivots pivots at a time, so that a row
// that it reads serves them all.
// The workgroups from `key_blocks` on count what is within reach of some pivots (count_within).
__global__ __launch_bounds__(kT) void group_key_kernel(const double* __restrict__ xp, int dp, const int32_t* __restrict__ pivot,
                                                       int cells, unsigned long long* __restrict__ key,
                                                       double* __restrict__ near2, int key_blocks,
                                                       int32_t* __restrict__ within) {
  if ((int)blockIdx.x >= key_blocks) {
    count_within(reinterpret_cast<const double2*>(xp), dp / 2, pivot, cells, ((int)blockIdx.x - key_blocks) * kKeyPivots, within);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int f0 = ((int)blockIdx.x * (kT / 64) + (threadIdx.x >> 6)) * kKeyPivots;
  if (f0 >= cells) return;
  const double2* __restrict__ xp2 = reinterpret_cast<const double2*>(xp);
  int from[kKeyPivots], found[3][kKeyPivots];
#pragma unroll
  for (int p = 0; p < kKeyPivots; ++p) from[p] = f0 + p < cells ? f0 + p : cells - 1;
#pragma unroll
  for (int level = 0; level < 3; ++level) {
    const int step = level == 0 ? 4 : level == 1 ? 16 : 64;
    const double2* q[kKeyPivots];
    double best[kKeyPivots], other[kKeyPivots];
    int at[kKeyPivots];
#pragma unroll
    for (int p = 0; p < kKeyPivots; ++p) {
      q[p] = xp2 + (int64_t)pivot[__builtin_amdgcn_readfirstlane(from[p])] * (dp / 2);
      best[p] = other[p] = INFINITY;
      at[p] = 0;
    }
    for (int c = lane; c * step < cells; c += 64) {
      double d2[kKeyPivots];
      pivot_distances(q, xp2 + (int64_t)pivot[c * step] * (dp / 2), dp / 2, d2);
#pragma unroll
      for (int p = 0; p < kKeyPivots; ++p) {
        if (c * step != from[p]) other[p] = fmin(other[p], d2[p]);
        if (d2[p] < best[p]) {
          best[p] = d2[p];
          at[p] = c * step;
        }
      }
    }
#pragma unroll
    for (int p = 0; p < kKeyPivots; ++p) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const double ob = __shfl_xor(best[p], o, 64);
        const int oa = __shfl_xor(at[p], o, 64);
        if (ob < best[p] || (ob == best[p] && oa < at[p])) {
          best[p] = ob;
          at[p] = oa;
        }
        other[p] = fmin(other[p], __shfl_xor(other[p], o, 64));
      }
      found[level][p] = at[p];
      if (level == 0 && lane == 0 && f0 + p < cells) near2[f0 + p] = other[p];
      from[p] = at[p];
    }
  }
  if (lane) return;
#pragma unroll
  for (int p = 0; p < kKeyPivots; ++p)
    if (f0 + p < cells)
      key[f0 + p] = ((unsigned long long)found[2][p] << 48) | ((unsigned long long)found[1][p] << 32) |
                    ((unsigned long long)found[0][p] << 16) | (unsigned)(f0 + p);
}

// info->within and info->far from the pivots' counts and near2.  One workgroup.
__global__ __launch_bounds__(1024) void group_measure_kernel(const double* __restrict__ near2,
                                                            const int32_t* __restrict__ within, int cells,
                                                            const ScreenScale* __restrict__ scale,
                                                            GroupInfo* __restrict__ info) {
  __shared__ double sums[2][16];
  double a = 0.0, b = (int)threadIdx.x < kWithin ? (double)within[threadIdx.x] : 0.0;
  for (int f = threadIdx.x; f < cells; f += 1024) a += near2[f];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    sums[0][threadIdx.x >> 6] = a;
    sums[1][threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x) return;
  for (int w = 1; w < 16; ++w) {
    a += sums[0][w];
    b += sums[1][w];
  }
  const double f = screen_factor(*scale);
  info->within = screen_usable(*scale) ? b / ((double)kWithin * cells) : 1.0;  // no grouping without a scale
  info->far = (float)(kGroupFar * (a / cells) * f * f);
}

// order[rank of f's key] = f.  A wave per pivot.
__global__ __launch_bounds__(kT) void group_rank_kernel(const unsigned long long* __restrict__ key, int cells,
                                                        int32_t* __restrict__ order) {
  const int lane = threadIdx.x & 63;
  const int f = (int)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
  if (f >= cells) return;
  const unsigned long long mine = key[f];
  int before = 0;
  for (int c = lane; c < cells; c += 64) before += key[c] < mine ? 1 : 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
  if (lane == 0) order[before] = f;  // the keys differ: every rank once
}

// base[f] = first tile of cell f; info->tiles.  One workgroup.
__global__ __launch_bounds__(1024) void group_scan_kernel(const int32_t* __restrict__ order, const int32_t* __restrict__ size,
                                                          int cells, int32_t* __restrict__ base,
                                                          GroupInfo* __restrict__ info) {
  __shared__ int32_t sums[16];
  const int tid = threadIdx.x, per = (cells + 1023) / 1024;
  const int lo = tid * per < cells ? tid * per : cells, hi = lo + per < cells ? lo + per : cells;
  int total = 0;
  for (int e = lo; e < hi; ++e) total += (size[order[e]] + 31) / 32;
  int incl = total;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if ((tid & 63) >= o) incl += up;
  }
  if ((tid & 63) == 63) sums[tid >> 6] = incl;
  __syncthreads();
  int run = incl - total;
  for (int w = 0; w < (tid >> 6); ++w) run += sums[w];
  for (int e = lo; e < hi; ++e) {
    const int f = order[e];
    base[f] = run;
    run += (size[f] + 31) / 32;
  }
  if (tid == 1023) info->tiles = run;
}

__global__ __launch_bounds__(kT) void group_place_kernel(const int32_t* __restrict__ cell, const int32_t* __restrict__ seat,
                                                         const int32_t* __restrict__ base, int64_t n,
                                                         int32_t* __restrict__ src) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < n) src[(int64_t)base[cell[i]] * 32 + seat[i]] = (int32_t)i;
}

__device__ __forceinline__ float group_margin(const ScreenScale& s, int dp) {
  return (float)(2e-6 + 8.0 * sqrt((double)dp) * 2.3e-16 * s.max_abs * screen_factor(s));
}

// centre and radius of every tile; the centre's coordinates 4 c .. 4 c + 3 at centre[c stride + tile].  A wave per tile: 64 / dp
// rows at a time, a lane per coordinate (two at 128).
template <int DP>
__global__ __launch_bounds__(kT) void group_ball_kernel(const double* __restrict__ xp, const double* __restrict__ mean,
                                                        const ScreenScale* __restrict__ scale, const int32_t* __restrict__ src,
                                                        const GroupInfo* __restrict__ info, int64_t stride,
                                                        float* __restrict__ centre, float* __restrict__ radius) {
  constexpr int PER = DP > 64 ? DP / 64 : 1, W = DP / PER, G = 64 / W;  // coordinates a lane, lanes a row, rows at a time
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
  if (t >= info->tiles) return;
  const int32_t own = lane < 32 ? src[t * 32 + lane] : -1;
  const int cnt = __popcll(__ballot(own >= 0));
  const double f = screen_factor(*scale);
  const int c = lane % W, g = lane / W;
  double mu[PER], sum[PER];
  float mid[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    mu[u] = mean[c + u * W];
    sum[u] = 0.0;
  }
  for (int p = g; p < 32; p += G) {
    const int32_t i = __shfl(own, p, 64);
    if (i < 0) continue;
#pragma unroll
    for (int u = 0; u < PER; ++u) sum[u] += (xp[(int64_t)i * DP + c + u * W] - mu[u]) * f;
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
#pragma unroll
    for (int o = W; o < 64; o <<= 1) sum[u] += __shfl_xor(sum[u], o, 64);
    mid[u] = (float)(sum[u] / (double)(cnt > 0 ? cnt : 1));
    if (g == 0) centre[((c + u * W) / 4 * stride + t) * 4 + (c + u * W) % 4] = mid[u];
  }
  double far = 0.0;
  for (int p0 = 0; p0 < 32; p0 += G) {
    const int32_t i = __shfl(own, p0 + g, 64);
    double d2 = 0.0;
    if (i >= 0) {
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const double df = (xp[(int64_t)i * DP + c + u * W] - mu[u]) * f - (double)mid[u];
        d2 = fma(df, df, d2);
      }
    }
#pragma unroll
    for (int o = 1; o < W; o <<= 1) d2 += __shfl_xor(d2, o, 64);
    far = fmax(far, d2);
  }
#pragma unroll
  for (int o = W; o < 64; o <<= 1) far = fmax(far, __shfl_xor(far, o, 64));
  if (lane == 0) radius[t] = (float)(sqrt(far) * 1.000001);
}

// near[near_stride b ..] = the tiles from kGroupAhead before query block b to kGroupAhead behind it.  A wave per block.
__global__ __launch_bounds__(64) void group_window_kernel(GroupInfo* __restrict__ info, int qt, int64_t tile0,
                                                          int64_t query_tiles, int least, int slices,
                                                          int32_t* __restrict__ near, int64_t near_stride,
                                                          int32_t* __restrict__ near_count, int4* __restrict__ parts,
                                                          uint32_t* __restrict__ maxima) {
  __shared__ int32_t place;
  const int64_t b = blockIdx.x;
  const int64_t tiles = info->tiles, q0 = tile0 + b * qt;
  int64_t lo = q0 - kGroupAhead, hi = q0 + qt + kGroupAhead;
  lo = lo < 0 ? 0 : lo;
  hi = hi > tiles ? tiles : hi;
  if (q0 >= tiles) hi = lo;
  const int tid = threadIdx.x;
  for (int64_t w = lo + tid; w < hi; w += 64) near[b * near_stride + (w - lo)] = (int32_t)w;
  if (tid == 0) near_count[b] = (int32_t)(hi - lo);
  group_emit_parts((int)b, (int)(hi - lo), least, slices, query_tiles, qt, tid, 64, &place, &info->nparts, parts, maxima);
}

// the counts of a list's parts and pairs start anew
__global__ void group_recount_kernel(GroupInfo* __restrict__ info) {
  info->pairs = 0ull;
  info->nparts = 0;
  info->lost = 0;
}

// The queries that the ranking handed on, from the tiles of their block's list in fp64: what is not beyond the bound of the k-th
// distance, ranked as there.  A workgroup per query.  Where the points are grouped a query's neighbours lie in few tiles and
// share classes, and now and then one's list of candidates runs over; a handful of such queries through all points, one workgroup
// per 64 of them, is what a search then lasted (62,000 normal points of 2 coordinates, 50 neighbours, 5.8 ms for 1.3 without
// groups; 100,000 even ones of 3, 100 neighbours, 17.5 for 4.2).
constexpr int kExactThreads = 512, kExactRoom = 4096;
__global__ __launch_bounds__(kExactThreads) void group_exact_kernel(
    const double* __restrict__ xp, int dp, const int32_t* __restrict__ src, int64_t q0, int qt, const int32_t* __restrict__ near,
    const int32_t* __restrict__ near_count, int64_t near_stride, const double* __restrict__ bound, int k,
    const GroupInfo* __restrict__ info, const int32_t* __restrict__ lost, int32_t* __restrict__ tile_flag,
    int32_t* __restrict__ tiles, int32_t* __restrict__ ntiles, int32_t* __restrict__ idx_out, double* __restrict__ dist_out) {
  __shared__ double dist[kExactRoom];
  __shared__ int32_t idx[kExactRoom];
  __shared__ int32_t kept;
  if (info->lost > kMostLost) {  // the fp64 kernel is needed anyway: these come on top of it (100,000 x 16 along a line 20.2 -> 18.7 ms)
    for (int l = blockIdx.x * kExactThreads + threadIdx.x; l < kMostLost; l += gridDim.x * kExactThreads) {
      const int64_t i = src[q0 + lost[l]];
      if (atomicExch(&tile_flag[i / kMq], 1) == 0) tiles[atomicAdd(ntiles, 1)] = (int32_t)(i / kMq);
    }
    return;
  }
  const int nlost = info->lost;
  for (int l = blockIdx.x; l < nlost; l += gridDim.x) {  // uniform over the workgroup
    const int64_t q = lost[l], i = src[q0 + q], b = q / (32 * qt);
    const double most = bound[i];
    const int32_t* __restrict__ mine = near + b * near_stride;
    const int64_t places = 32 * (int64_t)near_count[b];
    const double2* __restrict__ xp2 = reinterpret_cast<const double2*>(xp);
    const double2* __restrict__ qr = xp2 + i * (dp / 2);
    if (threadIdx.x == 0) kept = 0;
    __syncthreads();
    for (int64_t e = threadIdx.x; e < places; e += kExactThreads) {
      const int32_t j = src[32 * (int64_t)mine[e >> 5] + (e & 31)];
      if (j < 0 || j == i) continue;
      const double2* __restrict__ yr = xp2 + (int64_t)j * (dp / 2);
      double ex = 0.0;
#pragma unroll 4
      for (int t = 0; t < dp / 2; ++t) {
        const double2 qv = qr[t], yv = yr[t];
        const double d0 = qv.x - yv.x;
        ex = fma(d0, d0, ex);
        const double d1 = qv.y - yv.y;
        ex = fma(d1, d1, ex);
      }
      if (!(ex <= most)) continue;
      const int at = atomicAdd(&kept, 1);
      if (at < kExactRoom) {
        dist[at] = ex;
        idx[at] = j;
      }
    }
    __syncthreads();
    const int found = kept;
    if (found > kExactRoom || found < k) {
      if (threadIdx.x == 0 && atomicExch(&tile_flag[i / kMq], 1) == 0) tiles[atomicAdd(ntiles, 1)] = (int32_t)(i / kMq);
    } else {
      for (int c = threadIdx.x; c < found; c += kExactThreads) {
        const double v = dist[c];
        const int32_t id = idx[c];
        int rank = 0;
        for (int o = 0; o < found; ++o) rank += (dist[o] < v || (dist[o] == v && idx[o] < id)) ? 1 : 0;
        if (rank < k) {
          idx_out[i * k + rank] = id;
          dist_out[i * k + rank] = sqrt(v);
        }
      }
    }
    __syncthreads();  // before the next query's candidates
  }
}

// reach[t] = the largest bound of a k-th distance among the points of tile t, in the screen's scale.  A half-wave per tile.
__global__ __launch_bounds__(kT) void group_reach_kernel(const int32_t* __restrict__ src, const double* __restrict__ bound,
                                                         const GroupInfo* __restrict__ info, int64_t tile0, int64_t ntiles,
                                                         const ScreenScale* __restrict__ scale, float* __restrict__ reach) {
  const int64_t t = (int64_t)blockIdx.x * (kT / 32) + (threadIdx.x >> 5);
  if (t >= ntiles || tile0 + t >= info->tiles) return;
  const int32_t i = src[(tile0 + t) * 32 + (threadIdx.x & 31)];
  double far = i >= 0 ? bound[i] : 0.0;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) far = fmax(far, __shfl_xor(far, o, 32));
  if ((threadIdx.x & 31) == 0) reach[tile0 + t] = (float)(sqrt(far) * screen_factor(*scale) * 1.000001);
}

// The candidate tiles of query block b = tiles [tile0 + QT b, tile0 + QT (b + 1)), in ascending order.  A workgroup per
// block, a thread per candidate tile: first against a ball round the block, then against its tiles.
template <int DP, int QT>
__global__ __launch_bounds__(1024) void group_list_kernel(const f4* __restrict__ centre, int64_t stride,
                                                          const float* __restrict__ radius, const float* __restrict__ reach,
                                                          GroupInfo* __restrict__ info, const ScreenScale* __restrict__ scale,
                                                          int64_t tile0, int64_t query_tiles, int least, int slices,
                                                          int32_t* __restrict__ near, int64_t near_stride,
                                                          int32_t* __restrict__ near_count, int4* __restrict__ parts,
                                                          uint32_t* __restrict__ maxima) {
  constexpr int NT = 1024;
  __shared__ int32_t place;
  __shared__ f4 ctr[QT][DP / 4];
  __shared__ float far[QT], far_mid[QT];
  __shared__ int taken[2][NT / 64];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t tiles = info->tiles, q0 = tile0 + (int64_t)blockIdx.x * QT;
  if (q0 >= tiles) {
    if (tid == 0) near_count[blockIdx.x] = 0;
    return;
  }
  for (int e = tid; e < QT * DP / 4; e += NT) {
    const int64_t t = q0 + e % QT < tiles ? q0 + e % QT : tiles - 1;
    ctr[e % QT][e / QT] = centre[e / QT * stride + t];
  }
  // how far from the tile's centre a ball may begin; a NaN keeps everything
  if (tid < QT) far[tid] = q0 + tid < tiles ? radius[q0 + tid] + reach[q0 + tid] + group_margin(*scale, DP) : -INFINITY;
  __syncthreads();
  // the same from the middle tile's centre, for all of the block's tiles
  if (tid < QT) {
    float d2 = 0.0f;
    for (int c = 0; c < DP / 4; ++c)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float df = ctr[tid][c][u] - ctr[QT / 2][c][u];
        d2 = fmaf(df, df, d2);
      }
    far_mid[tid] = sqrtf(d2) * 1.00002f + far[tid];
  }
  __syncthreads();
  float block_far = far_mid[0];
#pragma unroll
  for (int q = 1; q < QT; ++q) block_far = far_mid[q] > block_far || far_mid[q] != far_mid[q] ? far_mid[q] : block_far;
  int32_t* __restrict__ out = near + (int64_t)blockIdx.x * near_stride;
  int listed = 0, side = 0;
  for (int64_t w0 = 0; w0 < tiles; w0 += NT, side ^= 1) {
    const int64_t w = w0 + tid, ws = w < tiles ? w : tiles - 1;
    const float r = radius[ws];
    float m2 = 0.0f;
#pragma unroll
    for (int c = 0; c < DP / 4; ++c) {
      const f4 y = centre[c * stride + ws], x = ctr[QT / 2][c];
#pragma unroll
      for (int u = 0; u < 4; ++u) m2 = fmaf(x[u] - y[u], x[u] - y[u], m2);
    }
    bool keep = !(sqrtf(m2) * 0.99998f - r > block_far) & (w < tiles);
    if (__any(keep)) {  // uniform over the wave
      float d2[QT];
#pragma unroll
      for (int q = 0; q < QT; ++q) d2[q] = 0.0f;
#pragma unroll 2
      for (int c = 0; c < DP / 4; ++c) {
        const f4 y = centre[c * stride + ws];
#pragma unroll
        for (int q = 0; q < QT; ++q) {
          const f4 x = ctr[q][c];
#pragma unroll
          for (int u = 0; u < 4; ++u) d2[q] = fmaf(x[u] - y[u], x[u] - y[u], d2[q]);
        }
      }
      bool any = false;
#pragma unroll
      for (int q = 0; q < QT; ++q) any = any | !(sqrtf(d2[q]) * 0.99998f - r > far[q]);
      keep = keep & any;
    }
    const unsigned long long mask = __ballot(keep);
    if (lane == 0) taken[side][wave] = __popcll(mask);
    __syncthreads();  // two sets of counts: one barrier a round
    int before = 0, all = 0;
#pragma unroll
    for (int o = 0; o < NT / 64; ++o) {
      const int c = taken[side][o];
      before += o < wave ? c : 0;
      all += c;
    }
    if (keep) out[listed + before + __popcll(mask & ((1ull << lane) - 1ull))] = (int32_t)w;
    listed += all;
  }
  if (tid == 0) {
    near_count[blockIdx.x] = listed;
    atomicAdd(&info->pairs, (unsigned long long)listed);
  }
  group_emit_parts((int)blockIdx.x, listed, least, slices, query_tiles, QT, tid, NT, &place, &info->nparts, parts, maxima);
}

// mask[w] = which of the 64 list entries 64 w .. 64 w + 63 name an edge that their row emits, cnt[w] = how many: a valid
// neighbour j != i, not listed earlier in the same row, and either i < j or i is not in j's list (else row j emits the pair).
// A thread per entry: a wave reads 64 consecutive entries and 64 rows that do not wait for one another (a thread per row,
// k rows one after the other and the same again to write the edges, took 133 + 196 us for
// 100,000 x 20 entries; these 39 + 20 us).
__global__ __launch_bounds__(kT) void pair_mark_kernel(const int32_t* __restrict__ idx, int64_t n, int k,
                                                       unsigned long long* __restrict__ mask, int32_t* __restrict__ cnt) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  bool emits = false;
  if (e < n * k) {
    const int64_t i = e / k;
    const int s = (int)(e - i * k);
    const int32_t j = idx[e];
    emits = j >= 0 && j < n && j != i;
    if (emits) {
      for (int q = 0; q < s; ++q) emits &= idx[i * k + q] != j;
      if (i > j) {
        const int32_t* __restrict__ other = idx + (int64_t)j * k;
#pragma unroll 4
        for (int q = 0; q < k; ++q) emits &= other[q] != (int32_t)i;
      }
    }
  }
  const unsigned long long m = __ballot(emits);
  if ((threadIdx.x & 63) == 0 && e < n * k) {
    mask[e >> 6] = m;
    cnt[e >> 6] = __popcll(m);
  }
}

__global__ __launch_bounds__(kT) void pair_emit_kernel(const int32_t* __restrict__ idx, const double* __restrict__ dist,
                                                       int64_t n, int k, const unsigned long long* __restrict__ mask,
                                                       const int32_t* __restrict__ offset, double inv_two_sigma2,
                                                       int32_t* __restrict__ eu, int32_t* __restrict__ ev,
                                                       double* __restrict__ val) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (e >= n * k) return;
  const int lane = threadIdx.x & 63;
  const unsigned long long m = mask[e >> 6];
  if (!((m >> lane) & 1ull)) return;
  const int64_t o = (int64_t)offset[e >> 6] + __popcll(m & ((1ull << lane) - 1ull));
  const int32_t i = (int32_t)(e / k), j = idx[e];
  const double dd = dist[e];
  eu[o] = i < j ? i : j;
  ev[o] = i < j ? j : i;
  val[o] = inv_two_sigma2 > 0.0 ? exp(-(dd * dd) * inv_two_sigma2) : dd;
}

}  // namespace

int knn_padded_dim(int d) {
  return d <= 8 ? 8 : d <= 16 ? 16 : d <= 32 ? 32 : d <= 64 ? 64 : d <= 128 ? 128 : (d + kDC - 1) / kDC * kDC;
}

size_t knn_search_lds_bytes(int d, int k) {
  const int dp = knn_padded_dim(d);
  if (dp <= 128)  // distances, thresholds, masks, indices of the MFMA kernel
    return 8 * ((size_t)k * kMq + kMq + kRound * kMq) + 4 * (size_t)k * kMq;
  return (size_t)kQ * ((size_t)dp * sizeof(double) + (size_t)k * (sizeof(double) + sizeof(int32_t)));
}

namespace {

hipError_t launch_knn_mfma(const double* xp, const double* xn, int64_t n, int k, int dp, const int32_t* tiles,
                           const double* bound, unsigned grid, size_t lds, int32_t* idx_out, double* dist_out, hipStream_t st) {
#define SC_KNN_MFMA(DPV)                                                                                       \
  do {                                                                                                         \
    if (lds > 64 * 1024) {                                                                                     \
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&knn_mfma_kernel<DPV>),           \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);          \
      if (e != hipSuccess) return e;                                                                           \
    }                                                                                                          \
    hipLaunchKernelGGL(knn_mfma_kernel<DPV>, dim3(grid), dim3(kMt), lds, st, xp, xn, n, k, tiles, bound,       \
                       idx_out, dist_out);                                                                     \
  } while (0)
  if (dp == 8) SC_KNN_MFMA(8);
  else if (dp == 16) SC_KNN_MFMA(16);
  else if (dp == 32) SC_KNN_MFMA(32);
  else if (dp == 64) SC_KNN_MFMA(64);
  else SC_KNN_MFMA(128);
#undef SC_KNN_MFMA
  return hipGetLastError();
}

// What the host decides by, to its memory; the word behind it last.
__global__ __launch_bounds__(64) void info_report_kernel(const int64_t* __restrict__ info, int count, int64_t* __restrict__ host) {
  if ((int)threadIdx.x < count) put_host(host + threadIdx.x, info[threadIdx.x]);
  host_written();
  if (threadIdx.x == 0) put_host(host + count, (int64_t)1);
}
static_assert(kLostSlots == 64, "a lane per slot");
__global__ __launch_bounds__(64) void lost_report_kernel(const int32_t* __restrict__ lost_count, int64_t* __restrict__ host) {
  int sum = lost_count[threadIdx.x * kLostStride];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (threadIdx.x != 0) return;
  put_host(host, (int64_t)sum);
  host_written();
  put_host(host + 1, (int64_t)1);
}

// How the bf16 screen goes about n points of d coordinates and k neighbours.
struct ScreenPlan {
  bool use = false;
  int dpb = 0, nq = 0;          // padded coordinates (a multiple of 16) and query tiles per wave
  int slices = 0, cap = 0;
  int64_t tiles = 0, chunk = 0; // tiles of 32 points; query tiles per round of launches
  size_t off_bound = 0, off_half = 0, off_norm = 0, off_nrm2 = 0, off_mean = 0, off_part = 0, off_scale = 0, off_maxima = 0, off_tau = 0,
         off_count = 0, off_list = 0, off_flag = 0, off_tiles = 0, off_ntiles = 0, bytes = 0;
};

// sets of 16 classes for k neighbours
int screen_least_slices(int k) {
  const int need = (5 * (k + 1) + 31) / 32;
  return need > 64 ? 64 : need;
}

ScreenPlan plan_screen(int64_t n, int d, int k) {
  ScreenPlan p;
  const int dp = knn_padded_dim(d);
  // more than 128 coordinates: the operands of a query tile do not fit the registers; fewer points than 512 or than 16
  // per neighbour: too few classes for a threshold (512 points of 3 coordinates, k = 5: 140 us with the fp64 kernel
  // alone, 80 us with the screen's eight launches; 700 points of 128: 1,043 and 109 us)
  if (dp > 128 || n < kScreenMinN || (int64_t)16 * (k + 1) > n) return p;
  p.use = true;
  p.dpb = dp < 16 ? 16 : dp;
  p.nq = p.dpb <= 32 ? 4 : 2;
  p.tiles = (n + 31) / 32;
  p.cap = 3 * k + 64;
  // classes: 16 per slice, 2.5 (k + 1) of them make the threshold almost that of the k-th neighbour itself; more slices
  // where the queries alone do not fill the 512 workgroups that are resident at a time
  const int need = screen_least_slices(k);
  const int64_t qblocks = (p.tiles + 4 * p.nq - 1) / (4 * p.nq);
  int best = need;
  double best_eff = 0.0;
  const int64_t most = p.tiles < 64 ? p.tiles : 64;
  for (int s = need; s <= most; ++s) {
    const double rounds = (double)(qblocks * s) / 512.0;
    const double eff = rounds / (double)((qblocks * s + 511) / 512);
    if (eff > best_eff + 0.03) {
      best = s;
      best_eff = eff;
    }
    if (rounds > 8.0) break;
  }
  p.slices = best;
  // scratch per query: maxima and list; rounds of at most 256 MB
  const size_t per_tile = 32 * ((size_t)p.slices * 16 + p.cap) * 4;
  int64_t chunk = (int64_t)(((size_t)256 << 20) / per_tile);
  chunk = chunk / (4 * p.nq) * (4 * p.nq);
  p.chunk = chunk < 4 * p.nq ? 4 * p.nq : (chunk > p.tiles ? p.tiles : chunk);
  size_t off = (size_t)p.tiles * (p.dpb / 16) * 2 * 1024;
  auto place = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) / 256 * 256;
    return at;
  };
  p.off_half = place((size_t)p.tiles * 32 * 4);
  p.off_norm = place((size_t)p.tiles * 32 * 4);
  p.off_nrm2 = place((size_t)n * 8);
  p.off_bound = place((size_t)n * 8);
  p.off_mean = place(128 * 8);
  p.off_part = place((size_t)kMomentBlocks * 2 * 128 * 8);
  p.off_scale = place(sizeof(ScreenScale));
  p.off_maxima = place((size_t)p.chunk * 32 * p.slices * 16 * 4);
  p.off_tau = place((size_t)p.chunk * 32 * 4);
  p.off_count = place((size_t)p.chunk * 32 * 4);
  p.off_list = place((size_t)p.chunk * 32 * p.cap * 4);
  p.off_flag = place(((size_t)((n + kMq - 1) / kMq) + 1 + kLostInts) * 4);
  p.off_tiles = place((size_t)((n + kMq - 1) / kMq) * 4);
  p.off_ntiles = p.off_flag + (size_t)((n + kMq - 1) / kMq) * 4;
  p.bytes = off;
  return p;
}

// The grouped form of the screen: cells, and the places of its points.
struct GroupPlan {
  bool use = false;
  int cells = 0, pivot_tiles = 0;
  int64_t tiles = 0, chunk = 0;  // the most tiles there can be; query tiles per round of launches
  int64_t blocks = 0;            // query blocks of a round
  int least = 0, slices = 0;     // parts that a list has at least; sets of 16 classes
  size_t off_pb = 0, off_half = 0, off_norm = 0, off_phalf = 0, off_pnorm = 0, off_src = 0, off_pivot = 0, off_size = 0,
         off_base = 0, off_order = 0, off_key = 0, off_near2 = 0, off_within = 0, off_cell = 0, off_seat = 0, off_info = 0, off_centre = 0, off_radius = 0,
         off_reach = 0, off_idle = 0, off_near = 0, off_near_count = 0, off_parts = 0, off_maxima = 0, off_tau = 0, off_count = 0,
         off_list = 0, off_lost = 0, bytes = 0;
};

GroupPlan plan_group(int64_t n, int d, int k) {
  GroupPlan g;
  const ScreenPlan p = plan_screen(n, d, k);
  if (!p.use || (double)n * (double)n * p.dpb < kGroupMinWork) return g;
  const int dp = knn_padded_dim(d);
  const int64_t cells = n / kGroupCell;
  g.cells = (int)(cells < kGroupMaxCells ? cells : kGroupMaxCells);
  g.pivot_tiles = (g.cells + 31) / 32;
  g.tiles = (n + 31) / 32 + g.cells + kFarCells;  // every cell's last tile may be a ragged one
  const int qt = 4 * p.nq;
  g.least = screen_least_slices(k);
  g.slices = g.least > 8 ? g.least : 8;
  const size_t per_tile = 32 * ((size_t)g.slices * 16 + p.cap) * 4;
  int64_t chunk = (int64_t)(((size_t)256 << 20) / per_tile) / qt * qt;
  chunk = chunk < qt ? qt : chunk;
  g.chunk = chunk < g.tiles ? chunk : g.tiles;
  g.blocks = (g.chunk + qt - 1) / qt;
  if ((size_t)g.blocks * g.tiles * 4 > (size_t)1 << 30) return g;
  const size_t piece = (size_t)(p.dpb / 16) * 2 * 1024;
  size_t off = (size_t)g.tiles * piece;
  auto place = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) / 256 * 256;
    return at;
  };
  g.off_pb = place((size_t)g.pivot_tiles * piece);
  g.off_half = place((size_t)g.tiles * 32 * 4);
  g.off_norm = place((size_t)g.tiles * 32 * 4);
  g.off_phalf = place((size_t)g.pivot_tiles * 32 * 4);
  g.off_pnorm = place((size_t)g.pivot_tiles * 32 * 4);
  g.off_src = place((size_t)g.tiles * 32 * 4);
  g.off_pivot = place((size_t)g.pivot_tiles * 32 * 4);
  g.off_size = place((size_t)(g.cells + kFarCells) * 4);
  g.off_base = place((size_t)(g.cells + kFarCells) * 4);
  g.off_order = place((size_t)(g.cells + kFarCells) * 4);
  g.off_key = place((size_t)g.cells * 8);
  g.off_near2 = place((size_t)g.cells * 8);
  g.off_within = place((size_t)kWithin * 4);
  g.off_cell = place((size_t)n * 4);
  g.off_seat = place((size_t)n * 4);
  g.off_info = place(sizeof(GroupInfo));
  g.off_centre = place((size_t)g.tiles * dp * 4);
  g.off_radius = place((size_t)g.tiles * 4);
  g.off_reach = place((size_t)g.tiles * 4);
  g.off_idle = place((size_t)kLostInts * 4);
  g.off_near = place((size_t)g.blocks * g.tiles * 4);
  g.off_near_count = place((size_t)g.blocks * 4);
  g.off_parts = place((size_t)g.blocks * (g.least + (g.tiles + kPartTiles - 1) / kPartTiles) * sizeof(int4));
  g.off_maxima = place((size_t)g.chunk * 32 * g.slices * 16 * 4);
  g.off_tau = place((size_t)g.chunk * 32 * 4);
  g.off_count = place((size_t)g.chunk * 32 * 4);
  g.off_list = place((size_t)g.chunk * 32 * p.cap * 4);
  g.off_lost = place((size_t)kMostLost * 4);
  g.bytes = off;
  g.use = true;
  return g;
}

}  // namespace

size_t knn_screen_workspace(int64_t n, int d, int k) { return plan_screen(n, d, k).bytes; }

size_t knn_group_workspace(int64_t n, int d, int k) { return plan_group(n, d, k).bytes; }

hipError_t launch_knn_screen(const double* xp, int64_t n, int d, int k, void* work, void* group_work, int32_t* host,
                             int32_t** tiles, int32_t** ntiles, double** bound, bool* grouped_out, int32_t* idx_out,
                             double* dist_out, hipStream_t st) {
  const ScreenPlan p = plan_screen(n, d, k);
  if (!p.use) return hipErrorInvalidValue;
  const int dp = knn_padded_dim(d), ks = p.dpb / 16;
  char* w = static_cast<char*>(work);
  u4* xb = reinterpret_cast<u4*>(w);
  float* half = reinterpret_cast<float*>(w + p.off_half);
  float* norm = reinterpret_cast<float*>(w + p.off_norm);
  double* nrm2 = reinterpret_cast<double*>(w + p.off_nrm2);
  double* mean = reinterpret_cast<double*>(w + p.off_mean);
  double* part = reinterpret_cast<double*>(w + p.off_part);
  ScreenScale* scale = reinterpret_cast<ScreenScale*>(w + p.off_scale);
  float* maxima = reinterpret_cast<float*>(w + p.off_maxima);
  float* tau = reinterpret_cast<float*>(w + p.off_tau);
  int32_t* count = reinterpret_cast<int32_t*>(w + p.off_count);
  int32_t* list = reinterpret_cast<int32_t*>(w + p.off_list);
  int32_t* flag = reinterpret_cast<int32_t*>(w + p.off_flag);
  *tiles = reinterpret_cast<int32_t*>(w + p.off_tiles);
  *ntiles = reinterpret_cast<int32_t*>(w + p.off_ntiles);
  int32_t* lost_count = *ntiles + 1;
  *bound = reinterpret_cast<double*>(w + p.off_bound);
  int64_t lost_before = 0;
  const size_t rank_lds = rank_lds_bytes(p.cap);
  const int rank_t = rank_threads(p.cap);
  const int qt = 4 * p.nq;
  hipError_t e = launch_fill_int32(flag, (n + kMq - 1) / kMq + 1 + kLostInts, 0, 0, st);  // the flags and the counts behind
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(screen_moments_kernel, dim3(kMomentBlocks), dim3(kT), 0, st, xp, n, dp, part);
  hipLaunchKernelGGL(screen_mean_kernel, dim3(1), dim3(1024), 0, st, part, kMomentBlocks, n, dp, mean, scale);
  hipLaunchKernelGGL(screen_norms_kernel, dim3(blocks(n)), dim3(kT), 0, st, xp, mean, n, dp, nrm2, scale);
  auto split = [&](const int32_t* src, int64_t count_tiles, u4* out, float* out_half, float* out_norm) {
    hipLaunchKernelGGL(screen_split_kernel, dim3(blocks(count_tiles * ks * 64)), dim3(kT), 0, st, xp, mean, nrm2, n, dp, ks,
                       scale, count_tiles, src, out, out_half, out_norm);
  };
  split(nullptr, p.tiles, xb, half, norm);

  // what the passes work on: the points as they are, or grouped
  int64_t all_tiles = p.tiles, chunk = p.chunk;
  const int32_t *src = nullptr, *near = nullptr, *near_count = nullptr;
  int64_t near_stride = 0;
  const GroupPlan g = group_work ? plan_group(n, d, k) : GroupPlan();
  char* gw = static_cast<char*>(group_work);
  GroupInfo* info = reinterpret_cast<GroupInfo*>(gw + g.off_info);
  int4* parts = reinterpret_cast<int4*>(gw + g.off_parts);
  int slices = p.slices;
  // most_parts: how many workgroups a pass over lists can need
  auto screen = [&](bool collect, int64_t t0, int64_t nt, int64_t most_parts) {
    const dim3 grid((unsigned)(src ? most_parts : (nt + qt - 1) / qt), src ? 1u : (unsigned)slices);
#define SC_SCREEN(DPV, NQV, COL, LISTED)                                                                              \
  hipLaunchKernelGGL((screen_kernel<DPV, NQV, COL, LISTED>), grid, dim3(kMt), 0, st, xb, half, n, all_tiles, t0, nt,  \
                     slices, scale, src, near, near_count, near_stride, parts, &info->nparts, maxima, tau, p.cap, count, list)
#define SC_SCREEN_DIM(COL, LISTED)                               \
  do {                                                           \
    if (p.dpb == 16) SC_SCREEN(16, 4, COL, LISTED);              \
    else if (p.dpb == 32) SC_SCREEN(32, 4, COL, LISTED);         \
    else if (p.dpb == 64) SC_SCREEN(64, 2, COL, LISTED);         \
    else SC_SCREEN(128, 2, COL, LISTED);                         \
  } while (0)
    if (src && collect) SC_SCREEN_DIM(true, true);
    else if (src) SC_SCREEN_DIM(false, true);
    else if (collect) SC_SCREEN_DIM(true, false);
    else SC_SCREEN_DIM(false, false);
#undef SC_SCREEN_DIM
#undef SC_SCREEN
  };
  auto threshold = [&](int64_t q0, int64_t nq, int32_t* lost) {
    const int64_t run = std::min<int64_t>(std::max<int64_t>(nq / 8192, 1), kThresholdRun), per = run * (kT / 64);
    // the most classes that may reach the cut: -log(1 - r / groups) groups, the entries of a list whose classes are filled
    // at random, up to 1.5 cap
    const int groups = slices * 16;
    const int most = (int)std::min((double)(groups - 1), std::floor(-std::expm1(-1.5 * p.cap / groups) * groups));
#define SC_THRESHOLD(NPV)                                                                                              \
  hipLaunchKernelGGL((screen_threshold_kernel<NPV>), dim3((unsigned)((nq + per - 1) / per)), dim3(kT), 0, st, maxima,  \
                     groups, k, p.dpb, norm, q0, nq, (int)run, src, near_count, qt, g.least, nrm2, most, scale, tau, count, *bound, lost)
    if (slices <= 4) SC_THRESHOLD(1);
    else if (slices <= 8) SC_THRESHOLD(2);
    else if (slices <= 16) SC_THRESHOLD(4);
    else if (slices <= 32) SC_THRESHOLD(8);
    else SC_THRESHOLD(16);
#undef SC_THRESHOLD
  };
  // the lists of the query tiles [t0, t0 + nt): the tiles around them, then what the reach that these leave does not rule out
  auto list_tiles = [&](int64_t t0, int64_t nt) {
    const f4* centre = reinterpret_cast<const f4*>(gw + g.off_centre);
    const float* radius = reinterpret_cast<const float*>(gw + g.off_radius);
    float* reach = reinterpret_cast<float*>(gw + g.off_reach);
    int32_t* out = reinterpret_cast<int32_t*>(gw + g.off_near);
    int32_t* out_count = reinterpret_cast<int32_t*>(gw + g.off_near_count);
    const int64_t nblocks = (nt + qt - 1) / qt;
    uint32_t* keys = reinterpret_cast<uint32_t*>(maxima);
    hipLaunchKernelGGL(group_recount_kernel, dim3(1), dim3(1), 0, st, info);
    hipLaunchKernelGGL(group_window_kernel, dim3((unsigned)nblocks), dim3(64), 0, st, info, qt, t0, nt, g.least, g.slices, out,
                       g.tiles, out_count, parts, keys);
    screen(false, t0, nt, nblocks * group_parts(qt + 2 * kGroupAhead, g.least));
    threshold(32 * t0, 32 * nt, reinterpret_cast<int32_t*>(gw + g.off_idle));
    hipLaunchKernelGGL(group_recount_kernel, dim3(1), dim3(1), 0, st, info);
    hipLaunchKernelGGL(group_reach_kernel, dim3(blocks(nt * 32)), dim3(kT), 0, st, src, *bound, info, t0, nt, scale, reach);
#define SC_GROUP_LIST(DPV, QTV)                                                                                           \
  hipLaunchKernelGGL((group_list_kernel<DPV, QTV>), dim3((unsigned)nblocks), dim3(1024), 0, st, centre, g.tiles, radius, \
                     reach, info, scale, t0, nt, g.least, g.slices, out, g.tiles, out_count, parts, keys)
    if (dp == 8) SC_GROUP_LIST(8, 16);
    else if (dp == 16) SC_GROUP_LIST(16, 16);
    else if (dp == 32) SC_GROUP_LIST(32, 16);
    else if (dp == 64) SC_GROUP_LIST(64, 8);
    else SC_GROUP_LIST(128, 8);
#undef SC_GROUP_LIST
  };
  static_assert(sizeof(GroupInfo) % 8 == 0 && sizeof(GroupInfo) + 8 <= kLostInts * 4, "whole words, and one behind them");
  int64_t* const words = reinterpret_cast<int64_t*>(host);
  constexpr int kInfoWords = sizeof(GroupInfo) / 8;
  auto read_info = [&](GroupInfo* to) -> hipError_t {
    words[kInfoWords] = 0;
    hipLaunchKernelGGL(info_report_kernel, dim3(1), dim3(64), 0, st, reinterpret_cast<const int64_t*>(info), kInfoWords, words);
    hipError_t r = hipGetLastError();
    if (r == hipSuccess) r = wait_for_word(words + kInfoWords, 1, st);
    if (r == hipSuccess) std::memcpy(to, host, sizeof(*to));
    return r;
  };
  int64_t nparts = 0;  // of the lists at hand
  bool grouped = g.use;
  if (grouped) {
    int32_t* pivot = reinterpret_cast<int32_t*>(gw + g.off_pivot);
    double* near2 = reinterpret_cast<double*>(gw + g.off_near2);
    int32_t* within = reinterpret_cast<int32_t*>(gw + g.off_within);
    const int per = kKeyPivots * (kT / 64);
    hipLaunchKernelGGL(group_init_kernel, dim3(blocks(g.tiles * 32)), dim3(kT), 0, st, n, g.tiles * 32, g.cells,
                       g.pivot_tiles * 32, reinterpret_cast<int32_t*>(gw + g.off_src), pivot,
                       reinterpret_cast<int32_t*>(gw + g.off_size), reinterpret_cast<int32_t*>(gw + g.off_order), info);
    const int key_blocks = (g.cells + per - 1) / per;
    hipLaunchKernelGGL(group_key_kernel, dim3((unsigned)(key_blocks + kWithin / kKeyPivots)), dim3(kT), 0, st, xp, dp, pivot,
                       g.cells, reinterpret_cast<unsigned long long*>(gw + g.off_key), near2, key_blocks, within);
    hipLaunchKernelGGL(group_measure_kernel, dim3(1), dim3(1024), 0, st, near2, within, g.cells, scale, info);
    GroupInfo got;
    e = read_info(&got);
    if (e != hipSuccess) return e;
    grouped = got.within < group_within(n, p.dpb, k);  // a NaN is no
  }
  if (grouped) {
    u4* gxb = reinterpret_cast<u4*>(gw);
    u4* pb = reinterpret_cast<u4*>(gw + g.off_pb);
    float* ghalf = reinterpret_cast<float*>(gw + g.off_half);
    float* gnorm = reinterpret_cast<float*>(gw + g.off_norm);
    float* phalf = reinterpret_cast<float*>(gw + g.off_phalf);
    float* pnorm = reinterpret_cast<float*>(gw + g.off_pnorm);
    int32_t* gsrc = reinterpret_cast<int32_t*>(gw + g.off_src);
    const int32_t* pivot = reinterpret_cast<const int32_t*>(gw + g.off_pivot);
    int32_t* size = reinterpret_cast<int32_t*>(gw + g.off_size);
    int32_t* base = reinterpret_cast<int32_t*>(gw + g.off_base);
    int32_t* order = reinterpret_cast<int32_t*>(gw + g.off_order);
    const unsigned long long* key = reinterpret_cast<const unsigned long long*>(gw + g.off_key);
    int32_t* cell = reinterpret_cast<int32_t*>(gw + g.off_cell);
    int32_t* seat = reinterpret_cast<int32_t*>(gw + g.off_seat);
    float* centre = reinterpret_cast<float*>(gw + g.off_centre);
    float* radius = reinterpret_cast<float*>(gw + g.off_radius);
    const unsigned tile_grid = (unsigned)((g.tiles + kT / 64 - 1) / (kT / 64));
    hipLaunchKernelGGL(group_rank_kernel, dim3(blocks((int64_t)g.cells * 64)), dim3(kT), 0, st, key, g.cells, order);
    split(pivot, g.pivot_tiles, pb, phalf, pnorm);
    const unsigned assign_grid = (unsigned)((p.tiles + 2 * (kT / 64) - 1) / (2 * (kT / 64)));
#define SC_GROUP_ASSIGN(DPV)                                                                                          \
  hipLaunchKernelGGL((group_assign_kernel<DPV>), dim3(assign_grid), dim3(kT), 0, st, xb, n, p.tiles, half, pb, phalf, \
                     g.pivot_tiles, g.cells, info, cell, seat, size)
    if (p.dpb == 16) SC_GROUP_ASSIGN(16);
    else if (p.dpb == 32) SC_GROUP_ASSIGN(32);
    else if (p.dpb == 64) SC_GROUP_ASSIGN(64);
    else SC_GROUP_ASSIGN(128);
#undef SC_GROUP_ASSIGN
    hipLaunchKernelGGL(group_scan_kernel, dim3(1), dim3(1024), 0, st, order, size, g.cells + kFarCells, base,
                       info);
    hipLaunchKernelGGL(group_place_kernel, dim3(blocks(n)), dim3(kT), 0, st, cell, seat, base, n, gsrc);
    split(gsrc, g.tiles, gxb, ghalf, gnorm);
#define SC_GROUP_BALLS(DPV)                                                                                            \
  hipLaunchKernelGGL((group_ball_kernel<DPV>), dim3(tile_grid), dim3(kT), 0, st, xp, mean, scale, gsrc, info, g.tiles, centre, \
                     radius)
    if (dp == 8) SC_GROUP_BALLS(8);
    else if (dp == 16) SC_GROUP_BALLS(16);
    else if (dp == 32) SC_GROUP_BALLS(32);
    else if (dp == 64) SC_GROUP_BALLS(64);
    else SC_GROUP_BALLS(128);
#undef SC_GROUP_BALLS
    all_tiles = g.tiles;
    chunk = g.chunk;
    src = gsrc;
    near = reinterpret_cast<const int32_t*>(gw + g.off_near);
    near_count = reinterpret_cast<const int32_t*>(gw + g.off_near_count);
    near_stride = g.tiles;
    slices = g.slices;
    xb = gxb;
    half = ghalf;
    norm = gnorm;
    maxima = reinterpret_cast<float*>(gw + g.off_maxima);
    tau = reinterpret_cast<float*>(gw + g.off_tau);
    count = reinterpret_cast<int32_t*>(gw + g.off_count);
    list = reinterpret_cast<int32_t*>(gw + g.off_list);
    list_tiles(0, g.chunk);
    GroupInfo got;
    e = read_info(&got);
    if (e != hipSuccess) return e;
    nparts = got.nparts;
    const int64_t here = got.tiles < g.chunk ? got.tiles : g.chunk;  // query tiles of the first round, whose lists are made
    all_tiles = got.tiles;
    if (!((double)got.pairs < group_most(p.dpb) * (double)p.tiles * (double)((here + qt - 1) / qt))) {  // as they are, then
      all_tiles = p.tiles;
      chunk = p.chunk;
      slices = p.slices;
      src = nullptr;
      xb = reinterpret_cast<u4*>(w);
      half = reinterpret_cast<float*>(w + p.off_half);
      norm = reinterpret_cast<float*>(w + p.off_norm);
      maxima = reinterpret_cast<float*>(w + p.off_maxima);
      tau = reinterpret_cast<float*>(w + p.off_tau);
      count = reinterpret_cast<int32_t*>(w + p.off_count);
      list = reinterpret_cast<int32_t*>(w + p.off_list);
    }
  }
  const int64_t places = src ? all_tiles * 32 : n;
  *grouped_out = src != nullptr;
  for (int64_t t0 = 0; t0 < all_tiles; t0 += chunk) {
    const int64_t nt = all_tiles - t0 < chunk ? all_tiles - t0 : chunk;
    const int64_t q0 = 32 * t0, nq = places - q0 < 32 * nt ? places - q0 : 32 * nt;
    if (src && t0 > 0) {
      list_tiles(t0, nt);
      GroupInfo got;
      e = read_info(&got);
      if (e != hipSuccess) return e;
      nparts = got.nparts;
    }
    screen(false, t0, nt, nparts);
    threshold(q0, nq, lost_count);
    // most queries lost: the second pass would be for nothing, an empty list sends them all to the fp64 kernel
    words[1] = 0;
    hipLaunchKernelGGL(lost_report_kernel, dim3(1), dim3(kLostSlots), 0, st, lost_count, words);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = wait_for_word(words + 1, 1, st);
    if (e != hipSuccess) return e;
    const int64_t lost = words[0] - lost_before;
    lost_before += lost;
    if (lost <= nq / 2) screen(true, t0, nt, nparts);
    int32_t* gone = reinterpret_cast<int32_t*>(gw + g.off_lost);
    hipLaunchKernelGGL(screen_rank_kernel, dim3((unsigned)((nq * 64 + rank_t - 1) / rank_t)), dim3(rank_t), rank_lds, st, xp, dp, q0, nq, src, k, p.cap, count,
                       list, &info->lost, gone, flag, *tiles, *ntiles, idx_out, dist_out);
    if (src)
      hipLaunchKernelGGL(group_exact_kernel, dim3(256), dim3(kExactThreads), 0, st, xp, dp, src, q0, qt, near, near_count,
                         near_stride, *bound, k, info, gone, flag, *tiles, *ntiles, idx_out, dist_out);
  }
  return hipGetLastError();
}

hipError_t launch_knn_pad(const double* x, int64_t ldx, int64_t n, int d, double* xp, hipStream_t st) {
  const int dp = knn_padded_dim(d);
  hipLaunchKernelGGL(pad_rows_kernel, dim3(blocks(n * dp)), dim3(kT), 0, st, x, ldx, n, d, dp, xp);
  return hipGetLastError();
}

hipError_t launch_knn_search(int64_t n, int d, int k, double* xp, const int32_t* tiles, int64_t ntiles,
                             const double* bound, int32_t* idx_out, double* dist_out, hipStream_t st) {
  if (n < 2 || d < 1 || k < 1 || k > n - 1 || n > INT32_MAX) return hipErrorInvalidValue;
  const int dp = knn_padded_dim(d);
  const size_t lds = knn_search_lds_bytes(d, k);
  int dev = 0, lds_max = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  if (e != hipSuccess) return e;
  if (lds > (size_t)lds_max) return hipErrorInvalidValue;
  if (dp <= 128) {
    double* xn = xp + (size_t)n * dp;
    hipLaunchKernelGGL(row_norms_kernel, dim3(blocks(n)), dim3(kT), 0, st, xp, n, dp, xn);
    const int64_t grid = tiles ? ntiles : (n + kMq - 1) / kMq;
    return launch_knn_mfma(xp, xn, n, k, dp, tiles, bound, (unsigned)grid, lds, idx_out, dist_out, st);
  }
  if (tiles) return hipErrorInvalidValue;
  if (lds > 64 * 1024) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&knn_search_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(knn_search_kernel, dim3((unsigned)((n + kQ - 1) / kQ)), dim3(kQ), lds, st, xp, n, dp, k, idx_out,
                     dist_out);
  return hipGetLastError();
}

size_t knn_pairs_workspace(int64_t n, int k) {
  const int64_t words = (n * k + 63) / 64;
  size_t scan_bytes = 0;
  (void)rocprim::exclusive_scan(nullptr, scan_bytes, (const int32_t*)nullptr, (int32_t*)nullptr, (int32_t)0, (size_t)words,
                                rocprim::plus<int32_t>(), (hipStream_t) nullptr);
  return (scan_bytes + 255) / 256 * 256 + 16 * (size_t)words;
}

hipError_t launch_knn_union_pairs(const int32_t* idx, const double* dist, int64_t n, int k, double sigma, void* work,
                                  size_t work_bytes, int32_t* eu, int32_t* ev, double* val, int64_t* host,
                                  hipStream_t st) {
  if (n < 1 || k < 1 || n > INT32_MAX || n * k > INT32_MAX) return hipErrorInvalidValue;
  const int64_t words = (n * k + 63) / 64;
  size_t scan_bytes = 0;
  hipError_t e = rocprim::exclusive_scan(nullptr, scan_bytes, (const int32_t*)nullptr, (int32_t*)nullptr, (int32_t)0,
                                         (size_t)words, rocprim::plus<int32_t>(), st);
  if (e != hipSuccess) return e;
  const size_t tmp = (scan_bytes + 255) / 256 * 256;
  if (work_bytes < tmp + 16 * (size_t)words) return hipErrorInvalidValue;
  char* base = static_cast<char*>(work);
  unsigned long long* mask = reinterpret_cast<unsigned long long*>(base + tmp);
  int32_t* cnt = reinterpret_cast<int32_t*>(mask + words);
  int32_t* off = cnt + words;
  hipLaunchKernelGGL(pair_mark_kernel, dim3(blocks(n * k)), dim3(kT), 0, st, idx, n, k, mask, cnt);
  size_t sb = scan_bytes;
  e = rocprim::exclusive_scan(base, sb, cnt, off, (int32_t)0, (size_t)words, rocprim::plus<int32_t>(), st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pair_emit_kernel, dim3(blocks(n * k)), dim3(kT), 0, st, idx, dist, n, k, mask, off,
                     sigma > 0.0 ? 1.0 / (2.0 * sigma * sigma) : 0.0, eu, ev, val);
  // the pair count = the last offset + the last count: both handed back for the host to add
  return launch_report(nullptr, off + (words - 1), cnt + (words - 1), host, st);
}

}  // namespace sceig
