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
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/device/device_select.hpp>
#include <rocprim/functional.hpp>
#include <rocprim/iterator/counting_iterator.hpp>

#include <cstdint>

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
// one, which leaves each tile of 64 queries to the fp64 kernel.  Bound by the matrix cores and, up to 32 coordinates, the vector work on the 16 results that a lane gets from
// each tile (subtract, running maximum).
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

// The operands in the order in which a wave reads them.  Tile t = points 32 t .. 32 t + 31; piece (t, s, part) = 64
// lanes x 8 bf16, lane l = coordinates 16 s + 8 (l / 32) + 0..7 of point 32 t + l % 32, part 0 = h, part 1 = m.  Points
// past the end are zeros with half[.] = +3e38, which no query ever prefers.  One thread per lane of a piece pair.
__global__ __launch_bounds__(kT) void screen_split_kernel(const double* __restrict__ xp, const double* __restrict__ mean,
                                                          const double* __restrict__ nrm2, int64_t n, int dp, int ks,
                                                          const ScreenScale* __restrict__ scale, int64_t tiles,
                                                          u4* __restrict__ xb, float* __restrict__ half,
                                                          float* __restrict__ norm) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (e >= tiles * ks * 64) return;
  const int l = (int)(e & 63);
  const int64_t ts = e >> 6;
  const int s = (int)(ts % ks);
  const int64_t t = ts / ks, i = 32 * t + (l & 31);
  const double f = screen_factor(*scale);
  union { __bf16 b[8]; u4 v; } h, m;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int c = 16 * s + 8 * (l >> 5) + q;
    const float x = i < n && c < dp ? (float)((xp[i * dp + c] - mean[c]) * f) : 0.0f;
    h.b[q] = (__bf16)x;
    m.b[q] = (__bf16)(x - (float)h.b[q]);
  }
  xb[(ts * 2) * 64 + l] = h.v;
  xb[(ts * 2 + 1) * 64 + l] = m.v;
  if (s == 0 && l < 32) {
    const double q = i < n ? nrm2[i] * f * f : 0.0;
    half[i] = i < n ? (float)(0.5 * q) : 3.0e38f;
    norm[i] = (float)(sqrt(q) * 1.000001);  // rounded up
  }
}

// One pass over all candidates for the queries of tiles qtile0 ...  A workgroup's four waves own NQ tiles of 32 queries
// each (B operands, in registers) and go through the candidate tiles slice, slice + slices, ... (A operands), staged
// through LDS in 16 KB chunks that all four read; the next chunk is in flight while this one is multiplied.  A lane
// then holds 16 candidates of one query: register r = candidate 8 (r / 4) + 4 (lane / 32) + r % 4 of the tile.
//   COLLECT false: maxima[(query - first query) * groups + slice * 16 + 8 (lane / 32) + r % 8]
//   COLLECT true:  candidates with v >= tau[query - first query] are appended to the query's list (count, list)
// Where the point set has no usable scale (a NaN among the coordinates, all points equal) there is nothing to screen.
template <int DP, int NQ, bool COLLECT>
__global__ __launch_bounds__(kMt) __attribute__((amdgpu_waves_per_eu(2))) void screen_kernel(
    const u4* __restrict__ xb, const float* __restrict__ half, int64_t n, int64_t tiles, int64_t qtile0, int64_t qtiles,
    int slices, const ScreenScale* __restrict__ scale, float* __restrict__ maxima, const float* __restrict__ tau, int cap,
    int32_t* __restrict__ count, int32_t* __restrict__ list) {
  if (!screen_usable(*scale)) return;  // uniform over the grid
  constexpr int KS = DP / 16;
  constexpr int CT = 8 / KS;             // candidate tiles per chunk: 16 KB
  constexpr int PT = KS * 2 * 64;        // 16-byte pieces per tile
  constexpr int NL = CT * PT / kMt;      // pieces a thread stages: 4
  __shared__ u4 stage[2][CT * PT];
  __shared__ float hstage[2][CT * 32];
  __shared__ int2 queue[COLLECT ? 4 : 1][COLLECT ? kQueue : 1];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int slice = (int)blockIdx.y;
  const int64_t qt0 = ((int64_t)blockIdx.x * 4 + wave) * NQ;  // relative to qtile0
  const int64_t nj = (tiles - slice + slices - 1) / slices;  // at least one: slices <= tiles
  const int64_t nchunk = (nj + CT - 1) / CT;

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
      thr[q] = qt0 + q < qtiles && t * 32 + (lane & 31) < n ? tau[(qt0 + q) * 32 + (lane & 31)] : INFINITY;
    else
#pragma unroll
      for (int r = 0; r < 8; ++r) best[q][r] = kNoValue;
  }

  u4 next[NL];
  float hnext = 0.0f;
  auto request = [&](int64_t chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int p = tid + u * kMt;
      int64_t j = chunk * CT + p / PT;
      j = j < nj ? j : nj - 1;  // the last tile again: skipped below
      next[u] = xb[(slice + j * slices) * PT + p % PT];
    }
    if (tid < CT * 32) {
      int64_t j = chunk * CT + tid / 32;
      j = j < nj ? j : nj - 1;
      hnext = half[(slice + j * slices) * 32 + tid % 32];
    }
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
      const int slot = atomicAdd(&count[entry.x], 1);
      if (slot < cap) list[(int64_t)entry.x * cap + slot] = entry.y;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    queued = 0;
  };

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
          float top[4];
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) top[r4] = fmaxf(fmaxf(fmaxf(v[4 * r4], v[4 * r4 + 1]), v[4 * r4 + 2]), v[4 * r4 + 3]);
          if (__any(fmaxf(fmaxf(fmaxf(top[0], top[1]), top[2]), top[3]) >= thr[q])) {  // uniform
            const int64_t c0 = (slice + j * slices) * 32 + 4 * (lane >> 5);
            const int64_t ql = (qt0 + q) * 32 + (lane & 31);  // relative to the first query
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
              if (!__any(top[r4] >= thr[q])) continue;  // uniform
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int64_t c = c0 + 8 * r4 + r;
                const bool hit = v[4 * r4 + r] >= thr[q] && c < n && c != qtile0 * 32 + ql;
                const unsigned long long mask = __ballot(hit);
                if (mask) {  // uniform
                  if (hit) queue[wave][queued + __popcll(mask & ((1ull << lane) - 1ull))] = make_int2((int)ql, (int)c);
                  queued += __popcll(mask);
                  if (queued > kQueue - 64) hand_on();
                }
              }
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
      float* __restrict__ out = maxima + ((qt0 + q) * 32 + (lane & 31)) * groups + slice * 16 + 8 * (lane >> 5);
#pragma unroll
      for (int r = 0; r < 8; r += 4) *reinterpret_cast<f4*>(out + r) = (f4){best[q][r], best[q][r + 1], best[q][r + 2], best[q][r + 3]};
    }
  }
}

// tau[q] = v* - 2 e, v* = the (k+1)-th largest of the query's maxima, found bit by bit; clears the query's list.  A wave
// per query.  bound[first query + q] = a squared distance that at least k others do not exceed: what the fp64 kernel
// starts from if it comes to that.  tau = +inf (nothing is listed, the query falls back) where the point set has no
// usable scale or far too many would be listed; the kLostSlots counters at `lost_count` count those between them (one counter for
// all of 100,000 such queries took 1 ms).
template <int NP>  // keys per lane: groups <= 64 NP
__global__ __launch_bounds__(kT) void screen_threshold_kernel(const float* __restrict__ maxima, int groups, int k, int dp,
                                                              const float* __restrict__ norm, int64_t q0, int64_t nq,
                                                              const double* __restrict__ nrm2, int cap,
                                                              const ScreenScale* __restrict__ scale,
                                                              float* __restrict__ tau, int32_t* __restrict__ count,
                                                              double* __restrict__ bound,
                                                              int32_t* __restrict__ lost_count) {
  const int lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
  if (q >= nq) return;
  uint32_t key[NP];  // order-preserving image of the floats
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    key[u] = 0u;
    if (64 * u + lane < groups) {
      const uint32_t b = __float_as_uint(maxima[q * groups + 64 * u + lane]);
      key[u] = b & 0x80000000u ? ~b : b | 0x80000000u;
    }
  }
  uint32_t low = 0u;  // the largest value that at least k + 1 keys reach
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t probe = low | (1u << bit);
    int reach = 0;
#pragma unroll
    for (int u = 0; u < NP; ++u) reach += __popcll(__ballot(key[u] >= probe));
    if (reach > k) low = probe;
  }
  const float vstar = __uint_as_float(low & 0x80000000u ? low & 0x7fffffffu : ~low);
  const ScreenScale s = *scale;
  if (!screen_usable(s) || !(vstar > -1.0e38f)) {  // uniform
    if (lane == 0) {
      count[q] = 0;
      tau[q] = INFINITY;
      bound[q0 + q] = INFINITY;
      atomicAdd(&lost_count[blockIdx.x % kLostSlots * kLostStride], 1);
    }
    return;
  }
  const double f = screen_factor(s), m = sqrt(__longlong_as_double((long long)s.m2)) * f * 1.000001;
  const double u23 = 1.1920928955078125e-07;  // 2^-23
  const double e = (double)norm[q0 + q] * m * (3.1 / 262144.0 + 1.02 * dp * u23) + u23 * m * m +
                   3.0 * m * sqrt((double)dp) * 2.220446049250313e-16 * s.max_abs * f + 9.1e-13 * m * m;
  const double t = (double)vstar - 2.0 * e;
  const float cut = (float)(t - 1.2e-7 * fabs(t));  // rounded down
  // how many will be listed: the classes that reach the cut say so, were they filled at random
  const uint32_t cb = __float_as_uint(cut), ck = cb & 0x80000000u ? ~cb : cb | 0x80000000u;
  int reach = 0;
#pragma unroll
  for (int u = 0; u < NP; ++u) reach += __popcll(__ballot(key[u] >= ck));
  if (lane) return;
  const bool lost = reach >= groups || -log1p(-(double)reach / groups) * groups > 1.5 * cap;
  count[q] = 0;
  tau[q] = lost ? INFINITY : cut;
  if (lost) atomicAdd(&lost_count[blockIdx.x % kLostSlots * kLostStride], 1);
  const double d2 = nrm2[q0 + q] * f * f - 2.0 * ((double)vstar - e);
  bound[q0 + q] = (d2 + 1e-6 * fabs(d2)) / (f * f);
}

// The k nearest of the listed candidates, by (exact squared distance, index).  A wave per query: a lane computes a
// candidate's distance as the other kernels do, its rank is the number of listed candidates before it.
__global__ __launch_bounds__(kT) void screen_rank_kernel(const double* __restrict__ xp, int dp, int64_t q0, int64_t nq,
                                                         int k, int cap, const int32_t* __restrict__ count,
                                                         const int32_t* __restrict__ list,
                                                         int32_t* __restrict__ tile_flag, int32_t* __restrict__ tiles,
                                                         int32_t* __restrict__ ntiles, int32_t* __restrict__ idx_out,
                                                         double* __restrict__ dist_out) {
  extern __shared__ double lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* dist = lds + (size_t)wave * cap;
  int32_t* idx = reinterpret_cast<int32_t*>(lds + (size_t)(kT / 64) * cap) + (size_t)wave * cap;
  const int64_t q = (int64_t)blockIdx.x * (kT / 64) + wave;
  if (q >= nq) return;
  const int64_t i = q0 + q;
  const int found = count[q];
  if (found > cap || found < k) {
    if (lane == 0 && atomicExch(&tile_flag[i / kMq], 1) == 0) tiles[atomicAdd(ntiles, 1)] = (int32_t)(i / kMq);
    return;
  }
  const double2* __restrict__ xp2 = reinterpret_cast<const double2*>(xp);
  const double2* __restrict__ qr = xp2 + i * (dp / 2);
  for (int c = lane; c < found; c += 64) {
    const int32_t j = list[q * cap + c];
    const double2* __restrict__ yr = xp2 + (int64_t)j * (dp / 2);
    double ex = 0.0;
#pragma unroll 8
    for (int t = 0; t < dp / 2; ++t) {
      const double2 qv = qr[t], yv = yr[t];
      const double d0 = qv.x - yv.x;
      ex = fma(d0, d0, ex);
      const double d1 = qv.y - yv.y;
      ex = fma(d1, d1, ex);
    }
    dist[c] = ex;
    idx[c] = j;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // the wave's own LDS operations complete in order
  __builtin_amdgcn_wave_barrier();
  for (int c = lane; c < found; c += 64) {
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

// Whether entry s of row i's list names an edge that this row emits: a valid neighbour j != i, not listed earlier in
// the same row, and either i < j or i is not in j's list (else row j emits the pair).
__device__ __forceinline__ bool emits(const int32_t* __restrict__ idx, int64_t n, int k, int64_t i, int s) {
  const int32_t j = idx[i * k + s];
  if (j < 0 || j >= n || j == i) return false;
  for (int q = 0; q < s; ++q)
    if (idx[i * k + q] == j) return false;
  if (i < j) return true;
  for (int q = 0; q < k; ++q)
    if (idx[(int64_t)j * k + q] == (int32_t)i) return false;
  return true;
}

__global__ __launch_bounds__(kT) void pair_count_kernel(const int32_t* __restrict__ idx, int64_t n, int k,
                                                        int32_t* __restrict__ cnt) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  int c = 0;
  for (int s = 0; s < k; ++s) c += emits(idx, n, k, i, s) ? 1 : 0;
  cnt[i] = c;
}

__global__ __launch_bounds__(kT) void pair_emit_kernel(const int32_t* __restrict__ idx, const double* __restrict__ dist,
                                                       int64_t n, int k, const int32_t* __restrict__ offset,
                                                       double inv_two_sigma2, int32_t* __restrict__ eu,
                                                       int32_t* __restrict__ ev, double* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  int64_t o = offset[i];
  for (int s = 0; s < k; ++s) {
    if (!emits(idx, n, k, i, s)) continue;
    const int32_t j = idx[i * k + s];
    const double dd = dist[i * k + s];
    eu[o] = (int32_t)i < j ? (int32_t)i : j;
    ev[o] = (int32_t)i < j ? j : (int32_t)i;
    val[o] = inv_two_sigma2 > 0.0 ? exp(-(dd * dd) * inv_two_sigma2) : dd;
    ++o;
  }
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

// How the bf16 screen goes about n points of d coordinates and k neighbours.
struct ScreenPlan {
  bool use = false;
  int dpb = 0, nq = 0;          // padded coordinates (a multiple of 16) and query tiles per wave
  int slices = 0, cap = 0;
  int64_t tiles = 0, chunk = 0; // tiles of 32 points; query tiles per round of launches
  size_t off_bound = 0, off_half = 0, off_norm = 0, off_nrm2 = 0, off_mean = 0, off_part = 0, off_scale = 0, off_maxima = 0, off_tau = 0,
         off_count = 0, off_list = 0, off_flag = 0, off_tiles = 0, off_ntiles = 0, bytes = 0;
};

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
  int need = (5 * (k + 1) + 31) / 32;
  need = need > 64 ? 64 : need;
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

}  // namespace

size_t knn_screen_workspace(int64_t n, int d, int k) { return plan_screen(n, d, k).bytes; }

hipError_t launch_knn_screen(const double* xp, int64_t n, int d, int k, void* work, int32_t* host, int32_t** tiles,
                             int32_t** ntiles, double** bound, int32_t* idx_out, double* dist_out, hipStream_t st) {
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
  const size_t rank_lds = (size_t)(kT / 64) * p.cap * 12;
  hipError_t e = launch_fill_int32(flag, (n + kMq - 1) / kMq + 1 + kLostInts, 0, 0, st);  // the flags and the counts behind
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(screen_moments_kernel, dim3(kMomentBlocks), dim3(kT), 0, st, xp, n, dp, part);
  hipLaunchKernelGGL(screen_mean_kernel, dim3(1), dim3(1024), 0, st, part, kMomentBlocks, n, dp, mean, scale);
  hipLaunchKernelGGL(screen_norms_kernel, dim3(blocks(n)), dim3(kT), 0, st, xp, mean, n, dp, nrm2, scale);
  hipLaunchKernelGGL(screen_split_kernel, dim3(blocks(p.tiles * ks * 64)), dim3(kT), 0, st, xp, mean, nrm2, n, dp, ks, scale,
                     p.tiles, xb, half, norm);
  for (int64_t t0 = 0; t0 < p.tiles; t0 += p.chunk) {
    const int64_t nt = p.tiles - t0 < p.chunk ? p.tiles - t0 : p.chunk;
    const int64_t q0 = 32 * t0, nq = n - q0 < 32 * nt ? n - q0 : 32 * nt;
    const dim3 grid((unsigned)((nt + 4 * p.nq - 1) / (4 * p.nq)), (unsigned)p.slices);
#define SC_SCREEN(DPV, NQV, COL)                                                                                      \
  hipLaunchKernelGGL((screen_kernel<DPV, NQV, COL>), grid, dim3(kMt), 0, st, xb, half, n, p.tiles, t0, nt, p.slices, \
                     scale, maxima, tau, p.cap, count, list)
#define SC_SCREEN_DIM(COL)                                       \
  do {                                                           \
    if (p.dpb == 16) SC_SCREEN(16, 4, COL);                      \
    else if (p.dpb == 32) SC_SCREEN(32, 4, COL);                 \
    else if (p.dpb == 64) SC_SCREEN(64, 2, COL);                 \
    else SC_SCREEN(128, 2, COL);                                 \
  } while (0)
    SC_SCREEN_DIM(false);
#define SC_THRESHOLD(NPV)                                                                                              \
  hipLaunchKernelGGL((screen_threshold_kernel<NPV>), dim3(blocks(nq * 64)), dim3(kT), 0, st, maxima, p.slices * 16, k, \
                     p.dpb, norm, q0, nq, nrm2, p.cap, scale, tau, count, *bound, lost_count)
    if (p.slices <= 4) SC_THRESHOLD(1);
    else if (p.slices <= 8) SC_THRESHOLD(2);
    else if (p.slices <= 16) SC_THRESHOLD(4);
    else if (p.slices <= 32) SC_THRESHOLD(8);
    else SC_THRESHOLD(16);
#undef SC_THRESHOLD
    // most queries lost: the second pass would be for nothing, an empty list sends them all to the fp64 kernel
    e = hipMemcpyAsync(host, lost_count, sizeof(int32_t) * kLostInts, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    int64_t lost = -lost_before;
    for (int q = 0; q < kLostSlots; ++q) lost += host[q * kLostStride];
    lost_before += lost;
    if (lost <= nq / 2) SC_SCREEN_DIM(true);
#undef SC_SCREEN_DIM
#undef SC_SCREEN
    hipLaunchKernelGGL(screen_rank_kernel, dim3(blocks(nq * 64)), dim3(kT), rank_lds, st, xp, dp, q0, nq, k, p.cap, count,
                       list, flag, *tiles, *ntiles, idx_out, dist_out);
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

size_t knn_pairs_workspace(int64_t n) {
  size_t scan_bytes = 0;
  (void)rocprim::exclusive_scan(nullptr, scan_bytes, (const int32_t*)nullptr, (int32_t*)nullptr, (int32_t)0, (size_t)n,
                                rocprim::plus<int32_t>(), (hipStream_t) nullptr);
  return (scan_bytes + 255) / 256 * 256 + 2 * (size_t)n * sizeof(int32_t) + 256;
}

hipError_t launch_knn_union_pairs(const int32_t* idx, const double* dist, int64_t n, int k, double sigma, void* work,
                                  size_t work_bytes, int32_t* eu, int32_t* ev, double* val, int32_t* last_two,
                                  hipStream_t st) {
  if (n < 1 || k < 1 || n > INT32_MAX || n * k > INT32_MAX) return hipErrorInvalidValue;
  size_t scan_bytes = 0;
  hipError_t e = rocprim::exclusive_scan(nullptr, scan_bytes, (const int32_t*)nullptr, (int32_t*)nullptr, (int32_t)0,
                                         (size_t)n, rocprim::plus<int32_t>(), st);
  if (e != hipSuccess) return e;
  const size_t tmp = (scan_bytes + 255) / 256 * 256;
  if (work_bytes < tmp + 2 * (size_t)n * sizeof(int32_t)) return hipErrorInvalidValue;
  char* base = static_cast<char*>(work);
  int32_t* cnt = reinterpret_cast<int32_t*>(base + tmp);
  int32_t* off = cnt + n;
  hipLaunchKernelGGL(pair_count_kernel, dim3(blocks(n)), dim3(kT), 0, st, idx, n, k, cnt);
  size_t sb = scan_bytes;
  e = rocprim::exclusive_scan(base, sb, cnt, off, (int32_t)0, (size_t)n, rocprim::plus<int32_t>(), st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pair_emit_kernel, dim3(blocks(n)), dim3(kT), 0, st, idx, dist, n, k, off,
                     sigma > 0.0 ? 1.0 / (2.0 * sigma * sigma) : 0.0, eu, ev, val);
  // the pair count = off[n-1] + cnt[n-1]: both handed back for the host to add
  e = hipMemcpyAsync(last_two, off + (n - 1), sizeof(int32_t), hipMemcpyDeviceToDevice, st);
  if (e != hipSuccess) return e;
  e = hipMemcpyAsync(last_two + 1, cnt + (n - 1), sizeof(int32_t), hipMemcpyDeviceToDevice, st);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace sceig
