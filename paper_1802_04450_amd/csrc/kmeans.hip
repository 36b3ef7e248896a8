// k-means on the rows of the eigenvector matrix (paper Section II Step 4, Section IV-C, Algorithms 4 and 5): device
// kernels.  The distance step is the paper's expanded form S = |v|^2 + |c|^2 - 2 V C^T with the product on the fp64
// matrix cores and the arg-min in the same launch (label_kernel, kernels.hip); |v|^2 does not change the arg-min and is left out.
// The centre update is sort based as in the paper (points ordered by label, every cluster a contiguous run), with a fixed summation
// order so that results are reproducible.  The seeding follows Algorithm 5 with uniform numbers from a counter-based
// generator; a draw is one distance pass that also leaves block sums and a walk over the sums, level by level, to the
// drawn point: all draws in one launch where its workgroups are all on the chip (seed_draws_kernel), else a launch or two
// a draw.
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

namespace sceig {
namespace {

constexpr int kT = 256;
inline unsigned blocks(int64_t n) { return (unsigned)((n + kT - 1) / kT); }

// X[i, t] (row-major, leading dimension ldx >= d, zero padded) from the caller's points: coordinate t of point i at
// v[t * ldv + i] (column-major, the eigenvector output) or v[i * ldv + t] (row-major).  64 x 64 tiles through LDS so
// that reads and writes both run over consecutive addresses in the column-major case.
__global__ __launch_bounds__(kT) void points_to_rowmajor_kernel(const double* __restrict__ v, int64_t ldv, int colmajor,
                                                                int64_t n, int d, double* __restrict__ x,
                                                                int64_t ldx) {
  __shared__ double tile[64][65];
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int t0 = blockIdx.y * 64;
  for (int idx = threadIdx.x; idx < 64 * 64; idx += kT) {
    // column-major source: consecutive threads walk the points; row-major source: they walk the coordinates
    const int a = idx / 64, b = idx % 64;
    const int64_t i = i0 + (colmajor ? b : a);
    const int t = t0 + (colmajor ? a : b);
    double val = 0.0;
    if (i < n && t < d) val = colmajor ? v[(int64_t)t * ldv + i] : v[i * ldv + t];
    tile[colmajor ? b : a][colmajor ? a : b] = val;  // tile[point][coordinate]
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 64 * 64; idx += kT) {
    const int r = idx / 64, c = idx % 64;
    if (i0 + r < n && t0 + c < ldx) x[(i0 + r) * ldx + t0 + c] = tile[r][c];
  }
}

// *out = the sum of one value per thread of the workgroup, in a fixed order
__device__ __forceinline__ void block_norm(double ss, double* __restrict__ out) {
  __shared__ double wsum[kT / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if (threadIdx.x % 64 == 0) wsum[threadIdx.x / 64] = ss;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
    for (int w = 0; w < kT / 64; ++w) tot += wsum[w];
    *out = tot;
  }
}

// ct[t * ldc + j] = c[j * ldx + t] (the right-hand operand of V C^T, zero padded to dpad rows), cnorm[j] = |c_j|^2, and
// the count of changed labels cleared.  One workgroup per centre.
__global__ __launch_bounds__(kT) void centroid_operand_kernel(const double* __restrict__ c, int64_t ldx, int d, int dpad,
                                                              double* __restrict__ ct, int64_t ldc,
                                                              double* __restrict__ cnorm, int* __restrict__ changes) {
  const int j = blockIdx.x;
  if (j == 0 && threadIdx.x < kChangeSlots) changes[threadIdx.x * kChangeStride] = 0;
  double ss = 0.0;
  for (int t = threadIdx.x; t < dpad; t += kT) {
    const double val = t < d ? c[(int64_t)j * ldx + t] : 0.0;
    ct[(int64_t)t * ldc + j] = val;
    ss += val * val;
  }
  block_norm(ss, cnorm + j);
}

__global__ __launch_bounds__(kT) void iota_fill_kernel(int32_t* __restrict__ a, int64_t n, int32_t value, int use_iota) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < n) a[i] = use_iota ? (int32_t)i : value;
}

// ---- grouping the points by label --------------------------------------------------------------------------------
// A stable counting sort in three launches: every block of 1,024 points counts its labels, a wave per cluster turns the
// counts into offsets, and the blocks write their points' indices in order.  (The library's radix sort of (label, index)
// pairs takes ten launches, 49 us at 100,000 points and 100 clusters; these three take 12 us.)  Up to kMaxBins
// clusters; beyond, a block's counters no longer fit the LDS and the radix sort is used.  A label outside [0, k), which
// only points without a finite distance have, belongs to no cluster.
constexpr int kMaxBins = 1024;
constexpr int kSortBlock = 4 * kT;

// The labelling's counts to the host's memory, by one wave (see launch_centroid_update).
// changes[kChangeSum], for the launches behind it: the labels changed; if none has, they leave everything as it is.
__device__ __forceinline__ void report_labelling(int* __restrict__ changes, const LabelReport& report) {
  int sum = changes[(threadIdx.x & 63) * kChangeStride];
  static_assert(kChangeSlots == 64, "a lane per slot");
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0) {
    changes[kChangeSum] = sum;
    put_host(report.host, sum);
    put_host(report.host + 1, changes[kChangeUndecided]);
    host_written();
    put_host(report.host + 2, report.number);
  }
}
__global__ __launch_bounds__(64) void label_report_kernel(int* __restrict__ changes, LabelReport report) {
  report_labelling(changes, report);
}

__global__ __launch_bounds__(kT) void label_count_kernel(const int32_t* __restrict__ label, int64_t n, int k, int nb,
                                                         int32_t* __restrict__ count, int* __restrict__ changes,
                                                         LabelReport report) {
  __shared__ int bin[kMaxBins];
  if (blockIdx.x == 0 && threadIdx.x < 64) report_labelling(changes, report);
  for (int c = threadIdx.x; c < k; c += kT) bin[c] = 0;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t i = (int64_t)blockIdx.x * kSortBlock + u * kT + threadIdx.x;
    if (i < n && (uint32_t)label[i] < (uint32_t)k) atomicAdd(&bin[label[i]], 1);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < k; c += kT) count[(int64_t)c * nb + blockIdx.x] = bin[c];
}

// count[c][.] becomes its exclusive prefix sum, total[c] the sum.  A wave per cluster.
__global__ __launch_bounds__(kT) void label_offset_kernel(int32_t* __restrict__ count, int k, int nb,
                                                          int32_t* __restrict__ total, const int* __restrict__ changed) {
  if (*changed == 0) return;
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
  if (c >= k) return;
  int32_t* row = count + (int64_t)c * nb;
  int sum = 0;
  for (int b0 = 0; b0 < nb; b0 += 64) {
    const int mine = b0 + lane < nb ? row[b0 + lane] : 0;
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    if (b0 + lane < nb) row[b0 + lane] = sum + incl - mine;
    sum += __shfl(incl, 63, 64);
  }
  if (lane == 0) total[c] = sum;
}

// start[c] = first position of cluster c, start[k] = number of grouped points; member[p] = the points in label order,
// ascending within a label
__global__ __launch_bounds__(kT) void label_scatter_kernel(const int32_t* __restrict__ label, int64_t n, int k, int bits,
                                                           int nb, const int32_t* __restrict__ count,
                                                           const int32_t* __restrict__ total,
                                                           int32_t* __restrict__ start, int32_t* __restrict__ member,
                                                           const int* __restrict__ changed) {
  if (*changed == 0) return;
  __shared__ int base[kT / 64][kMaxBins];
  __shared__ int wave_sum[kT / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t w0 = (int64_t)blockIdx.x * kSortBlock + wave * 256;  // the wave's 256 points
  for (int c = lane; c < k; c += 64) base[wave][c] = 0;
  __syncthreads();
  int lab[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t i = w0 + 64 * u + lane;
    lab[u] = i < n ? label[i] : -1;
    if ((uint32_t)lab[u] >= (uint32_t)k) lab[u] = -1;
    if (lab[u] >= 0) atomicAdd(&base[wave][lab[u]], 1);
  }
  // where every cluster starts: thread t has the clusters 4 t .. 4 t + 3
  int own[4], sum = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = 4 * (int)threadIdx.x + q;
    own[q] = c < k ? total[c] : 0;
    sum += own[q];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  int first = incl - sum;
  for (int w = 0; w < wave; ++w) first += wave_sum[w];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = 4 * (int)threadIdx.x + q;
    if (c < k) {
      if (blockIdx.x == 0) {
        start[c] = first;
        if (c == k - 1) start[k] = first + own[q];
      }
      int at = first + count[(int64_t)c * nb + blockIdx.x];
#pragma unroll
      for (int w = 0; w < kT / 64; ++w) {
        const int here = base[w][c];
        base[w][c] = at;
        at += here;
      }
    }
    first += own[q];
  }
  __syncthreads();
  // from here on a wave touches its own row of `base` only, one batch of 64 points after the other
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    uint64_t same = __ballot(lab[u] >= 0);
    for (int bit = 0; bit < bits; ++bit) {
      const bool set = (lab[u] >> bit) & 1;
      const uint64_t with = __ballot(set);
      same &= set ? with : ~with;
    }
    if (lab[u] >= 0) {
      const int rank = __popcll(same & ((1ull << lane) - 1ull));
      const int at = base[wave][lab[u]];
      member[at + rank] = (int32_t)(w0 + 64 * u + lane);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // every lane has read before the first of a label adds
      if (rank == 0) base[wave][lab[u]] = at + __popcll(same);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// start[c] = first position in the sorted label array with label >= c, c = 0 .. k
__global__ __launch_bounds__(kT) void cluster_starts_kernel(const int32_t* __restrict__ sorted_label, int64_t n, int k,
                                                            int32_t* __restrict__ start) {
  const int c = blockIdx.x * kT + threadIdx.x;
  if (c > k) return;
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (sorted_label[mid] < c) {
      lo = mid + 1;
    } else {
      hi = mid;
    }
  }
  start[c] = (int32_t)lo;
}

// part[(j * parts + q) * ldx + t] = sum over the q-th of `parts` equal pieces of cluster j's points.  Workgroup (j, q,
// column tile of 2 DL): DL lanes carry two columns each, the 256 / DL slots take every so many-th point of the piece,
// four in flight, and their sums are added in slot order.  One workgroup per cluster and 64 columns, a chain of one
// point's index and row after the other, took 194 us at 100,000 points, 100 coordinates and 100 clusters, this takes
// 17 us: 80 MB from the Infinity Cache.
template <int DL>
__global__ __launch_bounds__(kT) void cluster_sum_kernel(const double* __restrict__ x, int64_t ldx,
                                                         const int32_t* __restrict__ member,
                                                         const int32_t* __restrict__ start, int parts,
                                                         double* __restrict__ part, const int* __restrict__ changed) {
  if (*changed == 0) return;
  constexpr int S = kT / DL;
  __shared__ double2 red[kT];
  const int j = blockIdx.x, q = blockIdx.y;
  const int t = ((int)blockIdx.z * DL + (int)threadIdx.x % DL) * 2, slot = threadIdx.x / DL;
  const int m0 = start[j], len = start[j + 1] - m0;
  const int a = m0 + (int)((int64_t)len * q / parts), b = m0 + (int)((int64_t)len * (q + 1) / parts);
  double2 acc = make_double2(0.0, 0.0);
  if (t < ldx) {
    int m = a + slot;
    for (; m + 3 * S < b; m += 4 * S) {
      double2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const double2*>(x + (int64_t)member[m + u * S] * ldx + t);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        acc.x += v[u].x;
        acc.y += v[u].y;
      }
    }
    for (; m < b; m += S) {
      const double2 v = *reinterpret_cast<const double2*>(x + (int64_t)member[m] * ldx + t);
      acc.x += v.x;
      acc.y += v.y;
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  if (slot == 0 && t < ldx) {
#pragma unroll 8
    for (int s = 1; s < S; ++s) {
      const double2 v = red[s * DL + threadIdx.x];
      acc.x += v.x;
      acc.y += v.y;
    }
    *reinterpret_cast<double2*>(part + ((int64_t)j * parts + q) * ldx + t) = acc;
  }
}

// c[j, :] = mean of the points of cluster j from the sums of its pieces, added in order; an empty cluster keeps its
// centre.  What the next labelling needs is made on the way (see centroid_operand_kernel), and its count of changes is
// cleared.  One workgroup per centre.
__global__ __launch_bounds__(kT) void centroid_finish_kernel(const double* __restrict__ part, int parts,
                                                             const int32_t* __restrict__ start, int d, int64_t ldx,
                                                             double* __restrict__ c, double* __restrict__ ct, int64_t ldc,
                                                             double* __restrict__ cnorm, int* __restrict__ changes) {
  if (changes[kChangeSum] == 0) return;  // then the slots are zero
  const int j = blockIdx.x;
  if (j == 0 && threadIdx.x < kChangeSlots) changes[threadIdx.x * kChangeStride] = 0;
  const int len = start[j + 1] - start[j];
  double ss = 0.0;
  for (int t = threadIdx.x; t < ldx; t += kT) {
    double v = t < d ? c[(int64_t)j * ldx + t] : 0.0;
    if (len > 0 && t < d) {
      v = 0.0;
#pragma unroll 4
      for (int q = 0; q < parts; ++q) v += part[((int64_t)j * parts + q) * ldx + t];
      v /= (double)len;
      c[(int64_t)j * ldx + t] = v;
    }
    ct[(int64_t)t * ldc + j] = v;
    ss += v * v;
  }
  block_norm(ss, cnorm + j);
}

// ---- seeding -------------------------------------------------------------------------------------------------------
// A draw's distance pass: dist2[i] = |x_i - x_c|^2 (first) or min(dist2[i], |x_i - x_c|^2), c = *centre, and bsum[block] =
// the sum of the block's 64 values of dist2 in a fixed order.  All draws but the first leave out the points whose distance
// cannot shrink, by a bf16 copy of the points, a quarter of their bytes: with err_i >= |x_i - x~_i| (seed_copy_kernel), the
// distance is at least |x~_i - x~_c| - err_i - err_c, and if that is no less than the distance kept, the minimum stands.
// What is left is computed in fp64 as before, by 16 lanes per point, so the distances are the same to the last bit.  The
// copies are scaled by a power of two that takes the largest coordinate into [1, 2) (seed_mean_kernel), so that their
// float distance cannot overflow; it is taken to be off by (d + 8) 2^-23 of itself, which holds down to a square of
// kScreenFloor (below, what single squares lose to the denormal numbers is no longer negligible), and the lower bound has
// to exceed the distance kept by 1e-6 of it: more than the fp64 sums are off.  A NaN on the way fails the test and the
// point is computed; so is every point of data that have no such scale (scale 0: copies of zeros).
// Per draw at 100,000 points of 100 coordinates: 18.7 us reading 80 MB, 11.3 us with the copy, which an XCD's L2 keeps
// its part of from draw to draw (21 MB in all); what is left is the chain centre, its row, the point's row.  (Leaving points out
// by the triangle inequality with a kept assignment did not shorten the pass: it saves no load of the first row.)
constexpr int kSeedPoints = 64;   // points per block
constexpr int kExactLanes = 16;
// Up to this many blocks a pass finds its centre by itself: every workgroup reads all block sums once more, which then
// costs less than the launch of a kernel that does it for all (whole seeding at 100,000 points of 100 coordinates, 100
// draws: 1.64 against 1.88 ms; at 140,000 of 128, 128 draws: 2.82 against 2.64 ms).
constexpr int64_t kDrawBlocks = 1800;

// Two blocks a workgroup and a thread's copies requested before the draw, from kSeedWide blocks on and up to kSeedWideDim
// coordinates.  A draw inside the pass, us with one block / two / four: 80,000 x 100 11.1 / 10.0 / 10.9, 100,000 x 100 12.6 / 11.3 /
// 11.3, 115,000 x 64 11.2 / 10.4 / 10.3; fewer blocks leave the chip idle (60,000 x 100 9.7 / 9.2 / 10.5, 40,000 x 100 8.8 / 8.8 /
// 10.3), and with 128 coordinates the registers do (60,000 9.4 / 9.5 / 11.0, 100,000 11.5 / 11.4 / 11.6).  Without a draw inside:
// 140,000 x 32 12.2 / 11.5 / 12.1, 600,000 x 16 24.2 / 18.7 / 18.3, 200,000 x 100 21.1 / 19.1 / 22.1, of 128 18.3 / 21.9 / 26.6.
constexpr int64_t kSeedWide = 1024;
constexpr int kSeedWideDim = 112;
constexpr float kScreenFloor = 1e-30f;

// xh[i] = the centred and scaled point in bf16, padded with zeros to dpb coordinates (a multiple of 8); err[i] as above,
// rounded up, and beside it the exponent of the scale.  mean: any point will do (exactness does not depend on it); a bf16
// value is off by 2^-9 of its modulus at most, the centring by 2^-52 of the coordinates.  8 lanes per point.
__global__ __launch_bounds__(kT) void seed_copy_kernel(const double* __restrict__ x, int64_t ldx, int d, int64_t n,
                                                       const double* __restrict__ mean, const double* __restrict__ scale,
                                                       int dpb, __bf16* __restrict__ xh, float2* __restrict__ err) {
  const int lane = threadIdx.x % 8;
  const int64_t i = (int64_t)blockIdx.x * (kT / 8) + threadIdx.x / 8;
  if (i >= n) return;  // uniform over the point's lanes
  const double f = *scale;
  double moved = 0.0, size = 0.0;
  for (int c0 = lane * 8; c0 < dpb; c0 += 64) {
    union { __bf16 b[8]; uint4 v; } piece;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int t = c0 + q;
      const double xv = t < d ? x[i * ldx + t] : 0.0, mv = t < d ? mean[t] : 0.0;
      const double v = xv * f, m = mv * f, y = v - m;
      piece.b[q] = (__bf16)(float)y;
      const double off = y - (double)(float)piece.b[q];
      moved += off * off;
      size += v * v + m * m;
    }
    *reinterpret_cast<uint4*>(xh + i * dpb + c0) = piece.v;
  }
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) {
    moved += __shfl_xor(moved, o, 8);
    size += __shfl_xor(size, o, 8);
  }
  if (lane == 0)
    err[i] = make_float2((float)((sqrt(moved) + 4.5e-16 * sqrt(size)) * 1.00001) + 1e-37f, f > 0.0 ? (float)ilogb(f) : 0.0f);
}

// mean[t] of the points, in two steps with a fixed order: part[b][t] over the points b, b + gridDim.x, ..., top[b] = the
// upper word of their largest modulus of a coordinate (the exponent is all that is needed)
constexpr int kSeedParts = kT;
__global__ __launch_bounds__(kT) void seed_sum_kernel(const double* __restrict__ x, int64_t ldx, int64_t n,
                                                      double* __restrict__ part, uint32_t* __restrict__ top) {
  __shared__ uint32_t most_of_all;
  uint32_t most = 0u;
  if (threadIdx.x == 0) most_of_all = 0u;
  __syncthreads();
  for (int t = threadIdx.x; t < ldx; t += kT) {
    double acc = 0.0;
#pragma unroll 8
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
      const double v = x[i * ldx + t];
      const uint32_t m = (uint32_t)__double2hiint(v) & 0x7fffffffu;
      acc += v;
      most = m > most ? m : most;
    }
    part[(int64_t)blockIdx.x * ldx + t] = acc;
  }
  atomicMax(&most_of_all, most);
  __syncthreads();
  if (threadIdx.x == 0) top[blockIdx.x] = most_of_all;
}

// the second step; *scale = the power of two that takes the largest modulus into [1, 2), 0 where the squares of such
// numbers leave the range of a double (or one of them is no number)
__global__ __launch_bounds__(kT) void seed_mean_kernel(const double* __restrict__ part, const uint32_t* __restrict__ top,
                                                       int parts, int64_t ldx, int64_t n, double* __restrict__ mean,
                                                       double* __restrict__ scale) {
  if (blockIdx.x == 0) {
    __shared__ uint32_t most_of_all;
    if (threadIdx.x == 0) most_of_all = 0u;
    __syncthreads();
    atomicMax(&most_of_all, top[threadIdx.x]);
    __syncthreads();
    const int e = (int)(most_of_all >> 20) - 1023;
    if (threadIdx.x == 0) *scale = e > -330 && e < 330 ? ldexp(1.0, -e) : 0.0;
  }
  const int t = blockIdx.x * kT + threadIdx.x;
  if (t >= ldx) return;
  double acc = 0.0;
#pragma unroll 8
  for (int b = 0; b < parts; ++b) acc += part[(int64_t)b * ldx + t];
  mean[t] = acc / (double)n;
}

// Inclusive prefix sums of one value per lane over the wave (fixed shuffle tree).
__device__ __forceinline__ double wave_inclusive(double v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double up = __shfl_up(v, o, 64);
    if (lane >= o) v += up;
  }
  return v;
}

// The first position p in [0, count) with base + (v(0) + ... + v(p)) > r, searched by one wave in pieces of 64; *base
// receives the sum before that position.  -1 if there is none (then *base = base + the whole sum).
template <class Values>
__device__ int wave_first_exceeding(Values v, int64_t count, double r, double* base, int lane) {
  double acc = *base;
  for (int64_t p0 = 0; p0 < count; p0 += 64) {
    const double mine = p0 + lane < count ? v(p0 + lane) : 0.0;
    const double incl = wave_inclusive(mine, lane) + acc;
    const bool hit = p0 + lane < count && incl > r;
    const uint64_t mask = __ballot(hit);
    if (mask) {
      const int l = __ffsll((long long)mask) - 1;
      *base = __shfl(incl - mine, l, 64);
      return (int)p0 + l;
    }
    acc = __shfl(incl, 63, 64);
  }
  *base = acc;
  return -1;
}

// Algorithm 5's draw by one workgroup of T threads: total = sum of all dist2 (through the block sums), r = u * total, and
// the first point whose inclusive prefix sum exceeds r, found level by level: the threads each sum a contiguous run of
// block sums, their prefix sums name the run, one wave then finds the block inside the run and the point inside the
// block.  Every sum has a fixed order.  If rounding makes a level miss (the finer sums fall short of the coarser
// one) the last block / point of that level is taken; if no run qualifies (total = 0) the last point, as the
// definition says.  Every thread gets the point.
template <int T>
__device__ int64_t draw_point(const double* __restrict__ bsum, int64_t nb, const double* __restrict__ dist2, int64_t n,
                              double u) {
  __shared__ double wave_tot[T / 64];
  __shared__ double excl[T];
  __shared__ int first_run;
  __shared__ int32_t drawn;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t chunk = (nb + T - 1) / T;
  const int64_t j0 = (int64_t)t * chunk;
  int64_t j1 = j0 + chunk;
  j1 = j1 < nb ? j1 : nb;
  double run = 0.0;
#pragma unroll 4
  for (int64_t j = j0; j < j1; ++j) run += bsum[j];
  const double incl_w = wave_inclusive(run, lane);
  if (lane == 63) wave_tot[wave] = incl_w;
  if (t == 0) first_run = T;
  __syncthreads();
  double offset = 0.0, total = 0.0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    if (w < wave) offset += wave_tot[w];
    total += wave_tot[w];
  }
  const double incl = incl_w + offset;
  excl[t] = incl - run;
  const double r = u * total;
  if (j0 < j1 && incl > r) atomicMin(&first_run, t);
  __syncthreads();
  if (wave == 0) {
    const int tr = first_run;
    int32_t at = (int32_t)(n - 1);  // nothing exceeds r: all distances are zero (or u * total rounded up to the total)
    if (tr < T) {
      const int64_t b0 = (int64_t)tr * chunk;
      int64_t b1 = b0 + chunk;
      b1 = b1 < nb ? b1 : nb;
      double base = excl[tr];
      bool missed = false;
      int jb = wave_first_exceeding([&](int64_t p) { return bsum[b0 + p]; }, b1 - b0, r, &base, lane);
      if (jb < 0) {  // the run's own sum exceeded r but its block sums, added up one by one, do not: take its last block
        jb = (int)(b1 - b0) - 1;
        missed = true;
      }
      const int64_t p0 = (b0 + jb) * kSeedPoints;
      int64_t p1 = p0 + kSeedPoints;
      p1 = p1 < n ? p1 : n;
      int jp = missed ? -1 : wave_first_exceeding([&](int64_t p) { return dist2[p0 + p]; }, p1 - p0, r, &base, lane);
      if (jp < 0) jp = (int)(p1 - p0) - 1;
      at = (int32_t)(p0 + jp);
    }
    if (lane == 0) drawn = at;
  }
  __syncthreads();
  return drawn;
}

constexpr int kSelectThreads = 1024;
__global__ __launch_bounds__(kSelectThreads) void seed_select_kernel(const double* __restrict__ bsum, int64_t nb,
                                                                     const double* __restrict__ dist2, int64_t n, double u,
                                                                     int32_t* __restrict__ chosen) {
  const int64_t at = draw_point<kSelectThreads>(bsum, nb, dist2, n, u);
  if (threadIdx.x == 0) *chosen = (int32_t)at;
}

// What lane `lane` of kExactLanes adds to the squared distance of two rows of d doubles: its coordinates in order, E of either row
// on their way before the first is used.  (One after the other they were what a draw lasted: 100,000 x 100, 100 draws 1,520 ->
// 1,335 us; rows like those of an embedding, most workgroups with a point to compute, 3,220 -> 2,095.)
template <int E>
__device__ __forceinline__ double lane_square(const double* __restrict__ x, const double* __restrict__ y, int d, int lane) {
  double acc = 0.0;
  for (int base = lane; base - lane < d; base += E * kExactLanes) {
    double a[E], b[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int t = base + e * kExactLanes < d ? base + e * kExactLanes : 0;
      a[e] = x[t];
      b[e] = y[t];
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const double diff = base + e * kExactLanes < d ? a[e] - b[e] : 0.0;
      acc += diff * diff;
    }
  }
  return acc;
}

// Whether the distance kept stands, by the screen's squared distance of the copies.
__device__ __forceinline__ bool distance_stands(float acc, int d, float2 own_err, double centre_err, double kept) {
  const double low = sqrt((double)acc) * (1.0 - (d + 8) * 1.1920928955078125e-07) - (double)own_err.x - centre_err;
  const double l = ldexp(low, -(int)own_err.y);
  return acc >= kScreenFloor && low > 0.0 && l * l >= kept * (1.0 + 1e-6);
}
// The squared distance of two rows by kExactLanes lanes (each gets it).
__device__ __forceinline__ double row_square(const double* __restrict__ xi, const double* __restrict__ xc, int d, int lane) {
  double acc = d <= kExactLanes       ? lane_square<1>(xi, xc, d, lane)
               : d <= 2 * kExactLanes ? lane_square<2>(xi, xc, d, lane)
               : d <= 4 * kExactLanes ? lane_square<4>(xi, xc, d, lane)
                                      : lane_square<8>(xi, xc, d, lane);
#pragma unroll
  for (int o = kExactLanes / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, kExactLanes);
  return acc;
}

// The pass for the centre *centre (DRAW false), or for the centre that this draw itself takes from the distances before it
// (DRAW true; every workgroup finds it for itself from the block sums, workgroup 0 writes it down): dist2 and bsum go from
// one buffer to the other.
// SUB blocks per workgroup.  AHEAD (up to 128 coordinates): a thread requests its points' copies before the draw, which does
// not concern them.
template <bool SCREEN, bool DRAW, int SUB, bool AHEAD>
__global__ __launch_bounds__(kT) void seed_distance_kernel(const double* __restrict__ x, int64_t ldx, int d, int64_t n,
                                                           const __bf16* __restrict__ xh, int dpb,
                                                           const float2* __restrict__ err, double u,
                                                           int32_t* __restrict__ centre, int first,
                                                           const double* __restrict__ bsum_in, int64_t nb,
                                                           const double* __restrict__ dist2_in,
                                                           double* __restrict__ dist2, double* __restrict__ bsum) {
  constexpr int SL = 4;  // lanes per point of the screen: 64 points at a time
  constexpr int EP = kSeedPoints / (kT / kExactLanes);  // points per 16 lanes
  constexpr int P = SUB * kSeedPoints;
  static_assert(SUB <= kT / 64, "a wave per block sum");
  static_assert(SCREEN || SUB == 1, "the unscreened pass takes one block");
  __shared__ double pts[P];
  __shared__ int todo[P];
  __shared__ int ntodo;
  const int64_t i0 = (int64_t)blockIdx.x * P;
  const int here = n - i0 < P ? (int)(n - i0) : P;
  if (threadIdx.x == 0) ntodo = 0;
  if (threadIdx.x < P) pts[threadIdx.x] = threadIdx.x < here && !first ? dist2_in[i0 + threadIdx.x] : 0.0;
  const int sp = threadIdx.x / SL, sl = threadIdx.x % SL;
  union Piece { __bf16 b[8]; uint4 v; };
  Piece ahead[AHEAD ? SUB : 1][4];
  float2 own_err[SUB];
  if constexpr (AHEAD) {
#pragma unroll
    for (int r = 0; r < SUB; ++r) {
      const int p = sp + r * kSeedPoints;
      const int64_t i = i0 + (p < here ? p : here - 1);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = sl * 8 + v * SL * 8;
        ahead[r][v].v = *reinterpret_cast<const uint4*>(xh + i * dpb + (t < dpb ? t : 0));
      }
      own_err[r] = err[i];
    }
  }
  int64_t c;
  if constexpr (DRAW) {
    c = draw_point<kT>(bsum_in, nb, dist2_in, n, u);
    if (blockIdx.x == 0 && threadIdx.x == 0) *centre = (int32_t)c;
  } else {
    c = *centre;
    __syncthreads();
  }
  const int lane = threadIdx.x % kExactLanes, group = threadIdx.x / kExactLanes;
  if constexpr (SCREEN) {
    float acc[SUB];
#pragma unroll
    for (int r = 0; r < SUB; ++r) acc[r] = 0.0f;
    if constexpr (AHEAD) {
      Piece b[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = sl * 8 + v * SL * 8;
        b[v].v = *reinterpret_cast<const uint4*>(xh + c * dpb + (t < dpb ? t : 0));
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (v * SL * 8 >= dpb) break;  // uniform
        const bool in = sl * 8 + v * SL * 8 < dpb;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float bq = (float)b[v].b[q];
#pragma unroll
          for (int r = 0; r < SUB; ++r) {
            const float diff = in ? (float)ahead[r][v].b[q] - bq : 0.0f;
            acc[r] += diff * diff;
          }
        }
      }
    } else {
#pragma unroll
      for (int r = 0; r < SUB; ++r) {
        const int p = sp + r * kSeedPoints;
        const int64_t i = i0 + (p < here ? p : here - 1);
        own_err[r] = err[i];
#pragma unroll 4
        for (int t = sl * 8; t < dpb; t += SL * 8) {
          Piece a, b;
          a.v = *reinterpret_cast<const uint4*>(xh + i * dpb + t);
          b.v = *reinterpret_cast<const uint4*>(xh + c * dpb + t);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float diff = (float)a.b[q] - (float)b.b[q];
            acc[r] += diff * diff;
          }
        }
      }
    }
    const double centre_err = (double)err[c].x;
#pragma unroll
    for (int r = 0; r < SUB; ++r) {
      const int p = sp + r * kSeedPoints;
#pragma unroll
      for (int o = SL / 2; o > 0; o >>= 1) acc[r] += __shfl_xor(acc[r], o, SL);
      if (sl == 0 && p < here) {
        const float2 mine = own_err[r];
        if (!distance_stands(acc[r], d, mine, centre_err, pts[p])) todo[atomicAdd(&ntodo, 1)] = p;
      }
    }
    __syncthreads();
    const int count = ntodo;
    for (int s = group; s < count; s += kT / kExactLanes) {  // uniform over the point's lanes
      const int pt = todo[s];
      const double acc2 = row_square(x + (i0 + pt) * ldx, x + c * ldx, d, lane);
      if (lane == 0 && acc2 < pts[pt]) pts[pt] = acc2;
    }
  } else {  // the lanes take their four points together
    double acc[EP];
#pragma unroll
    for (int q = 0; q < EP; ++q) acc[q] = 0.0;
    for (int t = lane; t < d; t += kExactLanes) {
      const double cv = x[c * ldx + t];
#pragma unroll
      for (int q = 0; q < EP; ++q) {
        const int p = group + q * (kT / kExactLanes);
        const double diff = x[(i0 + (p < here ? p : here - 1)) * ldx + t] - cv;
        acc[q] += diff * diff;
      }
    }
#pragma unroll
    for (int q = 0; q < EP; ++q) {
#pragma unroll
      for (int o = kExactLanes / 2; o > 0; o >>= 1) acc[q] += __shfl_xor(acc[q], o, kExactLanes);
      const int p = group + q * (kT / kExactLanes);
      if (lane == 0 && p < here && (first || acc[q] < pts[p])) pts[p] = acc[q];
    }
  }
  __syncthreads();
  if (threadIdx.x < P) {  // whole waves: one per block
    double tot = pts[threadIdx.x];
    if (threadIdx.x < here) dist2[i0 + threadIdx.x] = tot;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tot += __shfl_xor(tot, o, 64);
    const int64_t block = (int64_t)blockIdx.x * SUB + (threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0 && block < nb) bsum[block] = tot;
  }
}

// ---- all draws in one launch -----------------------------------------------------------------------------------------
// A draw's pass is short once the points are where the compute units read them fastest, and then the launch, the loads at its
// start and the wait for its last workgroup are most of it.  Here the workgroups keep their blocks of points in LDS from the
// first draw to the last (the bf16 copy with the screen, else the points), with the distances.  A workgroup's blocks are what a
// thread of draw_point adds up, so that one sum a workgroup is all that the others need to find the run of blocks that the point
// lies in: every workgroup finds it for itself, with the sums in draw_point's order, and the one that holds the run finds the point
// and tells the others (which reading the run's distances would take longer: 256 workgroups at the same lines).  Three areas of
// sums take turns: once all sums of a draw are there, all workgroups are through with those of the draw before.
// The screen takes the distance of the copies from a product, |x|^2 + |c|^2 - 2 x.c, half an instruction a coordinate instead of
// three and a half.  That is off by (d + 12) 2^-23 (|x|^2 + |c|^2) for the sums of squares and as much for the product; twice
// as much is allowed for (kScreenFloor as above).
// What is left of a draw (100,000 x 100) is the exchange, the search for the point and the loads of its row and of the rows to
// compute, each waiting for the one before.
struct SeedDraws {
  const double* x;
  int64_t ldx, n, nb;
  int d, dpb, k, per;  // per: blocks a workgroup
  const __bf16* xh;
  const float2* err;
  uint64_t key;
  double *dist2, *bsum;  // distances to the first centre, their block sums; in the end, to all centres but the last
  double* ring;          // 3 x kRunCopies x workgroups, all ones
  uint64_t* points;      // kDrawTold x 16, no draw's
  int32_t* chosen;
  uint32_t* word;  // 0 before the launch
  int* done;       // workgroups that have finished; 0: not all of them started, and nothing has been done
  int polls;
};
constexpr int kDrawThreads = 512;
constexpr int kRunCopies = 8;  // of every sum: fewer workgroups that look at the same lines (all at one: 4.4 us, at eight: 2.4)
constexpr int kDrawTold = 16;  // places that a point is told at, on lines of their own
constexpr int kDrawGroups = kT;  // workgroups: draw_point's threads
constexpr int kDrawPer = (int)((kDrawBlocks + kDrawGroups - 1) / kDrawGroups);
static_assert(kDrawPer <= kDrawThreads / 64, "a wave per block sum, a thread per distance");

constexpr int kDrawPlaces = 3 * kRunCopies * kDrawGroups + kDrawTold * 16;  // ring and points
constexpr size_t kDrawShared = kDrawPlaces * 8 + 256;                      // ... arrivals and finished workgroups
inline size_t seed_draws_lds(int per, int d, int dpb, bool screen) {
  const size_t points = (size_t)per * kSeedPoints;
  return points * (8 + 4) + (screen ? points * (12 + 2 * (size_t)dpb) : points * (size_t)d * 8);
}

// draw_point from the sums of the runs (thread t: that of run t, 0 from `runs` on); block sums and distances of the own run in
// LDS.  Draw number m.
__device__ __forceinline__ int64_t draw_from_runs(double run, int runs, int own, int per, const double* block_sum, int blocks_here,
                                                  const double* pts, int64_t n, double u, uint32_t m, uint64_t* told, int* bad) {
  __shared__ double wave_tot[kT / 64];
  __shared__ double excl[kT];
  __shared__ int first_run;
  __shared__ int32_t drawn;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const double incl_w = wave_inclusive(run, lane);
  if (lane == 63 && t < kT) wave_tot[wave] = incl_w;
  if (t == 0) first_run = kT;
  __syncthreads();
  double offset = 0.0, total = 0.0;
#pragma unroll
  for (int w = 0; w < kT / 64; ++w) {
    if (w < wave) offset += wave_tot[w];
    total += wave_tot[w];
  }
  const double incl = incl_w + offset;
  if (t < kT) excl[t] = incl - run;
  const double r = u * total;
  if (t < runs && incl > r) atomicMin(&first_run, t);
  __syncthreads();
  const int tr = first_run;
  if (wave == 0) {
    if (tr == own) {
      double base = excl[tr];
      bool missed = false;
      int jb = wave_first_exceeding([&](int64_t p) { return block_sum[p]; }, blocks_here, r, &base, lane);
      if (jb < 0) {
        jb = blocks_here - 1;
        missed = true;
      }
      const int64_t p0 = ((int64_t)own * per + jb) * kSeedPoints;
      const int here = n - p0 < kSeedPoints ? (int)(n - p0) : kSeedPoints;
      int jp = missed ? -1 : wave_first_exceeding([&](int64_t p) { return pts[jb * kSeedPoints + p]; }, here, r, &base, lane);
      if (jp < 0) jp = here - 1;
      if (lane < kDrawTold)
        __hip_atomic_store(told + lane * 16, (uint64_t)m << 32 | (uint64_t)(p0 + jp), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (lane == 0) drawn = (int32_t)(p0 + jp);
    } else if (tr < runs) {
      if (lane == 0) {
        uint64_t seen = 0;
        int looks = 0;
        do
          seen = __hip_atomic_load(told + own % kDrawTold * 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        while (seen >> 32 != m && ++looks < kLooks);
        if (seen >> 32 != m) *bad = 1;
        drawn = seen >> 32 == m ? (int32_t)(seen & 0xffffffffu) : 0;
      }
    } else if (lane == 0) {
      drawn = (int32_t)(n - 1);  // nothing exceeds r: all distances are zero (or u * total rounded up to the total)
    }
  }
  __syncthreads();
  return drawn;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
union Bf16Piece {
  bf16x2 pair[4];
  uint4 v;
};
__device__ __forceinline__ float piece_product(const Bf16Piece& a, const Bf16Piece& b, float acc) {
#pragma unroll
  for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_fdot2_f32_bf16(a.pair[q], b.pair[q], acc, false);
  return acc;
}

// The first centre's index, and the places that seed_draws_kernel's workgroups share.  It stands for the centres up to `filled`
// until they are drawn: a launch behind seed_draws_kernel that reads the points chosen finds points also where that kernel's
// workgroups have not all started, which the host only learns later.
__global__ __launch_bounds__(kT) void seed_start_kernel(int32_t* __restrict__ chosen, int32_t first, int filled,
                                                        long long* __restrict__ shared, int count, uint32_t* __restrict__ word,
                                                        uint32_t value) {
  const int t = blockIdx.x * kT + threadIdx.x;
  if (t == 0 && word) *word = value;
  for (int e = t; e < filled; e += gridDim.x * kT) chosen[e] = first;
  for (int e = t; e < count; e += gridDim.x * kT) shared[e] = -1;
}

template <bool SCREEN>
__global__ __launch_bounds__(kDrawThreads) void seed_draws_kernel(SeedDraws a) {
  extern __shared__ uint4 draw_lds[];
  __shared__ int ntodo, there, bad;
  __shared__ double block_sum[kDrawThreads / 64];
  const int d = a.d, dpb = a.dpb, tid = threadIdx.x, wave = tid >> 6, wl = tid & 63;
  const int64_t nb = a.nb;
  const int points = a.per * kSeedPoints, runs = gridDim.x;
  __bf16* const rows_h = reinterpret_cast<__bf16*>(draw_lds);  // 16 bytes apiece
  double* const rows = reinterpret_cast<double*>(draw_lds);
  double* const pts = SCREEN ? reinterpret_cast<double*>(rows_h + (size_t)points * dpb) : rows + (size_t)points * d;
  float2* const errs = reinterpret_cast<float2*>(pts + points);
  float* const norms = reinterpret_cast<float*>(errs + points);
  int* const todo = SCREEN ? reinterpret_cast<int*>(norms + points) : reinterpret_cast<int*>(errs);
  const int64_t block0 = (int64_t)blockIdx.x * a.per, i0 = block0 * kSeedPoints;
  const int here = a.n - i0 < points ? (int)(a.n - i0) : points;
  const int blocks_here = nb - block0 < a.per ? (int)(nb - block0) : a.per;
  if (tid == 0) {
    if (blockIdx.x == 0) {
      __hip_atomic_store(a.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // before anyone counts up
    }
    arrive(a.word);
    bad = 0;
    ntodo = 0;
  }
  constexpr int SL = 4;  // lanes per point of the screen
  const int sl = tid % SL;
  if constexpr (SCREEN) {
    const uint4* __restrict__ from = reinterpret_cast<const uint4*>(a.xh + i0 * dpb);
#pragma unroll 8
    for (int e = tid; e < here * (dpb / 8); e += kDrawThreads) draw_lds[e] = from[e];
  } else {
    for (int p = tid / 16; p < here; p += kDrawThreads / 16)
#pragma unroll 4
      for (int t = tid % 16; t < d; t += 16) rows[(size_t)p * d + t] = a.x[(i0 + p) * a.ldx + t];
  }
  for (int p = tid; p < points; p += kDrawThreads) {
    pts[p] = p < here ? a.dist2[i0 + p] : 0.0;
    if constexpr (SCREEN) errs[p] = p < here ? a.err[i0 + p] : make_float2(0.0f, 0.0f);
  }
  double run = 0.0;
  if (tid < runs) {
    const int64_t j0 = (int64_t)tid * a.per, j1 = j0 + a.per < nb ? j0 + a.per : nb;
    for (int64_t j = j0; j < j1; ++j) run += a.bsum[j];
  }
  if (tid < blocks_here) block_sum[tid] = a.bsum[block0 + tid];
  if (tid == 0) there = all_arrived(a.word, gridDim.x, a.polls);
  __syncthreads();
  if (!there) return;
  if constexpr (SCREEN) {
    for (int p = tid / SL; p < here; p += kDrawThreads / SL) {
      float acc = 0.0f;
      for (int t = sl * 8; t < dpb; t += SL * 8) {
        Bf16Piece own;
        own.v = *reinterpret_cast<const uint4*>(rows_h + (size_t)p * dpb + t);
        acc = piece_product(own, own, acc);
      }
#pragma unroll
      for (int o = SL / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, SL);
      if (sl == 0) norms[p] = acc;
    }
  }

  const int lane = tid % kExactLanes, group = tid / kExactLanes;
  for (int m = 1; m + 1 < a.k; ++m) {  // centre m
    if (m > 1 && tid < runs) {
      double v[1];
      if (!get(a.ring + ((m - 1) % 3 * kRunCopies + (int)blockIdx.x % kRunCopies) * runs + tid, 0, 1, v)) bad = 1;
      run = v[0];
    }
    const int64_t c = draw_from_runs(run, runs, (int)blockIdx.x, a.per, block_sum, blocks_here, pts, a.n,
                                     seed_uniform(a.key, (uint64_t)m), (uint32_t)m, a.points, &bad);
    if (bad) return;
    if (tid < kRunCopies) {
      if (m > 2)  // everyone is through with these
        __hip_atomic_store(reinterpret_cast<long long*>(a.ring + ((m - 2) % 3 * kRunCopies + tid) * runs + blockIdx.x), -1ll,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (blockIdx.x == 0 && tid == 0) a.chosen[m] = (int32_t)c;
    }
    const double* __restrict__ xc = a.x + c * a.ldx;
    if constexpr (SCREEN) {
      const float centre_err = a.err[c].x;
      const __bf16* __restrict__ hc = a.xh + c * dpb;
      const float slack = (float)(4 * d + 48) * 1.1920928955078125e-07f;
      for (int p0 = tid / SL; p0 - tid / SL < here; p0 += 4 * (kDrawThreads / SL)) {  // four points a lane
        float acc[4] = {}, own_norm = 0.0f;
#pragma unroll 4
        for (int t = sl * 8; t < dpb; t += SL * 8) {
          Bf16Piece own, b;
          b.v = *reinterpret_cast<const uint4*>(hc + t);
          own_norm = piece_product(b, b, own_norm);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int p = p0 + u * (kDrawThreads / SL);
            own.v = *reinterpret_cast<const uint4*>(rows_h + (size_t)(p < here ? p : 0) * dpb + t);
            acc[u] = piece_product(own, b, acc[u]);
          }
        }
#pragma unroll
        for (int o = SL / 2; o > 0; o >>= 1) {
          own_norm += __shfl_xor(own_norm, o, SL);
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[u] += __shfl_xor(acc[u], o, SL);
        }
        // a lane per point: the four have the same sums
        float mine = acc[0];
#pragma unroll
        for (int u = 1; u < 4; ++u) mine = sl == u ? acc[u] : mine;
        const int p = p0 + sl * (kDrawThreads / SL);
        if (p < here) {
          const float both = norms[p] + own_norm;
          const float low2 = (both - 2.0f * mine) - slack * both;
          if (!(both >= kScreenFloor) || !distance_stands(low2, d, errs[p], (double)centre_err, pts[p])) todo[atomicAdd(&ntodo, 1)] = p;
        }
      }
      __syncthreads();
      const int count = ntodo;
      for (int s = group; s < count; s += kDrawThreads / kExactLanes) {  // uniform over the point's lanes
        const int p = todo[s];
        const double acc = row_square(a.x + (i0 + p) * a.ldx, xc, d, lane);
        if (lane == 0 && acc < pts[p]) pts[p] = acc;
      }
    } else {
      for (int p = group; p < here; p += kDrawThreads / kExactLanes) {
        const double acc = row_square(rows + (size_t)p * d, xc, d, lane);
        if (lane == 0 && acc < pts[p]) pts[p] = acc;
      }
    }
    __syncthreads();
    if (tid == 0) ntodo = 0;
    if (wave < blocks_here) {  // a wave per block
      double tot = pts[tid];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) tot += __shfl_xor(tot, o, 64);
      if (wl == 0) block_sum[wave] = tot;
    }
    __syncthreads();
    if (tid < kRunCopies && m + 2 < a.k) {
      double sum = 0.0;
      for (int b = 0; b < blocks_here; ++b) sum += block_sum[b];
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the place that is free again is so before that
      put(a.ring + (m % 3 * kRunCopies + tid) * runs + blockIdx.x, sum);
    }
  }
  if (tid < here) a.dist2[i0 + tid] = pts[tid];
  if (tid < blocks_here) a.bsum[block0 + tid] = block_sum[tid];
  if (tid == 0) __hip_atomic_fetch_add(a.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- labelling, screened -------------------------------------------------------------------------------------------
// Most points are clearly nearer to one centre than to all others, and a product of bf16 numbers shows which: with the
// centred points and centres, scaled by a power of two (seed_mean_kernel's mean and scale), in two bf16 parts each,
// x = h + m + r,
//   v~(x, c) = h.h' + (h.m' + m.h') - |c|^2 / 2      ( |x - c|^2 = |x|^2 - 2 v )
// is formed on the bf16 matrix cores, and a point whose largest v~ exceeds the second largest by more than twice the bound
// E of the error of any of its v~ gets that centre's label: the fp64 labelling would give the same, E including what that
// itself is off by.  Between two centres alone fp64 distances decide (screen_store); the other points are listed and labelled
// by label_kernel.  With the norms ex, ec of what the parts leave
// out and the largest norms C of a centre and Cu of an uncentred one (all measured when the parts are made),
//   E = |x| ec + ex (C + ec) + 1.05 2^-18 |x| C    the parts, and m.m' (|m| <= 2^-9 |x|)
//     + 1.05 (D + 8) 2^-23 |x| C                   D products summed in single precision, and the subtraction
//     + C^2 2^-24                                  |c|^2 / 2 rounded
//     + (2 d + 16) 2^-53 ((|x| + |mean|) Cu + Cu^2)   the fp64 sums of the uncentred labelling.
// A NaN fails the comparison, and without a usable scale every point is listed.  Per step at 100,000 points,
// 100 coordinates and 100 centres 29 us with the fp64 distances of the points between two centres (a tenth of them) and 5 us
// for the rest, instead of 84 us all in fp64: 45 MB of the copy, the products (4 us) and the search (5 us) one after another.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));

struct CentreBound {  // of one tile of 32 centres
  float norm, err, uncentred, pad;
};

// The rows of x as the matrix instruction takes them: piece (t, s, part) = 64 lanes x 8 bf16, lane l = coordinates 16 s +
// 8 (l / 32) + 0 .. 7 of row 32 t + l % 32, part 0 = h, part 1 = m; rows past the end are zeros.  bound[i] = (|y|, |y - h - m|)
// rounded up, y the scaled row.  A wave per tile, or (CENTRES: few rows) a workgroup, which leaves half[i] = |y|^2 / 2 (3e38
// past the end), most[t] = the largest norms of the tile, and *undecided = 0.
template <bool CENTRES>
__global__ __launch_bounds__(CENTRES ? 512 : kT) void label_copy_kernel(const double* __restrict__ x, int64_t ldx, int d,
                                                        int64_t n, int64_t tiles, int ks, const double* __restrict__ mean,
                                                        const double* __restrict__ scale, uint4* __restrict__ out,
                                                        float2* __restrict__ bound, float* __restrict__ half,
                                                        CentreBound* __restrict__ most, int* __restrict__ undecided) {
  constexpr int W = CENTRES ? 8 : 1;  // waves per tile
  __shared__ double parts[W][4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t t = CENTRES ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * (kT / 64) + wave;
  if (CENTRES && blockIdx.x == 0 && threadIdx.x == 0) *undecided = 0;
  if (t >= tiles) return;  // uniform over the workgroup where it meets below
  const int64_t i = 32 * t + (lane & 31);
  const double f = *scale;
  double moved = 0.0, size = 0.0, sum = 0.0, raw = 0.0;
  for (int s = CENTRES ? wave : 0; s < ks; s += W) {
    union { __bf16 b[8]; uint4 v; } h, m;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int c = 16 * s + 8 * (lane >> 5) + q;
      const double xv = i < n && c < d ? x[i * ldx + c] : 0.0, mv = i < n && c < d ? mean[c] : 0.0;
      const double v = xv * f, mu = mv * f, y = v - mu;
      h.b[q] = (__bf16)(float)y;
      const double rest = y - (double)(float)h.b[q];
      m.b[q] = (__bf16)(float)rest;
      const double off = rest - (double)(float)m.b[q];
      moved += off * off;
      size += v * v + mu * mu;
      sum += y * y;
      raw += v * v;
    }
    out[((t * ks + s) * 2) * 64 + lane] = h.v;
    out[((t * ks + s) * 2 + 1) * 64 + lane] = m.v;
  }
  if constexpr (CENTRES) {
    parts[wave][0][lane] = moved;
    parts[wave][1][lane] = size;
    parts[wave][2][lane] = sum;
    parts[wave][3][lane] = raw;
    __syncthreads();
    if (wave) return;
    for (int w = 1; w < W; ++w) {
      moved += parts[w][0][lane];
      size += parts[w][1][lane];
      sum += parts[w][2][lane];
      raw += parts[w][3][lane];
    }
  }
  moved += __shfl_xor(moved, 32, 64);
  size += __shfl_xor(size, 32, 64);
  sum += __shfl_xor(sum, 32, 64);
  float err = (float)((sqrt(moved) + 4.5e-16 * sqrt(size)) * 1.00001) + 1e-37f;
  float norm = (float)(sqrt(sum) * 1.00001) + 1e-37f;
  if constexpr (!CENTRES) {
    if (lane < 32 && i < n) bound[i] = make_float2(norm, err);
  } else {
    raw += __shfl_xor(raw, 32, 64);
    float unc = (float)(sqrt(raw) * 1.00001) + 1e-37f;
    if (lane < 32) half[i] = i < n ? (float)(0.5 * sum) : 3.0e38f;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) {  // a NaN stays
      const float on = __shfl_xor(norm, o, 64), oe = __shfl_xor(err, o, 64), ou = __shfl_xor(unc, o, 64);
      norm = on > norm || on != on ? on : norm;
      err = oe > err || oe != oe ? oe : err;
      unc = ou > unc || ou != ou ? ou : unc;
    }
    if (lane == 0) most[t] = CentreBound{norm, err, unc, 0.0f};
  }
}

// What a lane knows of one point: the best two of the centres it has seen, and the value of the third.
struct ScreenBest {
  float best, second, third;
  int at, at2;
  __device__ __forceinline__ void clear() {
    best = second = third = -INFINITY;
    at = at2 = 0;
  }
  __device__ __forceinline__ void take(float v, int j) {
    third = fmaxf(third, fminf(second, v));
    at2 = v > best ? at : v > second ? j : at2;
    second = fmaxf(second, fminf(best, v));
    at = v > best ? j : at;
    best = fmaxf(best, v);
  }
  // the products with the centres j0 + 8 r4 + r; their halved squared norms at chalf + j0
  __device__ __forceinline__ void look(const f16v& acc, const float* __restrict__ chalf, int j0) {
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const f4 h = *reinterpret_cast<const f4*>(chalf + j0 + 8 * r4);
#pragma unroll
      for (int r = 0; r < 4; ++r) take(acc[4 * r4 + r] - h[r], j0 + 8 * r4 + r);
    }
  }
  // what the lane's other half has seen of the same point
  __device__ __forceinline__ void meet() {
    const float ob = __shfl_xor(best, 32, 64), os = __shfl_xor(second, 32, 64), ot = __shfl_xor(third, 32, 64);
    const int oa = __shfl_xor(at, 32, 64), oa2 = __shfl_xor(at2, 32, 64);
    take(ob, oa);
    take(os, oa2);
    third = fmaxf(third, ot);
  }
};

// The largest norms of all centres (every lane alike); a NaN stays.
__device__ __forceinline__ CentreBound centre_bound(const CentreBound* __restrict__ most, int ctiles, int lane) {
  float n = 0.0f, e = 0.0f, u = 0.0f;
  for (int t = lane; t < ctiles; t += 64) {
    const CentreBound m = most[t];
    n = m.norm > n || m.norm != m.norm ? m.norm : n;
    e = m.err > e || m.err != m.err ? m.err : e;
    u = m.uncentred > u || m.uncentred != m.uncentred ? m.uncentred : u;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float on = __shfl_xor(n, o, 64), oe = __shfl_xor(e, o, 64), ou = __shfl_xor(u, o, 64);
    n = on > n || on != on ? on : n;
    e = oe > e || oe != oe ? oe : e;
    u = ou > u || ou != ou ? ou : u;
  }
  return CentreBound{n, e, u, 0.0f};
}

// |mean| in the screen's scale, rounded up (every lane alike)
__device__ __forceinline__ float scaled_norm(const double* __restrict__ mean, int d, double f, int lane) {
  double sum = 0.0;
  for (int c = lane; c < d; c += 64) sum += mean[c] * f * (mean[c] * f);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  return (float)(sqrt(sum) * 1.00001);
}

// The labels of tile t's points.  Where only two centres are within 2 E, their distances are formed in fp64, 16 lanes per
// point and four points at a time, and decide if they differ by more than they and the fp64 labelling can be off,
// (8 d + 64) 2^-53 ((|x| + |mean|) + Cu)^2; what is left is listed.
__device__ __forceinline__ void screen_store(ScreenBest mine, int64_t t, int64_t n, const double* __restrict__ x, int64_t ldx,
                                             const double* __restrict__ centres, const float2* __restrict__ bound,
                                             const CentreBound& c, float mnorm, int ks, int d, double f, int k, int lane,
                                             int32_t* __restrict__ label, int32_t* __restrict__ rows,
                                             int* __restrict__ changes, int slot) {
  mine.meet();
  const int64_t i = t * 32 + lane;
  const bool live = lane < 32 && i < n;
  bool clear = false, pair = false;
  float norm = 0.0f;
  const int before = live ? label[i] : 0;
  if (live && f > 0.0) {
    const float2 b = bound[i];
    norm = b.x + mnorm;
    const float e = b.x * c.err + b.y * (c.norm + c.err) +
                    b.x * c.norm * (1.05f * 3.8146973e-06f + 1.05f * (float)(16 * ks + 8) * 1.1920929e-07f) +
                    c.norm * c.norm * 5.9604645e-08f +
                    (float)(2 * d + 16) * 1.1102230e-16f * (norm * c.uncentred + c.uncentred * c.uncentred);
    clear = mine.best - mine.second > 2.0002f * e;
    pair = !clear && mine.best - mine.third > 2.0002f * e && mine.at < k && mine.at2 < k;
  }
  unsigned long long pairs = __ballot(pair);
  while (pairs) {  // uniform
    const int sub = lane >> 4;
    unsigned long long rest = pairs;
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (q < sub) rest &= rest - 1ull;
    const bool have = rest != 0ull;  // uniform over the 16 lanes
    const int from = have ? __ffsll((long long)rest) - 1 : 0;
    const int j1 = __shfl(mine.at, from, 64), j2 = __shfl(mine.at2, from, 64);
    const float pn = __shfl(norm, from, 64);
    double d1 = 0.0, d2 = 0.0;
    if (have) {
      const double* __restrict__ xi = x + (t * 32 + from) * ldx;
      const double *__restrict__ c1 = centres + (int64_t)j1 * ldx, *__restrict__ c2 = centres + (int64_t)j2 * ldx;
#pragma unroll 4
      for (int q = lane & 15; q < d; q += 16) {
        const double v = xi[q], a = v - c1[q], b = v - c2[q];
        d1 += a * a;
        d2 += b * b;
      }
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
      d1 += __shfl_xor(d1, o, 16);
      d2 += __shfl_xor(d2, o, 16);
    }
    const double off = (8.0 * d + 64.0) * 1.1102230246251565e-16 * (double)(pn + c.uncentred) * (double)(pn + c.uncentred);
    const bool first = (d2 - d1) * f * f > off, other = (d1 - d2) * f * f > off;
    // to the point's own lane
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (!pairs) break;  // uniform
      const int to = __ffsll((long long)pairs) - 1;
      pairs &= pairs - 1ull;
      const int qf = __shfl((int)first, 16 * q, 64), qo = __shfl((int)other, 16 * q, 64);
      if (lane == to) {
        clear = qf || qo;
        if (qo) mine.at = mine.at2;
      }
    }
  }
  const bool differs = clear && before != mine.at;
  if (differs) label[i] = mine.at;
  const unsigned long long open = __ballot(live && !clear);
  const int moved = __popcll(__ballot(differs));
  int place = 0;
  if (lane == 0) {
    if (moved) atomicAdd(&changes[slot % kChangeSlots * kChangeStride], moved);
    if (open) place = atomicAdd(&changes[kChangeUndecided], __popcll(open));
  }
  place = __builtin_amdgcn_readfirstlane(place);
  if (live && !clear) rows[place + __popcll(open & ((1ull << lane) - 1ull))] = (int32_t)i;
}

#define MFMA_BF16(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)

// Up to 128 coordinates.  A wave keeps a tile of points in registers (B operands) and requests the next one while it goes
// through the centres (A operands, two tiles at a time), which the workgroup holds in LDS: all of them where they fit
// `chunk` tiles, else chunk by chunk.  A lane gets 16 centres of one point from every product.  Two waves per SIMD: eight
// waves a workgroup and four per SIMD, without the request ahead, spill and took 43 instead of 29 us (100,000 points, 100
// coordinates, 100 centres).
template <int KS>
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(2))) void label_screen_kernel(
    const double* __restrict__ x, int64_t ldx,
    const double* __restrict__ centres, int k, const bf16x8* __restrict__ xb, const float2* __restrict__ bound, int64_t n, int64_t tiles, int d,
    const bf16x8* __restrict__ cb, const float* __restrict__ chalf, const CentreBound* __restrict__ most, int ctiles,
    int chunk, const double* __restrict__ mean, const double* __restrict__ scale, int32_t* __restrict__ label,
    int32_t* __restrict__ rows, int* __restrict__ changes) {
  extern __shared__ __align__(16) unsigned char smem[];
  bf16x8* stage = reinterpret_cast<bf16x8*>(smem);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double f = *scale;
  const float mnorm = scaled_norm(mean, d, f, lane);
  const CentreBound cbound = centre_bound(most, ctiles, lane);
  const int64_t stride = (int64_t)gridDim.x * (kT / 64);
  bf16x8 bh[KS], bm[KS], nh[KS], nm[KS];
  auto request = [&](int64_t t) __attribute__((always_inline)) {
    t = t < tiles ? t : tiles - 1;  // past the end: computed, never stored
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      nh[s] = xb[((t * KS + s) * 2) * 64 + lane];
      nm[s] = xb[((t * KS + s) * 2 + 1) * 64 + lane];
    }
  };
  int64_t t = (int64_t)blockIdx.x * (kT / 64) + wave;
  request(t);
  bool staged = false;
  for (int64_t g = (int64_t)blockIdx.x * (kT / 64); g < tiles; g += stride, t += stride) {  // uniform over the workgroup
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      bh[s] = nh[s];
      bm[s] = nm[s];
    }
    if (g + stride < tiles) request(t + stride);
    ScreenBest mine;
    mine.clear();
    for (int c0 = 0; c0 < ctiles; c0 += chunk) {
      const int nc = ctiles - c0 < chunk ? ctiles - c0 : chunk;  // even
      if (!staged || ctiles > chunk) {  // uniform
        if (staged) __syncthreads();    // the chunk before has been read
        for (int e = threadIdx.x; e < nc * KS * 128; e += kT) stage[e] = cb[(int64_t)c0 * KS * 128 + e];
        __syncthreads();
        staged = true;
      }
      for (int c = 0; c < nc; c += 2) {
        f16v acc[2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[a][r] = 0.0f;
#pragma unroll
        for (int s = 0; s < KS; ++s)  // the small cross terms first
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            const bf16x8 ah = stage[(((c + a) * KS + s) * 2) * 64 + lane], am = stage[(((c + a) * KS + s) * 2 + 1) * 64 + lane];
            acc[a] = MFMA_BF16(am, bh[s], acc[a]);
            acc[a] = MFMA_BF16(ah, bm[s], acc[a]);
          }
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            const bf16x8 ah = stage[(((c + a) * KS + s) * 2) * 64 + lane];
            acc[a] = MFMA_BF16(ah, bh[s], acc[a]);
          }
#pragma unroll
        for (int a = 0; a < 2; ++a) mine.look(acc[a], chalf, 32 * (c0 + c + a) + 4 * (lane >> 5));
      }
    }
    if (t < tiles)
      screen_store(mine, t, n, x, ldx, centres, bound, cbound, mnorm, KS, d, f, k, lane, label, rows, changes,
                   (int)blockIdx.x * (kT / 64) + wave);
  }
}

// More coordinates: a wave takes two tiles of points against two tiles of centres at a time, all pieces from the L2.
__global__ __launch_bounds__(kT) void label_screen_wide_kernel(
    const double* __restrict__ x, int64_t ldx,
    const double* __restrict__ centres, int k, const bf16x8* __restrict__ xb, const float2* __restrict__ bound, int64_t n, int64_t tiles, int ks, int d,
    const bf16x8* __restrict__ cb, const float* __restrict__ chalf, const CentreBound* __restrict__ most, int ctiles,
    const double* __restrict__ mean, const double* __restrict__ scale, int32_t* __restrict__ label,
    int32_t* __restrict__ rows, int* __restrict__ changes) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t t0 = ((int64_t)blockIdx.x * (kT / 64) + wave) * 2;
  if (t0 >= tiles) return;
  const int64_t t1 = t0 + 1 < tiles ? t0 + 1 : t0;
  const double f = *scale;
  const float mnorm = scaled_norm(mean, d, f, lane);
  const CentreBound cbound = centre_bound(most, ctiles, lane);
  ScreenBest mine[2];
  mine[0].clear();
  mine[1].clear();
  for (int c0 = 0; c0 < ctiles; c0 += 2) {
    f16v low[2][2], acc[2][2];  // [centre tile][point tile]: the cross terms apart, they are added last
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) low[a][q][r] = acc[a][q][r] = 0.0f;
    for (int s = 0; s < ks; ++s) {
      bf16x8 xh[2], xm[2], ch[2], cm[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int64_t t = q ? t1 : t0;
        xh[q] = xb[((t * ks + s) * 2) * 64 + lane];
        xm[q] = xb[((t * ks + s) * 2 + 1) * 64 + lane];
        ch[q] = cb[(((int64_t)(c0 + q) * ks + s) * 2) * 64 + lane];
        cm[q] = cb[(((int64_t)(c0 + q) * ks + s) * 2 + 1) * 64 + lane];
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          low[a][q] = MFMA_BF16(cm[a], xh[q], low[a][q]);
          low[a][q] = MFMA_BF16(ch[a], xm[q], low[a][q]);
          acc[a][q] = MFMA_BF16(ch[a], xh[q], acc[a][q]);
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][q][r] += low[a][q][r];
        mine[q].look(acc[a][q], chalf, 32 * (c0 + a) + 4 * (lane >> 5));
      }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (t0 + q < tiles)
      screen_store(mine[q], t0 + q, n, x, ldx, centres, bound, cbound, mnorm, ks, d, f, k, lane, label, rows, changes,
                   (int)blockIdx.x * (kT / 64) + wave);
}

// c[j, :] = x[index[j], :]
__global__ __launch_bounds__(kT) void gather_rows_kernel(const double* __restrict__ x, int64_t ldx,
                                                         const int32_t* __restrict__ index, int k,
                                                         double* __restrict__ c) {
  const int64_t idx = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (idx >= (int64_t)k * ldx) return;
  const int64_t j = idx / ldx;
  c[idx] = x[(int64_t)index[j] * ldx + (idx - j * ldx)];
}

// part[block] = sum over the block's points of |x_i - c_label(i)|^2; fixed assignment of points to threads and a
// fixed tree, so the partial sums are reproducible.  Grid-stride over points, one thread per point and trip.  A label
// outside [0, k), which a point without a finite distance has, names no row of c: that point's distance is NaN.
__global__ __launch_bounds__(kT) void objective_kernel(const double* __restrict__ x, int64_t ldx, int d, int64_t n,
                                                       const int32_t* __restrict__ label, int k,
                                                       const double* __restrict__ c, double* __restrict__ part) {
  __shared__ double red[kT];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
    const double* xi = x + i * ldx;
    const int32_t lab = label[i];
    if ((uint32_t)lab >= (uint32_t)k) {
      acc = __longlong_as_double(0x7ff8000000000000ll);
      continue;
    }
    const double* cj = c + (int64_t)lab * ldx;
    double s2 = 0.0;
    for (int t = 0; t < d; ++t) {
      const double diff = xi[t] - cj[t];
      s2 += diff * diff;
    }
    acc += s2;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = kT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// out[i * ldo + t] = c[j * ldx + t] for the caller's row-major k x d centre array
__global__ __launch_bounds__(kT) void copy_rows_kernel(const double* __restrict__ src, int64_t lds_, double* __restrict__ dst,
                                                       int64_t ldd, int rows, int cols) {
  const int64_t idx = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (idx >= (int64_t)rows * cols) return;
  const int64_t r = idx / cols;
  const int t = (int)(idx - r * cols);
  dst[r * ldd + t] = src[r * lds_ + t];
}

int bits_for(int64_t n) {
  int b = 1;
  while (b < 31 && ((int64_t)1 << b) < n) ++b;
  return b;
}

}  // namespace

hipError_t launch_points_to_rowmajor(const double* v, int64_t ldv, int colmajor, int64_t n, int d, double* x, int64_t ldx,
                                     hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(points_to_rowmajor_kernel, dim3((unsigned)((n + 63) / 64), (unsigned)((ldx + 63) / 64)), dim3(kT), 0,
                     st, v, ldv, colmajor, n, d, x, ldx);
  return hipGetLastError();
}

hipError_t launch_centroid_operand(const double* c, int64_t ldx, int k, int d, int dpad, double* ct, int64_t ldc,
                                   double* cnorm, int* changes, hipStream_t st) {
  hipLaunchKernelGGL(centroid_operand_kernel, dim3((unsigned)k), dim3(kT), 0, st, c, ldx, d, dpad, ct, ldc, cnorm, changes);
  return hipGetLastError();
}

hipError_t launch_fill_int32(int32_t* a, int64_t n, int32_t value, int use_iota, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(iota_fill_kernel, dim3(blocks(n)), dim3(kT), 0, st, a, n, value, use_iota);
  return hipGetLastError();
}

namespace {

// pieces per cluster: about 2,048 workgroups in all (eight per compute unit), at least 32 points each on average
int update_parts(int64_t n, int64_t ldx, int k) {
  const int64_t tiles = (ldx + 127) / 128;
  int64_t parts = 2048 / ((int64_t)k * tiles);
  const int64_t most = n / ((int64_t)k * 32) + 1;
  parts = parts < most ? parts : most;
  return (int)(parts < 1 ? 1 : parts);
}

size_t label_sort_bytes(int64_t n) {
  size_t bytes = 0;
  (void)rocprim::radix_sort_pairs(nullptr, bytes, (const int32_t*)nullptr, (int32_t*)nullptr, (const int32_t*)nullptr,
                                  (int32_t*)nullptr, (size_t)n, 0u, 32u, (hipStream_t) nullptr);
  return (bytes + 255) / 256 * 256;
}

}  // namespace

size_t kmeans_update_workspace(int64_t n, int64_t ldx, int k) {
  const size_t sums = ((size_t)k * update_parts(n, ldx, k) * (size_t)ldx * 8 + 255) / 256 * 256;
  const size_t nb = (size_t)((n + kSortBlock - 1) / kSortBlock);
  // sums | member[n] | counts[k][nb], total[k]   or   sums | member[n] | sorted_label[n], ident[n], temp
  const size_t group = k <= kMaxBins ? ((size_t)k * nb + (size_t)k) * 4 : (size_t)n * 8 + label_sort_bytes(n);
  return sums + ((size_t)n * 4 + 255) / 256 * 256 + group + 1024;
}

hipError_t launch_centroid_update(const double* x, int64_t ldx, int d, int64_t n, const int32_t* label, int k, void* work,
                                  size_t work_bytes, int32_t* start, double* c, double* ct, int64_t ldc, double* cnorm,
                                  int* changes, const LabelReport& report, int which, hipStream_t st) {
  if (n <= 0 || n > INT32_MAX || work_bytes < kmeans_update_workspace(n, ldx, k)) return hipErrorInvalidValue;
  const int parts = update_parts(n, ldx, k);
  char* base = static_cast<char*>(work);
  double* sums = reinterpret_cast<double*>(base);
  base += ((size_t)k * parts * (size_t)ldx * 8 + 255) / 256 * 256;
  int32_t* member = reinterpret_cast<int32_t*>(base);
  base += ((size_t)n * 4 + 255) / 256 * 256;
  if (k <= kMaxBins) {
    const int nb = (int)((n + kSortBlock - 1) / kSortBlock);
    int32_t* count = reinterpret_cast<int32_t*>(base);
    int32_t* total = count + (size_t)k * nb;
    if (which & kUpdateReport)
      hipLaunchKernelGGL(label_count_kernel, dim3((unsigned)nb), dim3(kT), 0, st, label, n, k, nb, count, changes, report);
    if (!(which & kUpdateCentres)) return hipGetLastError();
    hipLaunchKernelGGL(label_offset_kernel, dim3((unsigned)((k + 3) / 4)), dim3(kT), 0, st, count, k, nb, total, changes + kChangeSum);
    hipLaunchKernelGGL(label_scatter_kernel, dim3((unsigned)nb), dim3(kT), 0, st, label, n, k, bits_for(k), nb, count, total,
                       start, member, changes + kChangeSum);
  } else {
    int32_t* sorted_label = reinterpret_cast<int32_t*>(base);
    int32_t* ident = sorted_label + n;
    char* temp = reinterpret_cast<char*>(((uintptr_t)(ident + n) + 255) / 256 * 256);
    size_t sb = label_sort_bytes(n);
    if (which & kUpdateReport) hipLaunchKernelGGL(label_report_kernel, dim3(1), dim3(64), 0, st, changes, report);
    if (!(which & kUpdateCentres)) return hipGetLastError();
    hipLaunchKernelGGL(iota_fill_kernel, dim3(blocks(n)), dim3(kT), 0, st, ident, n, 0, 1);
    // one value more than there are clusters: a label outside [0, k), all ones in these bits, comes after them all
    const hipError_t e = rocprim::radix_sort_pairs(temp, sb, label, sorted_label, ident, member, (size_t)n, 0u,
                                                   (unsigned)bits_for((int64_t)k + 1), st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(cluster_starts_kernel, dim3(blocks(k + 1)), dim3(kT), 0, st, sorted_label, n, k, start);
  }
#define SC_SUM(DLV)                                                                                                     \
  hipLaunchKernelGGL((cluster_sum_kernel<DLV>), dim3((unsigned)k, (unsigned)parts, (unsigned)((ldx + 2 * DLV - 1) / (2 * DLV))), \
                     dim3(kT), 0, st, x, ldx, member, start, parts, sums, changes + kChangeSum)
  if (ldx <= 4) SC_SUM(2);
  else if (ldx <= 8) SC_SUM(4);
  else if (ldx <= 16) SC_SUM(8);
  else if (ldx <= 32) SC_SUM(16);
  else if (ldx <= 64) SC_SUM(32);
  else SC_SUM(64);
#undef SC_SUM
  hipLaunchKernelGGL(centroid_finish_kernel, dim3((unsigned)k), dim3(kT), 0, st, sums, parts, start, d, ldx, c, ct, ldc, cnorm,
                     changes);
  return hipGetLastError();
}

namespace {

// The bf16 copy costs three launches (70 us at 100,000 points of 100 coordinates) and pays once the points no longer fit
// the L2s and there are draws to spread that over: 100,000 x 100, 100 draws 2.04 -> 1.64 ms, 142,541 x 500, 500 draws
// 60 -> 27 ms; 140,000 x 8, 100 draws 1.47 -> 1.44 ms, 50,000 x 64, 16 draws 0.19 -> 0.23 ms.
bool seed_screened(int64_t n, int d, int k) { return n * (int64_t)d >= 4000000 && k >= 32; }
// Draws in one launch: as many blocks as seed_distance_kernel draws from; with the screen always (100,000 x 100, 100 draws 1,350 ->
// 1,110 us, 110,000 x 128, 128 draws 1,790 -> 1,380, 90,000 x 112, 33 draws 511 -> 479), else where workgroups, and with them the
// exchange, are few, and draws make up for the launch's own costs (2,000 x 128, 40 draws 359 -> 260, 2,000 x 2, 16 draws 134 -> 123,
// 10,000 x 2, 20 draws 171 -> 166; 20,000 x 64, 16 draws 165 -> 170, 40,900 x 30, 24 draws 230 -> 246).
bool seed_fused(int64_t nb, int k, bool screened) { return nb <= kDrawBlocks && (screened || (nb <= 256 && k >= 16)); }
inline int seed_dpb(int d) { return (d + 7) / 8 * 8; }

}  // namespace

size_t kmeans_seed_workspace(int64_t n, int64_t ldx, int d, int k, int screen) {
  // two of (dist2[n] | bsum[ceil(n / 64)])  and, with the screen,
  // sums[kSeedParts][ldx] | tops[kSeedParts] | err[n] | xh[n][dpb]
  const size_t nb = (size_t)((n + kSeedPoints - 1) / kSeedPoints);
  size_t bytes = 2 * ((size_t)n + nb) * 8 + 1024;
  if (seed_fused((int64_t)nb, k, screen && seed_screened(n, d, k))) bytes += kDrawShared;
  if (screen && seed_screened(n, d, k)) bytes += (size_t)(ldx + 1) * 8 * (kSeedParts + 1) + (size_t)n * (8 + 2 * (size_t)seed_dpb(d)) + 1024;
  return bytes;
}

// Algorithm 5 with the uniform numbers seed_uniform(key, 0 .. k-1).  chosen: device int32[k], the indices of the chosen points
// in the order they were drawn.  One or two launches per draw, or (f.groups > 0, the number of its workgroups) one for all but the
// last; whether that has come to run *f.done says once the stream is idle: f.groups, else 0, and the call has to be made again
// without (f.polls = kNeverFused).
hipError_t launch_kmeanspp(const double* x, int64_t ldx, int d, int64_t n, int k, uint64_t key, int screen, void* work,
                           size_t work_bytes, int32_t* chosen, double* centring, bool* centred, SeedFused& f, hipStream_t st) {
  f.groups = 0;
  if (n <= 0 || n > INT32_MAX || k < 1) return hipErrorInvalidValue;
  const int64_t nb = (n + kSeedPoints - 1) / kSeedPoints;
  if (work_bytes < kmeans_seed_workspace(n, ldx, d, k, screen)) return hipErrorInvalidValue;
  double* dist2[2] = {static_cast<double*>(work), static_cast<double*>(work) + n + nb};
  double *mean = centring, *scale = centring + ldx;
  double* sums = dist2[1] + n + nb;
  uint32_t* tops = reinterpret_cast<uint32_t*>(sums + (size_t)kSeedParts * ldx);
  float2* err = reinterpret_cast<float2*>(tops + kSeedParts);
  __bf16* xh = reinterpret_cast<__bf16*>(((uintptr_t)(err + n) + 15) / 16 * 16);
  const int dpb = seed_dpb(d);
  const bool screened = screen && seed_screened(n, d, k), draws = nb <= kDrawBlocks;
  *centred = screened;
  int64_t first = (int64_t)(seed_uniform(key, 0) * (double)n);
  first = first < n - 1 ? first : n - 1;
  const int per = (int)((nb + kDrawGroups - 1) / kDrawGroups);
  const size_t lds = seed_draws_lds(per, d, dpb, screened);
  const bool fused = f.polls != kNeverFused && seed_fused(nb, k, screened) && lds + 4096 <= f.lds_limit;  // beside what the draw takes
  double* const ring = fused ? reinterpret_cast<double*>(static_cast<char*>(work) + (work_bytes - kDrawShared) / 16 * 16) : nullptr;
  uint32_t* const words = fused ? reinterpret_cast<uint32_t*>(ring + kDrawPlaces) : nullptr;
  hipLaunchKernelGGL(seed_start_kernel, dim3(fused ? 8 : 1), dim3(kT), 0, st, chosen, (int32_t)first, fused ? k : 1,
                     reinterpret_cast<long long*>(ring), fused ? kDrawPlaces : 0, words, f.polls < 0 ? kStopped : 0u);
  if (screened) {
    hipLaunchKernelGGL(seed_sum_kernel, dim3(kSeedParts), dim3(kT), 0, st, x, ldx, n, sums, tops);
    hipLaunchKernelGGL(seed_mean_kernel, dim3(blocks(ldx)), dim3(kT), 0, st, sums, tops, kSeedParts, ldx, n, mean,
                       scale);
    hipLaunchKernelGGL(seed_copy_kernel, dim3(blocks(n * 8)), dim3(kT), 0, st, x, ldx, d, n, mean, scale, dpb, xh,
                       err);
  }
  int at = 0;  // the buffer with the distances to the centres so far
  auto pass = [&](int i) {  // the distances to centre i - 1
    const bool draw = draws && i > 1;
    const double *din = dist2[at], *bin = dist2[at] + n;
    if (i > 1) at ^= 1;
#define SC_SEED(SCR, DRW, SUBV, AHD)                                                                                     \
  hipLaunchKernelGGL((seed_distance_kernel<SCR, DRW, SUBV, AHD>), dim3((unsigned)((nb + SUBV - 1) / SUBV)), dim3(kT), 0, \
                     st, x, ldx, d, n, xh, dpb, err, seed_uniform(key, (uint64_t)i - 1), chosen + (i - 1), i == 1 ? 1 : 0, bin, nb, din, dist2[at], \
                     dist2[at] + n)
    if (screened && i > 1) {
      const bool wide = dpb <= kSeedWideDim && nb >= kSeedWide;
      if (draw && wide) SC_SEED(true, true, 2, true);
      else if (draw) SC_SEED(true, true, 1, false);
      else if (wide) SC_SEED(true, false, 2, true);
      else SC_SEED(true, false, 1, false);
    } else {
      if (draw) SC_SEED(false, true, 1, false); else SC_SEED(false, false, 1, false);
    }
#undef SC_SEED
  };
  if (fused) {
    pass(1);
    const void* kernel = screened ? reinterpret_cast<const void*>(seed_draws_kernel<true>) : reinterpret_cast<const void*>(seed_draws_kernel<false>);
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    f.done = reinterpret_cast<int*>(words + 32);
    f.groups = (int)((nb + per - 1) / per);
    SeedDraws a{x, ldx, n, nb, d, dpb, k, per, xh, err, key, dist2[0], dist2[0] + n, ring,
                reinterpret_cast<uint64_t*>(ring + 3 * kRunCopies * kDrawGroups), chosen, words, f.done, f.polls};
    if (screened)
      hipLaunchKernelGGL(seed_draws_kernel<true>, dim3((unsigned)f.groups), dim3(kDrawThreads), lds, st, a);
    else
      hipLaunchKernelGGL(seed_draws_kernel<false>, dim3((unsigned)f.groups), dim3(kDrawThreads), lds, st, a);
    hipLaunchKernelGGL(seed_select_kernel, dim3(1), dim3(kSelectThreads), 0, st, dist2[0] + n, nb, dist2[0], n,
                       seed_uniform(key, (uint64_t)k - 1), chosen + k - 1);
    return hipGetLastError();
  }
  for (int i = 1; i < k; ++i) {
    pass(i);
    if (!draws || i == k - 1)
      hipLaunchKernelGGL(seed_select_kernel, dim3(1), dim3(kSelectThreads), 0, st, dist2[at] + n, nb, dist2[at], n,
                         seed_uniform(key, (uint64_t)i), chosen + i);
  }
  return hipGetLastError();
}

namespace {

// Below, the fp64 product takes no more than the two launches of the screened form (4e8: 33 us).
bool label_screened(int64_t n, int64_t ldx, int k) { return (double)n * (double)ldx * (double)k >= 4.0e8; }

struct LabelScreen {
  int ks = 0, ctiles = 0;
  int64_t tiles = 0;
  size_t off_cb = 0, off_bound = 0, off_half = 0, off_most = 0, off_sums = 0, off_tops = 0, off_rows = 0, bytes = 0;
};

LabelScreen plan_label_screen(int64_t n, int64_t ldx, int k) {
  LabelScreen p;
  p.ks = (int)((ldx + 15) / 16);
  p.tiles = (n + 31) / 32;
  p.ctiles = (k + 63) / 64 * 2;
  size_t off = (size_t)p.tiles * p.ks * 2048;
  auto place = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) / 256 * 256;
    return at;
  };
  p.off_cb = place((size_t)p.ctiles * p.ks * 2048);
  p.off_bound = place((size_t)n * sizeof(float2));
  p.off_half = place((size_t)p.ctiles * 32 * 4);
  p.off_most = place((size_t)p.ctiles * sizeof(CentreBound));
  p.off_sums = place((size_t)kSeedParts * ldx * 8);
  p.off_tops = place((size_t)kSeedParts * 4);
  p.off_rows = place((size_t)n * 4);
  p.bytes = off;
  return p;
}

}  // namespace

// The reduced copy of the points costs about as much as a fp64 labelling, and a screened step saves a tenth to a half of one,
// so the number of steps decides.  Fitted to 290 shapes (2,500 to 2,000,000 points of 2 to 2,000 normal coordinates, 16 to
// 2,000 centres; us a step by the fp64 product, saved by the screen, and the copy): 100,000 x 100, 100 centres 115 / 30 / 90,
// 500,000 x 100, 128 480 / 257 / 453, 1,000,000 x 8, 64 169 / 31 / 216, 65,000 x 64, 1,000 236 / 105 / 60, 200,000 x 500, 64
// 541 / 163 / 747.  Never where a wave's chain over few tiles of points is what a step lasts (20,000 x 2,000, 64 centres 394 /
// -116 / 397, 5,000 x 100, 1,000 60 / -30 / 63, 45,000 x 16, 1,000 88 / -4 / 38) or where there is next to nothing to
// multiply (200,000 x 2, 1,000 238 / -28 / 78).  In the mean over the shapes 10 steps take 14 % less than by the product alone
// (4 % with the screen always), 3 steps 6 % less (14 % more).
int label_screen_steps(int64_t n, int64_t ldx, int k) {
  const double w = (double)n * (double)ldx * (double)k, m = (double)n;
  const double copy = 7.5e-6 * m * (double)((ldx + 15) / 16 * 16) + 1.3e-4 * m + 10.0;
  double gain = 0.0;
  if (ldx <= 128) {
    const bool few = ldx >= 64 ? (n >= 45000 && k >= 128) || (n >= 30000 && k >= 256) || (n >= 20000 && k >= 1000 && ldx >= 100)
                               : ldx >= 32 && n >= 45000 && k >= 1000;
    if ((ldx < 8 && n < 500000) || (n < 65000 && !few)) return INT32_MAX;
    gain = 3.5e-8 * w * (ldx <= 16 ? 0.25 : 1.0) * std::min(1.0, ((double)ldx + 24.0) / 88.0) * (n < 65000 ? 0.5 : 1.0) - 2.0 +
           4e-5 * std::max(0.0, m - 200000.0);
  } else {
    const bool few = (n >= 45000 && k >= 128) || (n >= 30000 && k >= 500 && ldx <= 512) || (n >= 20000 && k >= 1000 && ldx <= 320);
    if (n < 65000 && !few) return INT32_MAX;
    const double fill = std::min(1.0, m / 1e5);
    gain = 2.3e-8 * w * (ldx <= 320 ? fill : k >= 256 ? fill * std::sqrt(fill) : fill * fill) - 4.0;
  }
  if (gain < 4.0) return INT32_MAX;
  return std::max(3, (int)std::ceil(std::min(1.2 * copy / gain, 1e9)));
}

size_t label_screen_workspace(int64_t n, int64_t ldx, int k) {
  return label_screened(n, ldx, k) ? plan_label_screen(n, ldx, k).bytes : 0;
}

hipError_t launch_label_copy(const double* x, int64_t ldx, int d, int64_t n, int k, void* work, double* centring, bool centred,
                             hipStream_t st) {
  const LabelScreen p = plan_label_screen(n, ldx, k);
  char* w = static_cast<char*>(work);
  double *mean = centring, *scale = centring + ldx;
  double* sums = reinterpret_cast<double*>(w + p.off_sums);
  uint32_t* tops = reinterpret_cast<uint32_t*>(w + p.off_tops);
  if (!centred) {
    hipLaunchKernelGGL(seed_sum_kernel, dim3(kSeedParts), dim3(kT), 0, st, x, ldx, n, sums, tops);
    hipLaunchKernelGGL(seed_mean_kernel, dim3(blocks(ldx)), dim3(kT), 0, st, sums, tops, kSeedParts, ldx, n, mean, scale);
  }
  hipLaunchKernelGGL(label_copy_kernel<false>, dim3((unsigned)((p.tiles + kT / 64 - 1) / (kT / 64))), dim3(kT), 0, st, x, ldx,
                     d, n, p.tiles, p.ks, mean, scale, reinterpret_cast<uint4*>(w),
                     reinterpret_cast<float2*>(w + p.off_bound), nullptr, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_label_screened(const double* x, int64_t ldx, int d, int64_t n, const double* c, const double* ct,
                                 int64_t ldc, int k, const double* cnorm, void* work, const double* centring, int32_t* label, int* changes,
                                 hipStream_t st) {
  const LabelScreen p = plan_label_screen(n, ldx, k);
  char* w = static_cast<char*>(work);
  const double *mean = centring, *scale = centring + ldx;
  float* half = reinterpret_cast<float*>(w + p.off_half);
  CentreBound* most = reinterpret_cast<CentreBound*>(w + p.off_most);
  int32_t* rows = reinterpret_cast<int32_t*>(w + p.off_rows);
  const bf16x8* xb = reinterpret_cast<const bf16x8*>(w);
  const float2* bound = reinterpret_cast<const float2*>(w + p.off_bound);
  const bf16x8* cb = reinterpret_cast<const bf16x8*>(w + p.off_cb);
  hipLaunchKernelGGL(label_copy_kernel<true>, dim3((unsigned)p.ctiles), dim3(512), 0, st, c, ldx, d, (int64_t)k,
                     (int64_t)p.ctiles, p.ks, mean, scale, reinterpret_cast<uint4*>(w + p.off_cb), nullptr, half, most,
                     changes + kChangeUndecided);
  if (p.ks <= 8) {
    // 64 KB of centres: two workgroups per compute unit, which take equally many tiles of points each
    int chunk = 32 / p.ks / 2 * 2;
    chunk = chunk < p.ctiles ? chunk : p.ctiles;
    const int64_t groups = (p.tiles + kT / 64 - 1) / (kT / 64), rounds = (groups + 511) / 512;
    const unsigned grid = (unsigned)((groups + rounds - 1) / rounds);
#define SC_LABEL_SCREEN(KSV)                                                                                             \
  hipLaunchKernelGGL(label_screen_kernel<KSV>, dim3(grid), dim3(kT), (size_t)chunk * KSV * 2048, st, x, ldx, c, k, xb, bound, n, \
                     p.tiles, d, cb, half, most, p.ctiles, chunk, mean, scale, label, rows, changes)
    switch (p.ks) {
      case 1: SC_LABEL_SCREEN(1); break;
      case 2: SC_LABEL_SCREEN(2); break;
      case 3: SC_LABEL_SCREEN(3); break;
      case 4: SC_LABEL_SCREEN(4); break;
      case 5: SC_LABEL_SCREEN(5); break;
      case 6: SC_LABEL_SCREEN(6); break;
      case 7: SC_LABEL_SCREEN(7); break;
      default: SC_LABEL_SCREEN(8); break;
    }
#undef SC_LABEL_SCREEN
  } else {
    hipLaunchKernelGGL(label_screen_wide_kernel, dim3((unsigned)((p.tiles + 2 * (kT / 64) - 1) / (2 * (kT / 64)))), dim3(kT),
                       0, st, x, ldx, c, k, xb, bound, n, p.tiles, p.ks, d, cb, half, most, p.ctiles, mean, scale, label, rows, changes);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_label_listed(x, ldx, n, rows, changes + kChangeUndecided, ct, ldc, k, cnorm, label, changes, st);
}

hipError_t launch_gather_rows(const double* x, int64_t ldx, const int32_t* index, int k, double* c, hipStream_t st) {
  hipLaunchKernelGGL(gather_rows_kernel, dim3(blocks((int64_t)k * ldx)), dim3(kT), 0, st, x, ldx, index, k, c);
  return hipGetLastError();
}

int kmeans_objective_parts() { return 1024; }

hipError_t launch_objective(const double* x, int64_t ldx, int d, int64_t n, const int32_t* label, int k, const double* c,
                            double* part, hipStream_t st) {
  hipLaunchKernelGGL(objective_kernel, dim3((unsigned)kmeans_objective_parts()), dim3(kT), 0, st, x, ldx, d, n, label, k,
                     c, part);
  return hipGetLastError();
}

hipError_t launch_copy_rows(const double* src, int64_t lds, double* dst, int64_t ldd, int rows, int cols, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_rows_kernel, dim3(blocks((int64_t)rows * cols)), dim3(kT), 0, st, src, lds, dst, ldd, rows,
                     cols);
  return hipGetLastError();
}

}  // namespace sceig
