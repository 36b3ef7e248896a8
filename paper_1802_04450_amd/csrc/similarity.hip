// Similarity-graph construction (paper Section IV-A: the similarity measures and Algorithm 1; Algorithm 2 step 4, the
// COO to CSR conversion), device kernels.
//
// Algorithm 1 centres the data in place and gives one thread a row / an edge.  Here the data are read only: a first
// kernel stores the mean and the norm of every row (of the centred row for the cross correlation), and the edge
// kernel forms sum_t (x_it - m_i)(x_jt - m_j) directly, 4 or 16 lanes per edge with 16-byte loads.  Larger data are read bucket by
// bucket of rows, so that a row comes out of memory a few times instead of once per pair.  The conversion puts the entries into
// buckets of rows and sorts each in LDS; matrices that this does not suit go through rocPRIM's radix sort of (row, col) keys (a
// library primitive, the counterpart of the paper's library call) with row pointers by binary search.
#include <hip/hip_runtime.h>
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/device/device_select.hpp>
#include <rocprim/functional.hpp>
#include <rocprim/iterator/counting_iterator.hpp>

#include <cstdint>

#include "kernels.h"

namespace sceig {
namespace {

constexpr int kT = 256;
constexpr int kL = 16;  // lanes per row / per edge
inline unsigned blocks(int64_t n) { return (unsigned)((n + kT - 1) / kT); }

// v of another lane of the 16, by a DPP control word
template <int CTRL>
__device__ __forceinline__ double row_dpp(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// The sum over the 16 lanes of a DPP row, in the order of a butterfly over 8, 4, 2, 1: row_ror:8, row_ror:4 (the values
// repeat every 8 lanes by then), quad_perm [2,3,0,1], quad_perm [1,0,3,2].  All lanes of the row must be active.
__device__ __forceinline__ double group_sum(double v) {
  static_assert(kL == 16, "a DPP row");
  v += row_dpp<0x128>(v);
  v += row_dpp<0x124>(v);
  v += row_dpp<0x4e>(v);
  v += row_dpp<0xb1>(v);
  return v;
}

// ---- entries into buckets of rows ----------------------------------------------------------------------------------
// Bucket b takes the entries of the rows [b << shift, (b + 1) << shift) into slots b * room .. of `slots` (room <=
// kBucketRoom), in no particular order: a workgroup counts its entries per bucket in LDS, reserves that many
// slots of every bucket with one atomic addition and writes.  fill[b] ends up as the bucket's number of entries, more than
// `room` if they did not fit: what does not fit, and entries with an index out of range, go to the list `rest` (room for all of
// them, *nrest of them) or, where that is null, are dropped and the caller looks at the counts.
// A slot is (row within the bucket, column, payload), from the top, in 64 bits: in the order of these numbers the entries of a
// bucket are sorted.  Row and column take the upper half where they fit it (up to four million rows), else as much as they need:
// buckets have 2^25 entries at most, so that the payload fits the rest.
struct SlotBits {
  int col, pay;  // bits of a column, bits of a payload
};
constexpr int kBucketRoom = 4096;
constexpr int kMaxBuckets = 16384;
constexpr int kPartThreads = 1024;
// Entries per thread: 16, so that few additions reserve many slots, or 2 where 16 would leave the chip without workgroups
// (up to kPartFew entries; 200,000: 31 us with 16, 9 us with 2).
constexpr int kPartTrips = 16, kPartTripsFew = 2;
constexpr int64_t kPartFew = 256 * kPartThreads * kPartTripsFew;

// Neighbouring lanes of a wave with the same bucket count as one: a list in the order of its rows has 32 and more of them side by
// side, whose additions to one counter come one after the other (half of this kernel's time on 3.8 M voxel pairs).
struct LaneRun {
  int head, len;  // first lane of this lane's run, lanes of the run
};
__device__ __forceinline__ LaneRun lane_run(int b) {
  const int lane = threadIdx.x & 63;
  // wave_shr:1; lane 0 starts a run whatever it gets
  const int before = __builtin_amdgcn_update_dpp(0, b, 0x138, 0xf, 0xf, false);
  const uint64_t heads = __ballot(lane == 0 || before != b);
  const uint64_t upto = heads & (~0ull >> (63 - lane)), above = heads & ~(~0ull >> (63 - lane));
  LaneRun r;
  r.head = 63 - __clzll((long long)upto);
  r.len = (above ? __ffsll((unsigned long long)above) - 1 : 64) - r.head;
  return r;
}
// Adds one to count[b] for every lane with b >= 0 (all lanes of the wave call) and returns what the lane's addition found.
__device__ __forceinline__ int count_run(int32_t* count, int b) {
  const LaneRun r = lane_run(b);
  const int lane = threadIdx.x & 63;
  int at = 0;
  if (lane == r.head && b >= 0) at = atomicAdd(&count[b], r.len);
  return __shfl(at, r.head, 64) + (lane - r.head);
}

// The e-th entry is (row[e], col[e]) with payload e; with MIRROR the same again as (col[e], row[e]) with payload
// nnz_in + e unless the two are equal (rest is null then).  An index outside [0, n) sets *bad.
template <bool MIRROR, int TRIPS>
__global__ __launch_bounds__(kPartThreads) void partition_kernel(const int32_t* __restrict__ row,
                                                                 const int32_t* __restrict__ col, int64_t nnz_in, int64_t n,
                                                                 int shift, int nbuckets, int room,
                                                                 int32_t* __restrict__ fill, uint64_t* __restrict__ slots,
                                                                 SlotBits bits, uint32_t* __restrict__ rest, int32_t* __restrict__ nrest,
                                                                 int* __restrict__ bad) {
  __shared__ int32_t count[kMaxBuckets];
  __shared__ int32_t left, left0;
  constexpr int TR = MIRROR ? TRIPS / 2 : TRIPS;
  const int64_t e0 = (int64_t)blockIdx.x * (TR * kPartThreads);
  for (int b = threadIdx.x; b < nbuckets; b += kPartThreads) count[b] = 0;
  if (threadIdx.x == 0) left = 0;
  __syncthreads();
  int32_t r[TR], c[TR];
#pragma unroll
  for (int u = 0; u < TR; ++u) {
    const int64_t e = e0 + u * kPartThreads + threadIdx.x;
    r[u] = e < nnz_in ? row[e] : -1;
    c[u] = e < nnz_in ? col[e] : -1;
  }
  bool wrong = false;
#pragma unroll
  for (int u = 0; u < TR; ++u) {
    const int64_t e = e0 + u * kPartThreads + threadIdx.x;
    if (e < nnz_in && (r[u] < 0 || r[u] >= n || c[u] < 0 || c[u] >= n)) {
      wrong = true;
      r[u] = -1;
    }
    (void)count_run(count, r[u] < 0 ? -1 : r[u] >> shift);  // r = -1 past the end too
    if (MIRROR) (void)count_run(count, r[u] < 0 || r[u] == c[u] ? -1 : c[u] >> shift);
  }
  if (wrong) atomicOr(bad, 1);
  __syncthreads();
  for (int b = threadIdx.x; b < nbuckets; b += kPartThreads) {
    const int mine = count[b];
    if (mine) count[b] = atomicAdd(&fill[b], mine);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < TR; ++u) {
    const int64_t e = e0 + u * kPartThreads + threadIdx.x;
    const int slot = count_run(count, r[u] < 0 ? -1 : r[u] >> shift), at = r[u] < 0 ? room : slot;
    if (e >= nnz_in) {
      // nothing
    } else if (at < room) {
      slots[(int64_t)(r[u] >> shift) * room + at] =
          ((uint64_t)(r[u] & ((1 << shift) - 1)) << bits.col | (uint32_t)c[u]) << bits.pay | (uint64_t)e;
    } else if (rest) {
      c[u] = -2 - atomicAdd(&left, 1);  // its place among the workgroup's
    }
    if (MIRROR) {
      const bool there = r[u] >= 0 && r[u] != c[u];
      const int am = count_run(count, there ? c[u] >> shift : -1);
      if (there && am < room) {
        slots[(int64_t)(c[u] >> shift) * room + am] =
            ((uint64_t)(c[u] & ((1 << shift) - 1)) << bits.col | (uint32_t)r[u]) << bits.pay | (uint64_t)(nnz_in + e);
      }
    }
  }
  if (!rest) return;  // uniform
  // one addition to *nrest per workgroup (one per wave, 60,000 of them, took 600 us)
  __syncthreads();
  if (left == 0) return;  // uniform
  if (threadIdx.x == 0) left0 = atomicAdd(nrest, left);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < TR; ++u) {
    const int64_t e = e0 + u * kPartThreads + threadIdx.x;
    if (e < nnz_in && c[u] <= -2) rest[left0 + (-2 - c[u])] = (uint32_t)e;
  }
}

// base[b] = exclusive prefix sums of fill, *over |= 1 if a bucket overflowed.  One workgroup.
__global__ __launch_bounds__(kPartThreads) void bucket_scan_kernel(const int32_t* __restrict__ fill, int nbuckets,
                                                                   int room, int32_t* __restrict__ base, int* __restrict__ over) {
  __shared__ int32_t wave_sum[kPartThreads / 64];
  constexpr int PER = kMaxBuckets / kPartThreads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t v[PER], sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = (int)threadIdx.x * PER + q;
    v[q] = b < nbuckets ? fill[b] : 0;
    if (v[q] > room) atomicOr(over, 1);
    sum += v[q];
  }
  int32_t incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  int32_t at = incl - sum;
  for (int w = 0; w < wave; ++w) at += wave_sum[w];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = (int)threadIdx.x * PER + q;
    if (b < nbuckets) base[b] = at;
    at += v[q];
  }
}

// Threads of the workgroup that sorts a bucket: three workgroups' LDS fit a compute unit, with 256 threads each the waves
// were too few for the counting and the gather (7.6 M entries of 142,541 rows, the whole conversion 201 -> 175 us then).
constexpr int kST = 512;
// key[lo .. lo + len - 1] into ascending order by the whole workgroup: a bitonic network whose comparators all point
// upwards, so that those with a partner past the end can be left out.  The entries are there for every wave on entry, and
// again on return.
__device__ __forceinline__ void sort_run(uint64_t* key, int lo, int len) {
  for (int k = 2; k < 2 * len; k *= 2) {
    for (int j = k / 2; j > 0; j /= 2) {
      const int flip = j == k / 2 ? k - 1 : j;  // the first stage of a merge pairs an entry with its mirror image
      for (int q0 = threadIdx.x; 2 * (q0 & ~(j - 1)) < len; q0 += 4 * kST) {  // pair q: entries with bit j clear and set
        uint64_t a[4], b[4];
        int t[4], o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = q0 + u * kST;
          t[u] = 2 * (q & ~(j - 1)) | (q & (j - 1));
          o[u] = t[u] ^ flip;
          if (o[u] >= len) o[u] = t[u] = 0;  // left out: a partner is never entry 0
          a[u] = key[lo + t[u]];
          b[u] = key[lo + o[u]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (o[u] > 0 && a[u] > b[u]) {  // what was read for a pair left out may just be changing
            key[lo + t[u]] = b[u];
            key[lo + o[u]] = a[u];
          }
        }
      }
      // the wait is spelled out: with the barrier at the head of this loop the generated code (ROCm 7.2) had none for the LDS
      // writes of the stage before
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
      __syncthreads();
    }
  }
}

// The rows of a bucket, each sorted by (column, payload), to their place in the CSR.  One workgroup per bucket: the
// entries are grouped by row in LDS, then an entry's place is the number of entries of its row that come before it, or,
// in a row of more than kLongRow entries, where a sort leaves it.  The count is quadratic in the length: 200,000 entries, one
// row with 3,000 of them, took 757 us with it and take 119 us (145 in the radix sort); 128 entries as the limit were slower
// on rows of 200, 256 and 1,024 made no difference.
// Where row and column share 32 bits (NARROW) the count compares these alone, four entries a load: entries that are listed
// twice then have the same count, which shows once the entries are in order, and are put into the order of their payloads.  In
// order they are also written in order.
constexpr int kMaxBucketRows = 1024;
constexpr int kLongRow = 512;
constexpr int kSortTrips = kBucketRoom / kST;
template <bool NARROW>
__global__ __launch_bounds__(kST) void bucket_sort_kernel(const int32_t* __restrict__ fill, const int32_t* __restrict__ base,
                                                         const int* __restrict__ over, int shift, int room, int64_t n,
                                                         int64_t nnz_in, SlotBits bits,
                                                         const uint64_t* __restrict__ slots,
                                                         const double* __restrict__ val, int64_t* __restrict__ rowptr,
                                                         int32_t* __restrict__ col_out, double* __restrict__ val_out) {
  __shared__ __attribute__((aligned(16))) uint64_t key[kBucketRoom + 2];
  __shared__ int32_t next[kMaxBucketRows];
  __shared__ int32_t wave_sum[kST / 64];
  __shared__ int32_t long_row[kBucketRoom / kLongRow], nlong;
  if (*over) return;  // uniform over the grid
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int len = fill[b], rows = 1 << shift;
  const int64_t row0 = (int64_t)b << shift, at0 = base[b];
  const int row_bits = bits.col + bits.pay;
  for (int r = threadIdx.x; r < rows; r += kST) next[r] = 0;
  if (threadIdx.x == 0) nlong = 0;
  __syncthreads();
  const uint64_t* __restrict__ mine = slots + (int64_t)b * room;
  uint64_t own[kSortTrips];
#pragma unroll
  for (int u = 0; u < kSortTrips; ++u) {
    const int p = u * kST + (int)threadIdx.x;
    if (p < len) own[u] = mine[p];
  }
#pragma unroll
  for (int u = 0; u < kSortTrips; ++u)
    if (u * kST + (int)threadIdx.x < len) atomicAdd(&next[own[u] >> row_bits], 1);
  __syncthreads();
  {  // exclusive prefix sums over the rows: thread t has the rows 2 t and 2 t + 1
    int32_t v[kMaxBucketRows / kST], sum = 0;
#pragma unroll
    for (int q = 0; q < kMaxBucketRows / kST; ++q) {
      const int r = (int)threadIdx.x * (kMaxBucketRows / kST) + q;
      v[q] = r < rows ? next[r] : 0;
      sum += v[q];
    }
    int32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int32_t at = incl - sum;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
#pragma unroll
    for (int q = 0; q < kMaxBucketRows / kST; ++q) {
      const int r = (int)threadIdx.x * (kMaxBucketRows / kST) + q;
      if (r < rows) {
        next[r] = at;
        if (row0 + r < n) rowptr[row0 + r] = at0 + at;
        if (row0 + r == n - 1) rowptr[n] = at0 + at + v[q];
        if (v[q] > kLongRow) long_row[atomicAdd(&nlong, 1)] = r;
      }
      at += v[q];
    }
  }
  __syncthreads();
  const uint32_t cmask = (uint32_t)((1ull << bits.col) - 1);
  if (NARROW && nlong == 0) {  // uniform
    uint32_t* hi = reinterpret_cast<uint32_t*>(key);       // row and column
    uint32_t* pay = hi + kBucketRoom + 4;                   // payload
#pragma unroll
    for (int u = 0; u < kSortTrips; ++u) {
      if (u * kST + (int)threadIdx.x >= len) break;
      const int at = atomicAdd(&next[own[u] >> row_bits], 1);
      hi[at] = (uint32_t)(own[u] >> 32);
      pay[at] = (uint32_t)own[u];
    }
    if (threadIdx.x < 4) hi[len + (int)threadIdx.x] = 0xffffffffu;  // before nothing
    __syncthreads();
    // next[r] is now the end of row r and so the start of row r + 1
    uint32_t k[kSortTrips], e[kSortTrips];
    int to[kSortTrips];
#pragma unroll
    for (int u = 0; u < kSortTrips; ++u) {
      const int p = u * kST + (int)threadIdx.x;
      if (p >= len) break;
      k[u] = hi[p];
      e[u] = pay[p];
      const int r = (int)(k[u] >> bits.col), end = next[r];
      int q = (r ? next[r - 1] : 0) & ~3;  // up to three entries of the rows before come along: they are smaller
      int before = q;
      for (; q < end; q += 4) {  // and of the rows behind: they are not
        const uint4 h = *reinterpret_cast<const uint4*>(hi + q);
        before += h.x < k[u] ? 1 : 0;
        before += h.y < k[u] ? 1 : 0;
        before += h.z < k[u] ? 1 : 0;
        before += h.w < k[u] ? 1 : 0;
      }
      to[u] = before;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSortTrips; ++u) {
      if (u * kST + (int)threadIdx.x >= len) break;
      hi[to[u]] = k[u];
      pay[to[u]] = e[u];
    }
    __syncthreads();
    // A place that two entries share leaves the one behind it with what it held before, an entry of the same row that has its
    // own place: fewer different ones than places, which cannot all be in ascending order.
    int twice = 0;
    for (int p = threadIdx.x; p + 1 < len; p += kST) twice |= hi[p] >= hi[p + 1] ? 1 : 0;
    if (__syncthreads_or(twice)) {
      // the entries of one place side by side, each then counts the payloads below its own
      uint32_t* share = hi;
      for (int p = threadIdx.x; p < len; p += kST) share[p] = 0;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kSortTrips; ++u) {
        if (u * kST + (int)threadIdx.x >= len) break;
        pay[to[u] + (int)atomicAdd(&share[to[u]], 1u)] = e[u];
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kSortTrips; ++u) {
        if (u * kST + (int)threadIdx.x >= len) break;
        const int many = (int)share[to[u]], t0 = to[u];
        for (int q = 0; q < many; ++q) to[u] += pay[t0 + q] < e[u] ? 1 : 0;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kSortTrips; ++u) {
        if (u * kST + (int)threadIdx.x >= len) break;
        hi[to[u]] = k[u];
        pay[to[u]] = e[u];
      }
      __syncthreads();
    }
    for (int p = threadIdx.x; p < len; p += kST) {
      const int64_t e1 = (int64_t)pay[p];
      col_out[at0 + p] = (int32_t)(hi[p] & cmask);
      val_out[at0 + p] = val[e1 < nnz_in ? e1 : e1 - nnz_in];
    }
    return;
  }
#pragma unroll
  for (int u = 0; u < kSortTrips; ++u) {
    if (u * kST + (int)threadIdx.x >= len) break;
    key[atomicAdd(&next[own[u] >> row_bits], 1)] = own[u];
  }
  __syncthreads();
  for (int q = 0; q < nlong; ++q) {
    const int r = long_row[q], lo = r ? next[r - 1] : 0;
    sort_run(key, lo, next[r] - lo);
  }
  for (int p = threadIdx.x; p < len; p += kST) {
    const uint64_t k = key[p];
    const int r = (int)(k >> row_bits), lo = r ? next[r - 1] : 0, hi = next[r];
    int before = 0;
    if (hi - lo > kLongRow) {
      before = p - lo;
    } else {
#pragma unroll 4
      for (int q = lo; q < hi; ++q) before += key[q] < k ? 1 : 0;
    }
    const int64_t out = at0 + lo + before;
    const int64_t e = (int64_t)(k & ((1ull << bits.pay) - 1));
    col_out[out] = (int32_t)((uint32_t)(k >> bits.pay) & cmask);
    val_out[out] = val[e < nnz_in ? e : e - nnz_in];
  }
}

// mean[i] = (1/d) sum_t x_it (0 when centre == 0), norm[i] = |x_i - mean[i]|_2
__global__ __launch_bounds__(kT) void row_stats_kernel(const double* __restrict__ x, int64_t ldx, int64_t n, int d,
                                                       int centre, double* __restrict__ mean,
                                                       double* __restrict__ norm) {
  const int lane = threadIdx.x % kL;
  const int64_t i = (int64_t)blockIdx.x * (kT / kL) + threadIdx.x / kL;
  if (i >= n) return;
  const double* xi = x + i * ldx;
  constexpr int K = 8;  // coordinates of a lane that stay in registers for the second pass
  const bool once = d <= K * kL;
  double v[K], m = 0.0, ss = 0.0;
  if (once) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = lane + k * kL < d ? xi[lane + k * kL] : 0.0;
  }
  if (centre) {
    double acc = 0.0;
    if (once) {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (lane + k * kL < d) acc += v[k];
    } else {
      for (int t = lane; t < d; t += kL) acc += xi[t];
    }
    m = group_sum(acc) / (double)d;
  }
  if (once) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double c = v[k] - m;
      if (lane + k * kL < d) ss += c * c;
    }
  } else {
    for (int t = lane; t < d; t += kL) {
      const double c = xi[t] - m;
      ss += c * c;
    }
  }
  ss = group_sum(ss);
  if (lane == 0) {
    mean[i] = m;
    norm[i] = sqrt(ss);
  }
}

// The sum of a pair's products by P = 4 or 16 neighbouring lanes.  A unit is V coordinates; 16 sums, one for each residue of the
// units modulo 16, 16 / P in every lane, meet in the order of a butterfly over 8, 4, 2, 1: the same bits with either P.  With four
// lanes a wave's instructions work on 16 pairs: with 16 lanes a pair the instructions round the products took 72 % of the issue
// slots and were the bound of rows that come out of a cache or of LDS.
// The lanes read a chunk of P units with one load, and the chunks lie where the row b has its multiples of P units (64 or 256
// bytes): chunk q holds the units P q - s .. P q - s + P - 1 of the row, s = the row's offset from such a multiple, so that a
// chunk does not lie across one line of the L1 more than it must.  Lane j's m-th sum is then the one of the units (P m + j - s) mod
// 16, and the butterfly joins the same sums.
constexpr int kQ = 4;  // chunks in flight (8 and fewer waves: 3.8 M pairs of 90 coordinates 260 us for 238)
typedef double vec2 __attribute__((ext_vector_type(2)));

// NQ chunks from chunk c0 on (c0 a multiple of 16 / P).  LAST: they are the last ones that any row has; a row's last chunk may be
// the one before.  `a` and `b` point to where unit 0 of chunk 0 lies, s units before the rows; nothing outside the rows is
// read.  CENTRED: a has its mean taken out already (and is in LDS).
template <int P, int NQ, int V, bool LAST, bool DISTANCE, bool CENTRED>
__device__ __forceinline__ void pair_trip(const double* a, const double* __restrict__ b, double ma, double mb, int c0, int s,
                                          int dv, int j, double (&acc)[kL / P]) {
  vec2 av[NQ], bv[NQ];
  const int t0 = c0 * P + j;  // one address a row, the chunks at constant distances from it
  a += (int64_t)t0 * V;
  b += (int64_t)t0 * V;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int t = t0 + q * P;
    if ((q == 0 && t < s) || (LAST && q >= NQ - 2 && t >= dv + s)) continue;
    if (V == 2) {
      bv[q] = reinterpret_cast<const vec2*>(b)[q * P];
      if (!CENTRED) av[q] = reinterpret_cast<const vec2*>(a)[q * P];
    } else {
      bv[q].x = b[q * P];
      if (!CENTRED) av[q].x = a[q * P];
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int t = t0 + q * P;
    if ((q == 0 && t < s) || (LAST && q >= NQ - 2 && t >= dv + s)) continue;
    if (CENTRED) {
      if (V == 2) av[q] = reinterpret_cast<const vec2*>(a)[q * P];
      else av[q].x = a[q * P];
    }
#pragma unroll
    for (int h = 0; h < V; ++h) {
      if (DISTANCE) {
        const double g = av[q][h] - bv[q][h];
        acc[q % (kL / P)] += g * g;
      } else {
        acc[q % (kL / P)] += (CENTRED ? av[q][h] : av[q][h] - ma) * (bv[q][h] - mb);
      }
    }
  }
}

// The last NQ or fewer chunks, `left` of them (uniform).
template <int P, int NQ, int V, bool DISTANCE, bool CENTRED>
__device__ __forceinline__ void pair_last(const double* a, const double* __restrict__ b, double ma, double mb, int c0, int left,
                                          int s, int dv, int j, double (&acc)[kL / P]) {
  if constexpr (NQ > 0) {
    if (left == NQ) pair_trip<P, NQ, V, true, DISTANCE, CENTRED>(a, b, ma, mb, c0, s, dv, j, acc);
    else pair_last<P, NQ - 1, V, DISTANCE, CENTRED>(a, b, ma, mb, c0, left, s, dv, j, acc);
  }
}

// Chunks of a row of x at most.
inline int row_chunks(const double* x, int64_t ldx, int d, int v, int p) {
  const int dv = d / v;
  int s = p - 1;  // offset of a row from a multiple of p units at most
  if (ldx % (p * v) == 0) s = (int)(reinterpret_cast<uintptr_t>(x) / (8 * v) % p);
  return dv > 0 ? (dv + s + p - 1) / p : 0;
}

// All lanes of the pair get the sum.
template <int P, int V, bool DISTANCE, bool CENTRED>
__device__ __forceinline__ double pair_sum(const double* a, const double* __restrict__ b, double ma, double mb, int d, int nq,
                                           int j) {
  double acc[kL / P];
#pragma unroll
  for (int m = 0; m < kL / P; ++m) acc[m] = 0.0;
  const int dv = d / V, s = (int)(reinterpret_cast<uintptr_t>(b) / (8 * V) % P);
  const double *as = a - s * V, *bs = b - s * V;
  int c0 = 0;
#pragma unroll 1
  for (; c0 + kQ + 1 < nq; c0 += kQ) pair_trip<P, kQ, V, false, DISTANCE, CENTRED>(as, bs, ma, mb, c0, s, dv, j, acc);
  pair_last<P, kQ + 1, V, DISTANCE, CENTRED>(as, bs, ma, mb, c0, nq - c0, s, dv, j, acc);
  if (V == 2 && (d & 1) && j == s) {  // the last coordinate goes to the sum of unit 0
    const double f = a[d - 1], g = b[d - 1];
    if (DISTANCE) acc[0] += (f - g) * (f - g);
    else acc[0] += (CENTRED ? f : f - ma) * (g - mb);
  }
  double sum;
  if constexpr (P == 4) {
    sum = (acc[0] + acc[2]) + (acc[1] + acc[3]);
    sum += row_dpp<0x4e>(sum);  // quad_perm [2,3,0,1]
    sum += row_dpp<0xb1>(sum);  // quad_perm [1,0,3,2]
  } else {
    static_assert(P == kL, "4 or 16 lanes");
    sum = group_sum(acc[0]);
  }
  return sum;
}

// measure 0 / 1: val[e] = <x_u - m_u, x_v - m_v> / (norm_u norm_v)  (m = 0 for the cosine measure)
// measure 2:     val[e] = exp(-|x_u - x_v|^2 / (2 sigma^2))                                          (DISTANCE)
// By the P lanes of one pair.
template <int P, int V, bool DISTANCE>
__device__ __forceinline__ void edge_pair(const double* __restrict__ x, int64_t ldx, int d, const int32_t* __restrict__ eu,
                                          const int32_t* __restrict__ ev, int64_t e, int j, int nq, double inv_two_sigma2,
                                          const double* __restrict__ mean, const double* __restrict__ norm, int64_t n,
                                          int* __restrict__ bad, double* __restrict__ val) {
  const int64_t u = eu[e], v = ev[e];
  if (u < 0 || u >= n || v < 0 || v >= n) {  // uniform over the edge's lanes; no row is touched
    if (j == 0) {
      atomicOr(bad, 1);
      val[e] = __longlong_as_double(0x7ff8000000000000ll);
    }
    return;
  }
  const double mu = DISTANCE ? 0.0 : mean[u], mv = DISTANCE ? 0.0 : mean[v];
  const double nn = DISTANCE ? 1.0 : norm[u] * norm[v];
  const double sum = pair_sum<P, V, DISTANCE, false>(x + u * ldx, x + v * ldx, mu, mv, d, nq, j);
  if (j == 0) val[e] = DISTANCE ? exp(-sum * inv_two_sigma2) : sum / nn;
}

// every pair; an index out of range gives NaN and sets *bad
template <int P, int V, bool DISTANCE>
__global__ __launch_bounds__(kT) void edge_similarity_kernel(const double* __restrict__ x, int64_t ldx, int d,
                                                             const int32_t* __restrict__ eu,
                                                             const int32_t* __restrict__ ev, int64_t nedges, int nq,
                                                             double inv_two_sigma2, const double* __restrict__ mean,
                                                             const double* __restrict__ norm, int64_t n,
                                                             int* __restrict__ bad, double* __restrict__ val) {
  const int64_t e = (int64_t)blockIdx.x * (kT / P) + threadIdx.x / P;
  if (e >= nedges) return;
  edge_pair<P, V, DISTANCE>(x, ldx, d, eu, ev, e, threadIdx.x % P, nq, inv_two_sigma2, mean, norm, n, bad, val);
}

// the pairs list[0 .. *count - 1]: those that the buckets below have no room for, and those with an index out of range
template <int P, int V, bool DISTANCE>
__global__ __launch_bounds__(kT) void edge_list_kernel(const double* __restrict__ x, int64_t ldx, int d,
                                                       const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                                                       const uint32_t* __restrict__ list,
                                                       const int32_t* __restrict__ count, int nq, double inv_two_sigma2,
                                                       const double* __restrict__ mean, const double* __restrict__ norm,
                                                       int64_t n, int* __restrict__ bad, double* __restrict__ val) {
  const int64_t here = *count;
  for (int64_t p = (int64_t)blockIdx.x * (kT / P) + threadIdx.x / P; p < here; p += (int64_t)gridDim.x * (kT / P))
    edge_pair<P, V, DISTANCE>(x, ldx, d, eu, ev, list[p], threadIdx.x % P, nq, inv_two_sigma2, mean, norm, n, bad, val);
}

// exp() out of line: its constants, taken out of the loop over the pairs' chunks, would be spilled.
__device__ __attribute__((noinline)) double exp_apart(double v) { return exp(v); }

// The same for data that do not fit the L2s, by groups of neighbouring buckets of first rows: a workgroup keeps the rows of
// its group in LDS, puts the group's pairs into order of their second rows (bins, a counting sort in LDS) and reads those
// from memory: pairs that share one read it together.  The groups of an XCD are neighbours, so that where pairs join rows
// that are near one another (a voxel grid, a neighbour list after a renumbering) the second rows come from its L2 too.  A
// pair's value is formed by the same lanes in the same order as above.
// 3.8 M pairs of 142,541 rows of 90 doubles, listed offset by offset: 683 us with every row read from the Infinity Cache
// once per pair, 238 us by 16 lanes a pair (its instructions), 152 us by four: 113 of them the pairs' sums, for which the L1
// delivers 2.7 GB in lines of 64 bytes (80 us at one a clock), the rest is the staging and the ordering.  What follows a sum is done
// by a thread a pair: by the pair's lanes the division or the exponential was a fifth of the instructions.
// Rows of a workgroup (with 16 lanes a pair): 128 of them and one workgroup a compute unit 275 us, 64 and two 253, 32 and three 238.
// An XCD gets kRuns runs of neighbours from all over the rows, because first rows need not be spread evenly: with first
// rows drawn by a power law (half of the pairs in an eighth of the rows), one bucket a workgroup, one run per XCD took
// 1,880 us for the same number of pairs, 4 runs 1,000, 8 runs 865, 16 runs 775, and no buckets 945.  One counter of taken
// buckets per XCD, so that idle XCDs take over what is left, cost 200 us.
constexpr int kRuns = 16;
__host__ __device__ inline int edge_run(int nbuckets) { return (nbuckets + 8 * kRuns - 1) / (8 * kRuns); }
constexpr int kET = 512;         // threads of a workgroup
constexpr int kMaxGroup = 8;     // buckets of a workgroup at most
constexpr int kGroupRowBits = 9;  // bits of a row of a workgroup: kEdgeRowBytes hold 768 of the shortest rows, a bucket has 256 at most
constexpr int kEdgeBins = 1024;  // bins of second rows
constexpr int kPairsPerRow = 32;  // pairs ordered at a time, per first row (18 bytes of LDS each)
constexpr int kMaxPairTrips = 4;
constexpr int kBucketLanes = 4;  // lanes of a pair (8: 231 -> 258 us on the voxel list below; random second rows 180 -> 175)
// V: coordinates of a load (2 where all rows start on 16 bytes)
template <int V, bool DISTANCE>
__global__ __launch_bounds__(kET, 6) void edge_bucket_kernel(const double* __restrict__ x, int64_t ldx, int d, int shift,
                                                          int group, int nbuckets, int room, int cap,
                                                          const int32_t* __restrict__ fill,
                                                          const uint64_t* __restrict__ slots, SlotBits bits, int nq,
                                                          double inv_two_sigma2, const double* __restrict__ mean,
                                                          const double* __restrict__ norm, int64_t n,
                                                          double* __restrict__ val) {
  // rows (group << shift) x dl less their means, their norms, the pairs' sums, the ordered pairs (second row, place of the value,
  // bins, first row)
  extern __shared__ __attribute__((aligned(16))) double rows[];
  __shared__ int32_t wave_sum[kET / 64], before[kMaxGroup + 1];
  __shared__ int32_t vmin, vmax;
  const int ngroups = (nbuckets + group - 1) / group;
  const int wg = (int)(blockIdx.x / 8), run = edge_run(ngroups);
  const int gb = (wg / run * 8 + (int)(blockIdx.x % 8)) * run + wg % run;
  if (gb >= ngroups) return;  // uniform
  const int b0 = gb * group, dl = (d + 1) & ~1, nr = group << shift;
  const int64_t row0 = (int64_t)b0 << shift;
  double* nrow = rows + (size_t)nr * dl;
  double* total = nrow + nr;
  uint32_t* pv = reinterpret_cast<uint32_t*>(total + cap);
  uint32_t* pout = pv + cap;
  int32_t* bin = reinterpret_cast<int32_t*>(pout + cap);
  uint16_t* prow = reinterpret_cast<uint16_t*>(bin + kEdgeBins);
  if (threadIdx.x == 0) {
    int32_t sum = 0;
    for (int g = 0; g < group; ++g) {
      before[g] = sum;
      if (b0 + g < nbuckets) sum += fill[b0 + g] < room ? fill[b0 + g] : room;
    }
    before[group] = sum;
  }
  __syncthreads();
  const int count = before[group];
  if (count == 0) return;  // uniform
  {  // thread by thread the units of the rows one after the other, without a division a unit
    const int du = (d + V - 1) / V, step_r = kET / du, step_t = kET - step_r * du;
    int r = (int)threadIdx.x / du, t = (int)threadIdx.x - r * du;
#pragma unroll 2
    for (; r < nr && row0 + r < n;) {
      const double* __restrict__ from = x + (row0 + r) * ldx + V * t;
      const double m = DISTANCE ? 0.0 : mean[row0 + r];
      if (V == 2 && V * t + 1 < d) {
        vec2 v = *reinterpret_cast<const vec2*>(from);
        if (!DISTANCE) {
          v.x -= m;
          v.y -= m;
        }
        *reinterpret_cast<vec2*>(rows + r * dl + V * t) = v;
      } else {
        rows[r * dl + V * t] = DISTANCE ? *from : *from - m;
      }
      r += step_r;
      t += step_t;
      if (t >= du) {
        t -= du;
        ++r;
      }
    }
  }
  if (!DISTANCE) {
    for (int r = threadIdx.x; r < nr; r += kET) {
      if (row0 + r >= n) break;
      nrow[r] = norm[row0 + r];
    }
  }
  constexpr int P = kBucketLanes;
  const int j = threadIdx.x % P;
#pragma unroll 1
  for (int c0 = 0; c0 < count; c0 += cap) {  // uniform
    const int here = count - c0 < cap ? count - c0 : cap;
    __syncthreads();  // the pairs of the trip before are done with
    if (threadIdx.x == 0) {
      vmin = INT32_MAX;
      vmax = 0;
    }
    for (int i = threadIdx.x; i < kEdgeBins; i += kET) bin[i] = 0;
    __syncthreads();
    int lo = INT32_MAX, hi = 0;
    uint64_t* own = reinterpret_cast<uint64_t*>(total);  // the pairs as they come
    const uint32_t vmask = (uint32_t)((1ull << bits.col) - 1);
#pragma unroll
    for (int u = 0; u < kMaxPairTrips; ++u) {
      const int p = u * kET + (int)threadIdx.x;
      if (p >= here) break;
      int g = 0;
      while (c0 + p >= before[g + 1]) ++g;  // before[group] = count > c0 + p
      const uint64_t slot = slots[(int64_t)(b0 + g) * room + (c0 + p - before[g])];
      // the upper half: row of the group and second row
      own[p] = slot + ((uint64_t)(g << shift) << (bits.col + 32));
      const int v = (int)((uint32_t)(slot >> 32) & vmask);
      lo = min(lo, v);
      hi = max(hi, v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo = min(lo, __shfl_xor(lo, o, 64));
      hi = max(hi, __shfl_xor(hi, o, 64));
    }
    if ((threadIdx.x & 63) == 0) {
      atomicMin(&vmin, lo);
      atomicMax(&vmax, hi);
    }
    __syncthreads();
    const int first = vmin, spread = vmax - vmin;
    int wide = 0;
    while ((spread >> wide) >= kEdgeBins) ++wide;
#pragma unroll
    for (int u = 0; u < kMaxPairTrips; ++u) {
      const int p = u * kET + (int)threadIdx.x;
      if (p >= here) break;
      atomicAdd(&bin[((int)((uint32_t)(own[p] >> 32) & vmask) - first) >> wide], 1);
    }
    __syncthreads();
    {  // exclusive prefix sums: thread t has the bins 2 t and 2 t + 1
      static_assert(kEdgeBins == 2 * kET, "two bins a thread");
      const int a = bin[2 * threadIdx.x], sum = a + bin[2 * threadIdx.x + 1];
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o, 64);
        if ((int)(threadIdx.x & 63) >= o) incl += up;
      }
      if ((threadIdx.x & 63) == 63) wave_sum[threadIdx.x >> 6] = incl;
      __syncthreads();
      int at = incl - sum;
      for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) at += wave_sum[w];
      bin[2 * threadIdx.x] = at;
      bin[2 * threadIdx.x + 1] = at + a;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kMaxPairTrips; ++u) {
      const int p = u * kET + (int)threadIdx.x;
      if (p >= here) break;
      const uint64_t slot = own[p];
      const uint32_t v = (uint32_t)(slot >> 32) & vmask;
      const int at = atomicAdd(&bin[((int)v - first) >> wide], 1);
      pv[at] = v;
      pout[at] = (uint32_t)slot;
      prow[at] = (uint16_t)(slot >> (bits.col + 32));
    }
    __syncthreads();
#pragma unroll 1
    for (int p = threadIdx.x / P; p < here; p += kET / P) {  // uniform over the pair's lanes
      const uint32_t vi = pv[p];
      const double mv = DISTANCE ? 0.0 : mean[vi];
      const double sum = pair_sum<P, V, DISTANCE, true>(rows + prow[p] * dl, x + (int64_t)vi * ldx, 0.0, mv, d, nq, j);
      if (j == 0) total[p] = sum;
    }
    __syncthreads();
    // what follows the sum, a thread a pair
#pragma unroll 1
    for (int p = threadIdx.x; p < here; p += kET)
      val[pout[p]] = DISTANCE ? exp_apart(-total[p] * inv_two_sigma2) : total[p] / (nrow[prow[p]] * norm[pv[p]]);
  }
}

// key[p] = row << bits | col of output entry p, src[p] = the listed entry it copies.  Entry e gives output e; with
// symmetrize its mirror (col, row) is output nnz_in + e, or a key of row n (sorted past the end, then dropped) when
// row == col.
__global__ __launch_bounds__(kT) void coo_keys_kernel(const int32_t* __restrict__ row, const int32_t* __restrict__ col,
                                                      int64_t nnz_in, int symmetrize, int64_t n, int bits,
                                                      uint64_t* __restrict__ key, uint32_t* __restrict__ src,
                                                      int* __restrict__ bad) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (e >= nnz_in) return;
  const int64_t r = row[e], c = col[e];
  const uint64_t none = (uint64_t)n << bits;
  src[e] = (uint32_t)e;
  if (symmetrize) src[nnz_in + e] = (uint32_t)e;
  if (r < 0 || r >= n || c < 0 || c >= n) {
    atomicOr(bad, 1);
    key[e] = none;
    if (symmetrize) key[nnz_in + e] = none;
    return;
  }
  key[e] = ((uint64_t)r << bits) | (uint64_t)c;
  if (symmetrize) key[nnz_in + e] = r == c ? none : (((uint64_t)c << bits) | (uint64_t)r);
}

// rowptr[i] = first sorted position whose row is >= i, i = 0 .. n
__global__ __launch_bounds__(kT) void coo_rowptr_kernel(const uint64_t* __restrict__ key, int64_t total, int64_t n, int bits,
                                                        int64_t* __restrict__ rowptr) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i > n) return;
  int64_t lo = 0, hi = total;
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if ((int64_t)(key[mid] >> bits) < i) {
      lo = mid + 1;
    } else {
      hi = mid;
    }
  }
  rowptr[i] = lo;
}

__global__ __launch_bounds__(kT) void coo_emit_kernel(const uint64_t* __restrict__ key, const uint32_t* __restrict__ src,
                                                      const double* __restrict__ val, int64_t nnz_out, int bits,
                                                      int32_t* __restrict__ col_out, double* __restrict__ val_out) {
  const int64_t p = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (p >= nnz_out) return;
  col_out[p] = (int32_t)(key[p] & ((1ull << bits) - 1ull));
  val_out[p] = val[src[p]];
}

int key_bits(int64_t n) {
  int b = 1;
  while (b < 32 && ((int64_t)1 << b) < n) ++b;
  return b;
}

}  // namespace

hipError_t launch_row_stats(const double* x, int64_t ldx, int64_t n, int d, int centre, double* mean, double* norm,
                            hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(row_stats_kernel, dim3(blocks(n * kL)), dim3(kT), 0, st, x, ldx, n, d, centre, mean, norm);
  return hipGetLastError();
}

// Lanes of a pair where rows are read pair by pair: 16 where long rows come out of memory, whose loads then ask for whole lines
// (300,000 x 128, 6 random pairs a row: 512 us, 550 with 4 lanes; 300,000 x 90, 3 voxel pairs a row: 158 and 184), else 4 (30,000 x
// 64, 26 voxel pairs a row: 100 and 116; 142,541 x 8, 38 pairs: 149 and 384).
inline int edge_lanes(int64_t n, int d) { return d >= 32 && n * d >= 5000000 ? kL : 4; }

hipError_t launch_edge_similarity(const double* x, int64_t ldx, int d, const int32_t* eu, const int32_t* ev,
                                  int64_t nedges, int measure, double sigma, const double* mean, const double* norm,
                                  int64_t n, int* bad, double* val, hipStream_t st) {
  if (nedges <= 0) return hipSuccess;
  const int vec_ok = (ldx % 2 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0) ? 1 : 0;
  const double inv = measure == 2 ? 1.0 / (2.0 * sigma * sigma) : 0.0;
  const int p = edge_lanes(n, d);
#define SC_EDGE(V, DISTANCE)                \
  do {                                      \
    if (p == 4) SC_EDGE_(4, V, DISTANCE);   \
    else SC_EDGE_(kL, V, DISTANCE);         \
  } while (0)
#define SC_EDGE_(P, V, DISTANCE)                                                                                            \
  hipLaunchKernelGGL((edge_similarity_kernel<P, V, DISTANCE>), dim3(blocks(nedges * P)), dim3(kT), 0, st, x, ldx, d, eu, ev, \
                     nedges, row_chunks(x, ldx, d, V, P), inv, mean, norm, n, bad, val)
  if (vec_ok) {
    if (measure == 2) SC_EDGE(2, true); else SC_EDGE(2, false);
  } else {
    if (measure == 2) SC_EDGE(1, true); else SC_EDGE(1, false);
  }
#undef SC_EDGE
#undef SC_EDGE_
  return hipGetLastError();
}

namespace {

struct BucketPlan {
  bool use = false;
  int shift = 0, buckets = 0, room = 0;
  SlotBits bits = {0, 0};
  size_t slot_count() const { return (size_t)buckets * room; }  // 8 bytes each
};

// Slots per bucket: as many as the LDS takes, but no more than `most` per entry in all unless that is little anyway
// (64 MB).  Entries that find no room cost more than unused slots do: 131,072 rows of 380 coordinates with 8 pairs a row
// get 512 slots for 64 pairs a bucket on average.
int bucket_room(int64_t buckets, int64_t entries, int64_t most) {
  int room = kBucketRoom;
  while (room > 64 && buckets * room > most * entries && buckets * room * 12 > (int64_t)64 << 20) room /= 2;
  return room;
}

// Rows per bucket: about 2,048 entries in a bucket that holds 4,096, fewer where that leaves the chip without work.
BucketPlan plan_buckets(int64_t total, int64_t n) {
  BucketPlan p;
  if (n < 1) return p;
  int64_t target = total / 1024;
  target = target < 256 ? 256 : (target > kBucketRoom / 2 ? kBucketRoom / 2 : target);
  while (p.shift < 10 && ((int64_t)2 << p.shift) * total <= target * n) ++p.shift;
  const int64_t nb = ((n - 1) >> p.shift) + 1;
  // more buckets than a workgroup has counters, or rows so long that ranking their entries (quadratic in the length) costs
  // more than the sort: 2,000 rows of 2,000 entries take 1,124 us in buckets and 390 us in the radix sort
  // or so few entries that most buckets are next to empty
  p.use = nb <= kMaxBuckets && total <= nb * (kBucketRoom / 2) && total <= 256 * n && (nb <= 1024 || nb * 128 <= total);
  p.buckets = (int)nb;
  p.room = bucket_room(nb, total, 8);
  p.bits.col = key_bits(n);
  p.bits.pay = p.bits.col + p.shift <= 32 ? 32 : 64 - p.bits.col - p.shift;
  return p;
}

void launch_partition(const int32_t* row, const int32_t* col, int64_t nnz_in, int64_t n, bool mirror, const BucketPlan& p,
                      int32_t* fill, uint64_t* slots, uint32_t* rest, int32_t* nrest, int* bad,
                      hipStream_t st) {
  const int64_t total = mirror ? 2 * nnz_in : nnz_in;
  const int64_t per = (int64_t)kPartThreads * (total <= kPartFew ? kPartTripsFew : kPartTrips);
#define SC_PARTITION(MIR, TRIPS)                                                                                       \
  hipLaunchKernelGGL((partition_kernel<MIR, TRIPS>), dim3((unsigned)((total + per - 1) / per)), dim3(kPartThreads), 0, \
                     st, row, col, nnz_in, n, p.shift, p.buckets, p.room, fill, slots, p.bits, rest, nrest, bad)
  if (total <= kPartFew) {
    if (mirror) SC_PARTITION(true, kPartTripsFew); else SC_PARTITION(false, kPartTripsFew);
  } else {
    if (mirror) SC_PARTITION(true, kPartTrips); else SC_PARTITION(false, kPartTrips);
  }
#undef SC_PARTITION
}

size_t up256(size_t bytes) { return (bytes + 255) / 256 * 256; }

size_t radix_workspace(int64_t total) {
  size_t sort_bytes = 0;
  (void)rocprim::radix_sort_pairs(nullptr, sort_bytes, (const uint64_t*)nullptr, (uint64_t*)nullptr,
                                  (const uint32_t*)nullptr, (uint32_t*)nullptr, (size_t)total, 0u, 64u,
                                  (hipStream_t) nullptr);
  // temp | key[total] | key_sorted[total] | src[total] | src_sorted[total]
  return up256(sort_bytes) + (size_t)total * 24 + 1024;
}

}  // namespace

size_t coo_to_csr_workspace(int64_t total, int64_t n, int radix) {
  const BucketPlan p = plan_buckets(total, n);
  // over, fill[buckets] | base[buckets] | slots
  if (p.use && !radix) return 2 * up256((size_t)p.buckets * 4 + 8) + p.slot_count() * 8 + 1024;
  return radix_workspace(total);
}

// Entries sorted by (row, col); listed duplicates stay separate entries in listing order.  rowptr_out[n] is the number
// of entries emitted; col_out / val_out need room for `total` entries, total = nnz_in * (symmetrize ? 2 : 1) < 2^31.
// bad: device int[2]; bad[0] |= 1 if an index is out of range; bad[1] = 1 if a bucket overflowed and nothing was done: the
// caller then calls again with radix = 1, as it does where the scratch of the buckets cannot be had.  A row that is longer
// than a bucket thus costs the partition on top of the sort: 200,000 entries 152 -> 159 us, 3.8 M 535 -> 559 us.
//
// 3.8 M pairs of 142,541 rows (7.6 M entries): radix sort of 64-bit keys 640 us, with the keys, row pointers and gather
// round it 730 us; buckets 125 us: partition 25 (50 with every lane adding for itself and slots of 12 bytes), sort 66 (95 while the
// ranking compared 64 bits, an entry a load, and the entries were written where they ranked; bound by the ranking's compares and
// the gather of the values).
hipError_t coo_to_csr(const int32_t* row, const int32_t* col, const double* val, int64_t nnz_in, int64_t n,
                      int symmetrize, int radix, void* work, size_t work_bytes, int64_t* rowptr_out, int32_t* col_out,
                      double* val_out, int* bad, hipStream_t st) {
  const int64_t total = nnz_in * (symmetrize ? 2 : 1);
  if (total <= 0 || total > INT32_MAX || work_bytes < coo_to_csr_workspace(total, n, radix)) return hipErrorInvalidValue;
  char* base = static_cast<char*>(work);
  const BucketPlan p = plan_buckets(total, n);
  if (p.use && !radix) {
    int32_t* fill = reinterpret_cast<int32_t*>(base);
    int32_t* first = reinterpret_cast<int32_t*>(base + up256((size_t)p.buckets * 4 + 8));
    uint64_t* slots = reinterpret_cast<uint64_t*>(base + 2 * up256((size_t)p.buckets * 4 + 8));
    hipError_t e = launch_fill_int32(fill, p.buckets, 0, 0, st);
    if (e != hipSuccess) return e;
    launch_partition(row, col, nnz_in, n, symmetrize != 0, p, fill, slots, nullptr, nullptr, bad, st);
    hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(kPartThreads), 0, st, fill, p.buckets, p.room, first, bad + 1);
#define SC_BUCKET_SORT(NARROW)                                                                                            \
  hipLaunchKernelGGL((bucket_sort_kernel<NARROW>), dim3((unsigned)p.buckets), dim3(kST), 0, st, fill, first, bad + 1, p.shift, \
                     p.room, n, nnz_in, p.bits, slots, val, rowptr_out, col_out, val_out)
    if (p.bits.pay == 32) SC_BUCKET_SORT(true); else SC_BUCKET_SORT(false);
#undef SC_BUCKET_SORT
    return hipGetLastError();
  }
  size_t sort_bytes = 0;
  hipError_t e = rocprim::radix_sort_pairs(nullptr, sort_bytes, (const uint64_t*)nullptr, (uint64_t*)nullptr,
                                           (const uint32_t*)nullptr, (uint32_t*)nullptr, (size_t)total, 0u, 64u, st);
  if (e != hipSuccess) return e;
  uint64_t* key = reinterpret_cast<uint64_t*>(base + up256(sort_bytes));
  uint64_t* key_sorted = key + total;
  uint32_t* src = reinterpret_cast<uint32_t*>(key_sorted + total);
  uint32_t* src_sorted = src + total;
  const int bits = key_bits(n + 1);  // row n stands for dropped entries
  hipLaunchKernelGGL(coo_keys_kernel, dim3(blocks(nnz_in)), dim3(kT), 0, st, row, col, nnz_in, symmetrize, n, bits, key,
                     src, bad);
  size_t sb = sort_bytes;
  e = rocprim::radix_sort_pairs(base, sb, key, key_sorted, src, src_sorted, (size_t)total, 0u, (unsigned)(2 * bits), st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(coo_rowptr_kernel, dim3(blocks(n + 1)), dim3(kT), 0, st, key_sorted, total, n, bits, rowptr_out);
  // entries past rowptr[n] are the dropped ones; emitting them too is harmless but the caller's arrays hold exactly
  // `total` slots, so emit everything and let rowptr[n] say how many count
  hipLaunchKernelGGL(coo_emit_kernel, dim3(blocks(total)), dim3(kT), 0, st, key_sorted, src_sorted, val, total, bits,
                     col_out, val_out);
  return hipGetLastError();
}

namespace {

// Rows of a bucket: a power of two that fits kEdgeRowBytes, about half a bucket's room of pairs.  Used where the data exceed what
// the L2s hold between them and a row occurs in several pairs: 142,541 x 90 with 27 pairs a row 726 -> 478 us, 60,000 x 90 with 26
// 322 -> 226 us, 142,541 x 128 with 38 1,382 -> 535 us (now 215, 121 and 355);
// 142,541 x 33 with 27 448 -> 436 us, 30,000 x 64 with 26 115 -> 148 us, 142,541 x 90 with 3 111 -> 151 us.
// Where that would be more buckets than a workgroup of the partition counts, they get up to twice the bytes: 142,541 x 200 with 27
// pairs a row 1,660 -> 410 us, 1,000,000 x 64 with 27 4,030 -> 1,240, 300,000 x 128 with 10 random pairs a row 1,085 -> 705.
constexpr int64_t kEdgeRowBytes = 24 * 1024;  // rows of a workgroup, beside its pairs
BucketPlan plan_edge_buckets(int64_t n, int d, int64_t nedges) {
  BucketPlan p;
  if (n * (int64_t)d < 5000000 || nedges < 8 * n) return p;
  const int64_t row_bytes = (int64_t)((d + 1) & ~1) * 8 + 16;
  while (p.shift < 8 && ((int64_t)2 << p.shift) * nedges <= kBucketRoom / 2 * n &&
         ((int64_t)2 << p.shift) * row_bytes <= (((n - 1) >> p.shift) + 1 > kMaxBuckets ? 2 * kEdgeRowBytes : kEdgeRowBytes))
    ++p.shift;
  const int64_t nb = ((n - 1) >> p.shift) + 1;
  p.bits.col = key_bits(n);
  p.bits.pay = 32;
  if (p.shift < 3 || nb > kMaxBuckets || nedges > nb * (kBucketRoom / 2) || p.bits.col + kGroupRowBits > 32) return p;
  p.use = true;
  p.buckets = (int)nb;
  p.room = bucket_room(nb, nedges, 8);
  return p;
}

}  // namespace

size_t edge_buckets_workspace(int64_t n, int d, int64_t nedges) {
  const BucketPlan p = plan_edge_buckets(n, d, nedges);
  // fill[buckets] | slots | rest[nedges]
  return p.use ? up256((size_t)p.buckets * 4) + p.slot_count() * 8 + (size_t)nedges * 4 + 1024 : 0;
}

hipError_t launch_edge_similarity_buckets(const double* x, int64_t ldx, int d, const int32_t* eu, const int32_t* ev,
                                          int64_t nedges, int measure, double sigma, const double* mean,
                                          const double* norm, int64_t n, void* work, size_t work_bytes, int* bad,
                                          int32_t* nrest, double* val, hipStream_t st) {
  const BucketPlan p = plan_edge_buckets(n, d, nedges);
  if (!p.use || work_bytes < edge_buckets_workspace(n, d, nedges)) return hipErrorInvalidValue;
  int32_t* fill = static_cast<int32_t*>(work);
  uint64_t* slots = reinterpret_cast<uint64_t*>(static_cast<char*>(work) + up256((size_t)p.buckets * 4));
  uint32_t* rest = reinterpret_cast<uint32_t*>(slots + p.slot_count());
  const hipError_t e = launch_fill_int32(fill, p.buckets, 0, 0, st);
  if (e != hipSuccess) return e;
  launch_partition(eu, ev, nedges, n, false, p, fill, slots, rest, nrest, bad, st);
  const int vec_ok = (ldx % 2 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0) ? 1 : 0;
  const double inv = measure == 2 ? 1.0 / (2.0 * sigma * sigma) : 0.0;
  // Buckets of a workgroup: as many as its LDS takes (few coordinates), while there are eight workgroups a compute unit.
  const int64_t row_bytes = (int64_t)(((d + 1) & ~1) + 2) * 8;
  int group = 1;
  while (group < kMaxGroup && ((int64_t)2 * group << p.shift) * row_bytes <= kEdgeRowBytes &&
         p.buckets / (2 * group) >= 2048)
    group *= 2;
  const int nr = group << p.shift;
  int cap = nr * kPairsPerRow / 4 * 4;
  cap = cap < kET ? kET : (cap > kMaxPairTrips * kET ? kMaxPairTrips * kET : cap);
  size_t lds = (size_t)nr * row_bytes + (size_t)cap * 18 + kEdgeBins * 4;
  while (lds > 160 * 1024 - 512 && cap > kET) {
    cap -= kET;
    lds -= (size_t)kET * 18;
  }
  const int ngroups = (p.buckets + group - 1) / group;
#define SC_EDGE_BUCKETS(V, DISTANCE)                                                                                   \
  do {                                                                                                                  \
    const hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&edge_bucket_kernel<V, DISTANCE>),         \
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                   \
    if (ea != hipSuccess) return ea;                                                                                    \
    hipLaunchKernelGGL((edge_bucket_kernel<V, DISTANCE>), dim3((unsigned)(8 * kRuns * edge_run(ngroups))), dim3(kET),  \
                       lds, st, x, ldx, d, p.shift, group, p.buckets, p.room, cap, fill, slots, p.bits,                \
                       row_chunks(x, ldx, d, V, kBucketLanes), inv, mean, norm, n, val);                               \
  } while (0)
  if (vec_ok) {
    if (measure == 2) SC_EDGE_BUCKETS(2, true); else SC_EDGE_BUCKETS(2, false);
  } else {
    if (measure == 2) SC_EDGE_BUCKETS(1, true); else SC_EDGE_BUCKETS(1, false);
  }
#undef SC_EDGE_BUCKETS
#define SC_EDGE_LIST(V, DISTANCE)                                                                                       \
  hipLaunchKernelGGL((edge_list_kernel<kL, V, DISTANCE>), dim3(2048), dim3(kT), 0, st, x, ldx, d, eu, ev, rest, nrest,  \
                     row_chunks(x, ldx, d, V, kL), inv, mean, norm, n, bad, val)
  if (vec_ok) {
    if (measure == 2) SC_EDGE_LIST(2, true); else SC_EDGE_LIST(2, false);
  } else {
    if (measure == 2) SC_EDGE_LIST(1, true); else SC_EDGE_LIST(1, false);
  }
#undef SC_EDGE_LIST
  return hipGetLastError();
}

}  // namespace sceig
