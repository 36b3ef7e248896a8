// Chebyshev start-block filter with the iterates resident in LDS.
//
// The filter applies d steps of the three-term recurrence  u+ = alpha (S u - shift u) - beta u-  to a block of b
// vectors (Algorithm 3 leaves the start vector free; the solver filters its re-injection blocks).  One launch of the
// general product kernel per step gathers, for every matrix entry, a whole operand row from the L2 caches, and the
// rate of those gathers - not HBM - bounds it.  But the similarity graphs here are block diagonal (one diagonal block
// per connected component, contiguous rows after the solver's renumbering), and a step of the recurrence on one block
// needs nothing from outside the block.  So one workgroup takes one diagonal block (or a 16-column slice of it), keeps
// the two iterates u and u- in LDS for all d steps and the block's matrix entries in registers: after the first step
// nothing is read from memory, and nothing is written until the last.
//
//   * A lane carries 8 adjacent columns; CL = 4 lanes (32 columns) or 2 lanes (16 columns) form a lane group that
//     works on one piece of one row at a time, so a step needs no sum across lanes at all.
//   * Rows are cut into chunks of at most 8 CL entries (32 or 16) and the chunks, numbered in row order, are dealt
//     to the 1024 / CL lane groups; a group owns at most two chunks and keeps their entries - eight (column, value)
//     pairs per lane - in registers for the whole launch.  A hub row of several hundred entries is thus spread over
//     as many groups as it has chunks instead of being walked by one.  The kNN graphs' rows are ordered by length
//     inside a component, so the chunks that share a wave are equally long.
//   * One round: every lane group hands the round's entry from the lane that holds it to its other lanes with a DPP
//     quad permute (an ALU move, no LDS traffic), reads the 64 bytes of its 8 columns of that operand row from LDS
//     and does 8 multiply-adds.  A lane's 8 columns are four 16-byte pieces CL apart, so that one read instruction
//     of a lane group covers 16 CL contiguous bytes (a "segment": a quarter of the row).  A row of 8 CL doubles is a
//     whole number of LDS bank periods, so lane groups that read the same segment of different rows in the same
//     instruction hit the same banks.  Neighbouring lane groups therefore take the four segments in rotated order
//     (group w reads segment (t + w) mod 4 in its t-th read; its t-th pair of accumulators belongs to that segment
//     throughout), and the four groups of a 16-lane pass always touch four different segments.  Measured per step
//     on 2,000 blocks of 250 rows, 32 columns: 92 us with every group reading the segments in the same order, 59 us
//     with a row-dependent xor placement of the pieces (bank-conflict cycles still 49 % of the LDS-active cycles),
//     42 us with the rotation (conflict cycles below 0.2 %); the product-per-step kernel takes 166 us.
//   * The group that owns the first chunk of a row applies the recurrence with its own sum and stores the new row over
//     u- in place (only the row's owner reads it); the other chunks of a row park their sums in LDS, and after a
//     barrier the row's owner adds them in chunk order (fixed, so results are reproducible).  Blocks without hub rows
//     skip that barrier.  One more barrier ends the step and the two buffers swap roles.
//   * Work items (row0, rows, col0, CL, extra chunks) are built by the host from the diagonal blocks and their chunk
//     counts; an item's LDS need is 2 rows x 8 CL doubles for the iterates, 8 CL doubles per extra chunk, and two
//     int32 per row for the block's row pointers and chunk offsets.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <type_traits>

#include <rocprim/device/device_scan.hpp>
#include <rocprim/functional.hpp>
#include <rocprim/device/device_select.hpp>
#include <rocprim/iterator/counting_iterator.hpp>

#include "kernels.h"

namespace sceig {
namespace {

constexpr int kRT = 1024;  // threads per workgroup
constexpr int kRK = 8;     // entries per lane and chunk
constexpr int kRS = 2;     // chunks per lane group
constexpr int kShape16 = 8, kShape8 = 9, kShape4 = 10;  // shape words of the sliced items

__host__ __device__ inline size_t resident_lds_bytes(int nrows, int cl, int extra) {
  const size_t bs = (size_t)8 * cl;
  return ((size_t)2 * nrows * bs * sizeof(double) + (size_t)extra * bs * sizeof(double) +
          (size_t)2 * (nrows + 1) * sizeof(int32_t) + 15) / 16 * 16;
}

// Entry idx = i * b + t of a random start block (the same numbers as random_block_kernel writes: uniform in [-1, 1)
// from the output function of splitmix64 applied to key + idx, key = mix of seed and block number made on the host).
__device__ __forceinline__ uint64_t res_mix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}
__device__ __forceinline__ double random_entry(uint64_t key, int64_t idx) {
  const uint64_t h = res_mix64(key + (uint64_t)idx);
  return 2.0 * ((double)(h >> 11) * (1.0 / 9007199254740992.0)) - 1.0;
}

template <int CTRL>
__device__ __forceinline__ int dpp_int(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
  return __hiloint2double(dpp_int<CTRL>(__double2hiint(v)), dpp_int<CTRL>(__double2loint(v)));
}
template <int CTRL>
__device__ __forceinline__ float dpp_float(float v) {
  return __int_as_float(dpp_int<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_value(double v) { return dpp_double<CTRL>(v); }
template <int CTRL>
__device__ __forceinline__ float dpp_value(float v) { return dpp_float<CTRL>(v); }
// two adjacent columns of an iterate, in the precision of the step
template <typename T> struct Pair;
template <> struct Pair<double> { using type = double2; };
template <> struct Pair<float> { using type = float2; };
// quad permute that gives every lane of a CL-lane group the value held by the group's lane Q
template <int CL, int Q>
struct GroupBcast {
  static constexpr int ctrl = CL == 4 ? Q * 0x55 : (Q == 0 ? 0xA0 : 0xF5);
};

template <int CL>
__device__ __forceinline__ void resident_item(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                              const double* __restrict__ val, const double* __restrict__ x,
                                              double* __restrict__ y, int64_t ldy, int b, int d, double alpha_first,
                                              double alpha_rest, double shift, int row0, int nr, int col0, int nx,
                                              unsigned char* smem, int d32, uint64_t rnd_key, int use_rnd) {
  constexpr int BS = 8 * CL;     // columns of the item
  constexpr int CH = kRK * CL;   // entries per chunk
  constexpr int G = kRT / CL;    // lane groups
  constexpr int RW = BS / 2;     // double2 per operand row
  double* bufa = reinterpret_cast<double*>(smem);
  double* bufb = bufa + (size_t)nr * BS;
  double* part = bufb + (size_t)nr * BS;
  int32_t* rpl = reinterpret_cast<int32_t*>(part + (size_t)nx * BS);
  int32_t* cst = rpl + (nr + 1);
  const int tid = threadIdx.x;
  const int q = tid % CL, g = tid / CL;
  // this lane's t-th piece (double2 index inside a row): segment (t + g) mod 4, position q inside the segment
  const int pc0 = ((g + 0) & 3) * CL + q, pc1 = ((g + 1) & 3) * CL + q, pc2 = ((g + 2) & 3) * CL + q,
            pc3 = ((g + 3) & 3) * CL + q;
  const int pcs[4] = {pc0, pc1, pc2, pc3};
  const int64_t ebase = rowptr[row0];
  const int nnz_local = (int)(rowptr[row0 + nr] - ebase);

  // ---- stage: row pointers relative to the block's first entry, chunk counts, u = the slice of x, u- = 0
  // (the first d32 steps run in single precision, on float iterates that take the first half of each buffer)
  for (int r = tid; r <= nr; r += kRT) rpl[r] = (int)(rowptr[row0 + r] - ebase);
  for (int idx = tid; idx < nr * BS; idx += kRT) {
    const int r = idx / BS, t = idx - r * BS;
    // the operand, or (use_rnd, uniform) the random start block's entry made on the spot instead of read
    const int64_t gi = (int64_t)(row0 + r) * b + col0 + t;
    const double xv = use_rnd ? random_entry(rnd_key, gi) : x[gi];
    if (d32 > 0) {  // uniform
      reinterpret_cast<float*>(bufa)[idx] = (float)xv;
      reinterpret_cast<float*>(bufb)[idx] = 0.0f;
    } else {
      bufa[idx] = xv;
      bufb[idx] = 0.0;
    }
  }
  __syncthreads();
  for (int r = tid; r < nr; r += kRT) {
    const int len = rpl[r + 1] - rpl[r];
    cst[r + 1] = len > CH ? (len + CH - 1) / CH : 1;  // an empty row still is one (empty) chunk
  }
  if (tid == 0) cst[0] = 0;
  __syncthreads();
  if (tid < 64) {  // exclusive prefix sums of the chunk counts: 64 lanes, a contiguous run of rows each
    const int per = (nr + 63) / 64;
    const int lo = tid * per < nr ? tid * per : nr, hi = lo + per < nr ? lo + per : nr;
    int total = 0;
    for (int r = lo; r < hi; ++r) total += cst[r + 1];
    int incl = total;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (tid >= o) incl += up;
    }
    int run = incl - total;
    for (int r = lo; r < hi; ++r) {
      run += cst[r + 1];
      cst[r + 1] = run;
    }
  }
  __syncthreads();
  const int nv = cst[nr];  // chunks of the block; the host made sure that nv <= kRS * G and nv - nr == nx

  const int32_t* cp = col + ebase;
  const double* vp = val + ebase;
  const unsigned last_row = (unsigned)(nr - 1);

  // ---- the group's chunks: row, place among the row's chunks, entries (kept in registers for all steps)
  int32_t kc[kRS][kRK];
  double ka[kRS][kRK];
  int crow[kRS], cidx[kRS], cnum[kRS], krounds[kRS];
#pragma unroll
  for (int sl = 0; sl < kRS; ++sl) {
    const int v = g + sl * G;
    const bool valid = v < nv;
    int lo = 0, hi = nr;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (cst[mid] <= (valid ? v : 0)) lo = mid; else hi = mid;
    }
    const int r = lo;
    const int j = valid ? v - cst[r] : 0;
    const int e0 = rpl[r] + j * CH;
    int e1 = rpl[r + 1];
    e1 = e1 < e0 + CH ? e1 : e0 + CH;
    if (!valid) e1 = e0;
    crow[sl] = valid ? r : -1;
    cidx[sl] = j;
    cnum[sl] = cst[r + 1] - cst[r];
#pragma unroll
    for (int k = 0; k < kRK; ++k) {
      int idx = e0 + k * CL + q;
      const bool in = idx < e1;
      idx = in ? idx : (nnz_local > 0 ? (e1 > 0 ? e1 - 1 : 0) : 0);
      unsigned lc = 0;
      double av = 0.0;
      if (nnz_local > 0) {  // uniform over the workgroup
        lc = (unsigned)(cp[idx] - row0);
        av = vp[idx];
      }
      kc[sl][k] = (int32_t)(lc < last_row ? lc : last_row);  // a column outside the block stays inside LDS
      ka[sl][k] = in ? av : 0.0;
    }
    // rounds of this slot that any lane of the wave needs (uniform over the wave)
    int need = (e1 - e0 + CL - 1) / CL;
    if (valid && need < 1) need = 1;  // an empty row still gets its recurrence update
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const int other = __shfl_xor(need, o, 64);
      need = need > other ? need : other;
    }
    krounds[sl] = __builtin_amdgcn_readfirstlane(need);
  }

  // The steps [s0, s1) of the recurrence in the precision of `tag` (double or float), on iterates of that type in
  // the two buffers (their first halves for float); returns the buffer that holds the last iterate.
  float kaf[kRS][kRK];  // the entries once more in single precision
#pragma unroll
  for (int sl = 0; sl < kRS; ++sl)
#pragma unroll
    for (int k = 0; k < kRK; ++k) kaf[sl][k] = (float)ka[sl][k];
  // NE = columns per LDS read of a lane (its 8 columns are 8 / NE pieces, CL pieces apart): 2 in double precision
  // (16-byte reads, four pieces, as described at the top), 4 in single precision (16-byte reads again, two pieces).
  auto run_steps = [&](auto tag, auto ne_tag, int s0, int s1, void* bcur, void* bprev) __attribute__((always_inline)) -> void* {
  using T = decltype(tag);
  constexpr int NE = decltype(ne_tag)::value;
  constexpr int NP = 8 / NE;      // pieces per lane
  constexpr int RWv = BS / NE;    // pieces per operand row
  typedef T TV __attribute__((ext_vector_type(NE)));
  T* cur = static_cast<T*>(bcur);
  T* prev = static_cast<T*>(bprev);
  T* partt = reinterpret_cast<T*>(part);
  // this lane's t-th piece: segment (t + g) mod NP, position q inside the segment
  int pv[NP];
#pragma unroll
  for (int t = 0; t < NP; ++t) pv[t] = ((g + t) & (NP - 1)) * CL + q;
  for (int step = s0; step < s1; ++step) {
    const T alpha = (T)(step == 0 ? alpha_first : alpha_rest);
    const T beta = step == 0 ? (T)0 : (T)1;
    const T shiftt = (T)shift;
    const TV* __restrict__ curv = reinterpret_cast<const TV*>(cur);
    TV* prevv = reinterpret_cast<TV*>(prev);
#pragma unroll
    for (int sl = 0; sl < kRS; ++sl) {
      if (krounds[sl] == 0) continue;  // no lane of this wave has a chunk in this slot
      T acc[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] = (T)0;
#define SC_RES_ENTRY(K, Q)                                                                   \
  if constexpr (Q < CL) {                                                                    \
    const int cb = dpp_int<GroupBcast<CL, Q>::ctrl>(kc[sl][K]);                              \
    T av_;                                                                                   \
    if constexpr (sizeof(T) == 4) av_ = (T)kaf[sl][K]; else av_ = (T)ka[sl][K];              \
    const T ab = dpp_value<GroupBcast<CL, Q>::ctrl>(av_);                                    \
    const TV* zp = curv + cb * RWv;                                                          \
    TV z_[NP];                                                                               \
    _Pragma("unroll") for (int t = 0; t < NP; ++t) z_[t] = zp[pv[t]];                        \
    _Pragma("unroll") for (int t = 0; t < NP; ++t)                                           \
      _Pragma("unroll") for (int e = 0; e < NE; ++e) acc[NE * t + e] += ab * z_[t][e];       \
  }
#define SC_RES_ROUND(K)               \
  if (K < krounds[sl]) {              \
    SC_RES_ENTRY(K, 0)                \
    SC_RES_ENTRY(K, 1)                \
    SC_RES_ENTRY(K, 2)                \
    SC_RES_ENTRY(K, 3)                \
  }
      SC_RES_ROUND(0)
      SC_RES_ROUND(1)
      SC_RES_ROUND(2)
      SC_RES_ROUND(3)
      SC_RES_ROUND(4)
      SC_RES_ROUND(5)
      SC_RES_ROUND(6)
      SC_RES_ROUND(7)
#undef SC_RES_ROUND
#undef SC_RES_ENTRY
      const int r = crow[sl];
      if (r >= 0) {
        if (cidx[sl] == 0) {  // first chunk of its row: the recurrence with this chunk's sum, stored over u-
          const TV* own = curv + r * RWv;
          TV* out = prevv + r * RWv;
#pragma unroll
          for (int t = 0; t < NP; ++t) {
            const int at = pv[t];
            const TV o = own[at], pw = out[at];
            TV w;
#pragma unroll
            for (int e = 0; e < NE; ++e) w[e] = alpha * (acc[NE * t + e] - shiftt * o[e]) - beta * pw[e];
            out[at] = w;
          }
        } else {  // a further chunk: its sum waits in LDS for the row's owner
          TV* out = reinterpret_cast<TV*>(partt) + (size_t)(g + sl * G - r - 1) * RWv;
#pragma unroll
          for (int t = 0; t < NP; ++t) {
            TV w;
#pragma unroll
            for (int e = 0; e < NE; ++e) w[e] = acc[NE * t + e];
            out[pv[t]] = w;
          }
        }
      }
    }
    if (nx > 0) {  // uniform over the workgroup
      __syncthreads();
#pragma unroll
      for (int sl = 0; sl < kRS; ++sl) {
        const int r = crow[sl];
        if (r >= 0 && cidx[sl] == 0 && cnum[sl] > 1) {
          // the row's further chunks are chunks cst[r] + 1 ... of the block; chunk v parks at slot v - row(v) - 1
          const TV* src = reinterpret_cast<const TV*>(partt) + (size_t)(g + sl * G - r) * RWv;
          TV sum[NP];
#pragma unroll
          for (int t = 0; t < NP; ++t) sum[t] = src[pv[t]];
          for (int j = 2; j < cnum[sl]; ++j) {
            const TV* more = src + (size_t)(j - 1) * RWv;
#pragma unroll
            for (int t = 0; t < NP; ++t) sum[t] += more[pv[t]];
          }
          TV* out = prevv + r * RWv;
#pragma unroll
          for (int t = 0; t < NP; ++t) {
            const int at = pv[t];
            TV w = out[at];
            w += alpha * sum[t];
            out[at] = w;
          }
        }
      }
    }
    __syncthreads();  // every row of the new iterate is in place; nobody reads the old u- any more
    T* t = cur;
    cur = prev;
    prev = t;
  }
  return cur;
  };
  using Two = std::integral_constant<int, 2>;
  using Four = std::integral_constant<int, 4>;
  double* cur = bufa;
  if (d32 > 0) {
    // Single-precision steps first.  What their rounding adds to an iterate has components along every eigenvector,
    // and the steps that follow damp the unwanted ones like everything else below the interval's end: by the last six
    // double-precision steps they are back below what double precision leaves (measured on the first-step residuals:
    // no difference from six such steps on, a factor 5 at four).
    const bool in_b = run_steps(0.0f, Four{}, 0, d32, bufa, bufb) == static_cast<void*>(bufb);
    // both iterates from float to double, each inside its own buffer: everything is read before anything is written
    constexpr int PER = 10;  // nr * BS <= 10,240 (two double iterates fit the LDS)
    float ta[PER], tb[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int idx = tid + u * kRT;
      ta[u] = idx < nr * BS ? reinterpret_cast<const float*>(bufa)[idx] : 0.0f;
      tb[u] = idx < nr * BS ? reinterpret_cast<const float*>(bufb)[idx] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int idx = tid + u * kRT;
      if (idx < nr * BS) {
        bufa[idx] = (double)ta[u];
        bufb[idx] = (double)tb[u];
      }
    }
    __syncthreads();
    cur = static_cast<double*>(run_steps(0.0, Two{}, d32, d, in_b ? bufb : bufa, in_b ? bufa : bufb));
  } else {
    cur = static_cast<double*>(run_steps(0.0, Two{}, 0, d, bufa, bufb));
  }
  for (int idx = tid; idx < nr * BS; idx += kRT) {
    const int r = idx / BS, t = idx - r * BS;
    y[(int64_t)(row0 + r) * ldy + col0 + t] = cur[idx];
  }
}

// The sliced form, for diagonal blocks whose entries do not fit the registers: items of C = 16, 8 or 4 columns, one iterate u
// in LDS (up to 1,270, 2,540 or 5,080 rows), the other one, u-, in the registers of the lanes that own its rows (only its
// own row's recurrence reads it), and the entries read again in every step from a copy of the block made for that:
//   * The block's rows in slices of RS = 64 / LPR rows, LPR = C / 4 lanes per row, four columns a lane; rows padded to the
//     slice's longest with zero entries, in groups of four rounds: a lane gets a group's four column numbers with one 8-byte
//     load and its values with two 16-byte loads, kSliceAhead groups before they are multiplied.  Columns are stored in units of
//     32 bytes of the iterate (16 bits).
//   * A row's entries beyond kSliceLong are extra rows of their own (hubs of several hundred entries beside rows of thirty
//     would be what a step waits for): extra rows have slices like others, a lane parks its sum in LDS, and the row's owner
//     adds the sums in order once the step's reads are over.  Where LDS has no room for these sums (a block of 1,000 rows with
//     more than 300 entries each) all rows keep their entries: there they are long throughout.
//   * The slices are dealt to the sixteen waves one by one, extra rows first, each to the wave with the least to do (a step
//     lasts as long as its slowest wave); a wave's slices lie one behind the other in the copy, so that it reads its entries as
//     one stream over slice and step boundaries.
//   * A round is two 16-byte LDS reads of the operand row and four multiply-adds per lane; row sums never leave the lane.  An
//     item is bound by these reads and by the entry stream out of the L2 / Infinity Cache; 16 columns read the stream once
//     per step for all of a 16-column block, 4 columns make enough items where the blocks are few.
//   * When a wave is through its slices its new rows wait in registers (where u- was) for a barrier, then change places with
//     the old ones in LDS: what was u becomes u-.  (With both iterates in LDS, 8 columns and half as many rows, a lane per row
//     and a fixed pair of slices per wave, a filter step of 500,000 rows in 500 components took 58 us for the 60 % of the
//     rows that fitted and 53 us by the general product for the others; now 38 us for all of them.  100,000 rows in 100
//     components: 12.5 us in items of 4 columns, 28 us by the general product.)
constexpr int kSliceWaves = kRT / 64;
constexpr int kSliceOwn = 5;    // slices of rows a wave may own
constexpr int kSliceExtra = 5;  // slices of extra rows
constexpr int kSliceLong = 64;  // entries of a row before its extra rows
constexpr int kSliceAhead = 1;  // groups requested ahead of the one that is multiplied (2 and 3: 2 to 5 % slower, spills)

__host__ __device__ inline int sliced_slices(int rows, int cols) { return (rows + 256 / cols - 1) / (256 / cols); }
// places for slices that a wave has: its share, and one more up to three (more of them cost registers)
__host__ __device__ inline int sliced_places(int slices, int most) {
  const int share = (slices + kSliceWaves - 1) / kSliceWaves;
  return share == 0 || share >= 3 || share >= most ? share : share + 1;
}
__host__ __device__ inline int sliced_slots(int rows, int cols) { return sliced_places(sliced_slices(rows, cols), kSliceOwn); }
__host__ __device__ inline int sliced_extra_slots(int extra, int cols) {
  return sliced_places(sliced_slices(extra, cols), kSliceExtra);
}

template <int C, int MAXS>
__device__ __forceinline__ void resident_item_sliced(const uint16_t* __restrict__ scol, const double* __restrict__ sval,
                                                     const int64_t* __restrict__ slice_base,
                                                     const int32_t* __restrict__ slice_len,
                                                     const double* __restrict__ x, double* __restrict__ y, int64_t ldy, int b,
                                                     int d, double alpha_first, double alpha_rest, double shift,
                                                     const int32_t* __restrict__ slice_first,
                                                     const int32_t* __restrict__ row_extra, int row0, int nr, int col0,
                                                     int slice0, int nx, unsigned char* smem, uint64_t rnd_key,
                                                     int use_rnd) {
  constexpr int LPR = C / 4, RS = 64 / LPR, NB = kSliceAhead + 1, MAXT = kSliceOwn + kSliceExtra;
  double* u = reinterpret_cast<double*>(smem);
  const int parked = nr * C * 8;  // byte offset of the extra rows' sums
  int32_t* groups = reinterpret_cast<int32_t*>(u + (size_t)(nr + nx) * C);  // [wave][MAXT]
  int32_t* places = groups + kSliceWaves * MAXT;                            // [wave][MAXT]: the slices' first rows
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int j = lane / LPR, h = lane % LPR;
  for (int idx = tid; idx < nr * C; idx += kRT) {
    const int r = idx / C, t = idx - r * C;
    const int64_t gi = (int64_t)(row0 + r) * b + col0 + t;
    u[idx] = use_rnd ? random_entry(rnd_key, gi) : x[gi];
  }
  const int xslots = sliced_extra_slots(nx, C), slots = xslots + sliced_slots(nr, C), first = slice0 + wave * slots;
  // the wave's groups, slices of extra rows and slices of rows (in this order; a place without a slice has no groups)
  int total = 0, xown = 0, own = 0;
  {
    const int g = lane < slots ? (slice_len[first + lane] + 3) / 4 : 0;
    const unsigned long long some = __ballot(g > 0);
    if (g > 0) {
      const int at = wave * MAXT + __popcll(some & ((1ull << lane) - 1ull));
      groups[at] = g;
      places[at] = slice_first[first + lane];
    }
    xown = __popcll(some & ((1ull << xslots) - 1ull));
    own = __popcll(some) - xown;
    int sum = g;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    total = __builtin_amdgcn_readfirstlane(sum);
  }
  __syncthreads();
  if (total == 0) {  // a wave without rows keeps the barriers company
    for (int step = 0; step < d; ++step) {
      __syncthreads();
      __syncthreads();
    }
  } else {
    // a lane's 32 bytes of a row are two pieces; lanes of even and odd rows read them in opposite order, and a row's entries
    // are ordered so that the rows of a 16-lane pass fall on different banks (slice_fill_kernel)
    const int swap = (j & 1) * 16;
    char* ub = reinterpret_cast<char*>(u);
    const int part = h * 32 + swap;
    const int64_t base = slice_base[first];
    const uint16_t* cp0 = scol + base + 4 * j;
    const double* vp0 = sval + base + 2 * j;
    struct Group {
      uint2 c;
      double2 v0, v1;
    };
    Group buf[NB];
    int ahead = 0;  // the next group to request
    auto request = [&](Group& g) __attribute__((always_inline)) {
      const int64_t off = (int64_t)ahead * (4 * RS);
      g.c = *reinterpret_cast<const uint2*>(cp0 + off);
      g.v0 = *reinterpret_cast<const double2*>(vp0 + off);
      g.v1 = *reinterpret_cast<const double2*>(vp0 + off + 2 * RS);
      ahead = ahead + 1 < total ? ahead + 1 : 0;
    };
    double keep[MAXS][4];  // the rows' u-; a queue: slot s is at the front when its turn comes
    int extra[MAXS];       // the rows' extra rows: first << 16 | number
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
      const int r = s < own ? places[wave * MAXT + xown + s] + j : nr;
      extra[s] = nx > 0 && r < nr ? row_extra[row0 + r] : 0;
    }
    double acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = 0.0;
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t) keep[s][t] = 0.0;
    auto round = [&](uint32_t c, double a) __attribute__((always_inline)) {
      const int at = (int)(c * 32u) + part;
      const double2 z0 = *reinterpret_cast<const double2*>(ub + at);
      const double2 z1 = *reinterpret_cast<const double2*>(ub + (at ^ 16));
      acc[0] += a * z0.x;
      acc[1] += a * z0.y;
      acc[2] += a * z1.x;
      acc[3] += a * z1.y;
    };
    auto push = [&](const double (&last)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s + 1 < MAXS; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t) keep[s][t] = keep[s + 1][t];
#pragma unroll
      for (int t = 0; t < 4; ++t) keep[MAXS - 1][t] = last[t];
    };
    int step = 0, slot = 0;
    int left = __builtin_amdgcn_readfirstlane(groups[wave * MAXT]);
#pragma unroll
    for (int q = 0; q < kSliceAhead; ++q) request(buf[q]);
    for (bool more = true; more;) {
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        request(buf[(q + kSliceAhead) % NB]);
        round(buf[q].c.x & 0xffffu, buf[q].v0.x);
        round(buf[q].c.x >> 16, buf[q].v0.y);
        round(buf[q].c.y & 0xffffu, buf[q].v1.x);
        round(buf[q].c.y >> 16, buf[q].v1.y);
        if (--left > 0) continue;  // uniform over the wave, as all that follows
        if (slot < xown) {  // a slice of extra rows is done
          const int e = places[wave * MAXT + slot] + j;
          if (e < nx) {
            const int at = parked + e * (C * 8) + part;
            *reinterpret_cast<double2*>(ub + at) = make_double2(acc[0], acc[1]);
            *reinterpret_cast<double2*>(ub + (at ^ 16)) = make_double2(acc[2], acc[3]);
          }
        } else {  // a slice of rows is done: the new iterate without the extra rows' sums
          const int r = places[wave * MAXT + slot] + j;
          const int at = (r < nr ? r : nr - 1) * (C * 8) + part;
          const double2 o0 = *reinterpret_cast<const double2*>(ub + at);
          const double2 o1 = *reinterpret_cast<const double2*>(ub + (at ^ 16));
          const double alpha = step == 0 ? alpha_first : alpha_rest, beta = step == 0 ? 0.0 : 1.0;
          const double next[4] = {alpha * (acc[0] - shift * o0.x) - beta * keep[0][0],
                                  alpha * (acc[1] - shift * o0.y) - beta * keep[0][1],
                                  alpha * (acc[2] - shift * o1.x) - beta * keep[0][2],
                                  alpha * (acc[3] - shift * o1.y) - beta * keep[0][3]};
          push(next);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = 0.0;
        ++slot;
        if (slot == xown + own) {  // the step is done
          for (int s = own; s < MAXS; ++s) {
            const double front[4] = {keep[0][0], keep[0][1], keep[0][2], keep[0][3]};
            push(front);
          }
          __syncthreads();  // nobody reads this step's operand any more, and the extra rows' sums are there
          const double alpha = step == 0 ? alpha_first : alpha_rest;
#pragma unroll
          for (int s = 0; s < MAXS; ++s) {
            const int r = s < own ? places[wave * MAXT + xown + s] + j : nr;
            if (r < nr) {
              for (int q = 0; q < (extra[s] & 0xffff); ++q) {
                const int from = parked + ((extra[s] >> 16) + q) * (C * 8) + part;
                const double2 e0 = *reinterpret_cast<const double2*>(ub + from);
                const double2 e1 = *reinterpret_cast<const double2*>(ub + (from ^ 16));
                keep[s][0] += alpha * e0.x;
                keep[s][1] += alpha * e0.y;
                keep[s][2] += alpha * e1.x;
                keep[s][3] += alpha * e1.y;
              }
              const int at = r * (C * 8) + part;
              double2* p0 = reinterpret_cast<double2*>(ub + at);
              double2* p1 = reinterpret_cast<double2*>(ub + (at ^ 16));
              const double2 o0 = *p0, o1 = *p1;
              *p0 = make_double2(keep[s][0], keep[s][1]);
              *p1 = make_double2(keep[s][2], keep[s][3]);
              keep[s][0] = o0.x;
              keep[s][1] = o0.y;
              keep[s][2] = o1.x;
              keep[s][3] = o1.y;
            }
          }
          __syncthreads();  // every row of the new iterate is in place
          slot = 0;
          if (++step == d) {
            more = false;
            break;
          }
        }
        left = __builtin_amdgcn_readfirstlane(groups[wave * MAXT + slot]);
      }
    }
  }
  for (int idx = tid; idx < nr * C; idx += kRT) {
    const int r = idx / C, t = idx - r * C;
    y[(int64_t)(row0 + r) * ldy + col0 + t] = u[idx];
  }
}

__global__ __launch_bounds__(kRT) void cheb_resident_kernel(const int64_t* __restrict__ rowptr,
                                                            const int32_t* __restrict__ col,
                                                            const double* __restrict__ val,
                                                            const double* __restrict__ x, double* __restrict__ y,
                                                            int64_t ldy, int b, int d, double alpha_first,
                                                            double alpha_rest, double shift,
                                                            const int32_t* __restrict__ items,
                                                            const uint16_t* __restrict__ scol,
                                                            const double* __restrict__ sval,
                                                            const int64_t* __restrict__ slice_base,
                                                            const int32_t* __restrict__ slice_len,
                                                            const int32_t* __restrict__ slice_first,
                                                            const int32_t* __restrict__ row_extra, int d32,
                                                            uint64_t rnd_key, int use_rnd, int nitems, int copies,
                                                            uint64_t rnd_key2) {
  extern __shared__ __align__(16) unsigned char smem[];
  int item = (int)blockIdx.x;
  if (copies == 2) {
    // an item of the one block and of the other on one XCD, one after the other: the sliced form's entries meet in its L2
    item = (int)(blockIdx.x / 16 * 8 + blockIdx.x % 8);
    if (item >= nitems) return;  // uniform
    if (blockIdx.x / 8 % 2) {
      y += b;
      rnd_key = rnd_key2;
    }
  }
  const int32_t* it = items + kItemInts * (int64_t)item;
  const int row0 = it[0], nr = it[1], col0 = it[2], cl = it[3] & 15, nx = it[3] >> 4;  // uniform over the workgroup
  if (cl == 4)
    resident_item<4>(rowptr, col, val, x, y, ldy, b, d, alpha_first, alpha_rest, shift, row0, nr, col0, nx, smem, d32, rnd_key, use_rnd);
  else if (cl == 2)
    resident_item<2>(rowptr, col, val, x, y, ldy, b, d, alpha_first, alpha_rest, shift, row0, nr, col0, nx, smem, d32, rnd_key, use_rnd);
  else {  // sliced form: its first slot takes the chunk count's place, the last word is the block's number of extra rows
#define SC_SLICED(CV, MAXSV)                                                                                             \
  resident_item_sliced<CV, MAXSV>(scol, sval, slice_base, slice_len, x, y, ldy, b, d, alpha_first, alpha_rest, shift,    \
                                  slice_first, row_extra, row0, nr, col0, nx, it[4], smem, rnd_key, use_rnd)
    const int cols = cl == kShape16 ? 16 : cl == kShape8 ? 8 : 4;
    const int slots = sliced_slots(nr, cols);
#define SC_SLICED_SLOTS(CV)                                                                                        \
  do {                                                                                                             \
    if (slots <= 3) SC_SLICED(CV, 3); else if (slots == 4) SC_SLICED(CV, 4); else SC_SLICED(CV, kSliceOwn);        \
  } while (0)
    if (cl == kShape16) SC_SLICED_SLOTS(16);
    else if (cl == kShape8) SC_SLICED_SLOTS(8);
    else if (cl == kShape4) SC_SLICED_SLOTS(4);
#undef SC_SLICED_SLOTS
#undef SC_SLICED
  }
}

// ---- sliced copy of diagonal blocks ------------------------------------------------------------------------------------
// What a slice of the copy holds: `rows` consecutive rows of the matrix from `first` on (none: a place without a slice), or as
// many extra rows of the list, of a block of blk_rows rows from blk0 on whose extra rows begin at extra0 of the list (extra
// = 1), for items of `cols` columns.  A row's first `piece` entries are its own, `piece` more of them go to each extra row.
struct SliceDesc {
  int32_t first, rows, blk0, blk_rows, cols, extra, extra0, piece;
};

// Entries [*from, *from + return value) of row `*row` of the matrix: what place j of the slice holds.
__device__ __forceinline__ int slice_row(const SliceDesc& sd, int j, const int64_t* __restrict__ rowptr,
                                         const int32_t* __restrict__ list, const int32_t* __restrict__ row_extra,
                                         int64_t* from) {
  if (j >= sd.rows) {
    *from = 0;
    return 0;
  }
  const int64_t r = sd.extra ? (int64_t)list[sd.first + j] : (int64_t)sd.first + j;
  // the extra row's number within its row
  const int chunk = sd.extra ? sd.first + j - sd.extra0 - (row_extra[r] >> 16) + 1 : 0;
  const int64_t e0 = rowptr[r];
  const int len = (int)(rowptr[r + 1] - e0) - chunk * sd.piece;
  *from = e0 + (int64_t)chunk * sd.piece;
  return len < sd.piece ? len : sd.piece;
}

// The extra rows of the sliced blocks, blocks[kSliceBlockInts t ..] = (first row, rows, place of its first extra row in the
// list, extra rows, columns, first slot, piece): list[.] = the row each belongs to, row_extra[r] = place of row r's first one
// within the block << 16 | their number.  A wave per block.
__global__ __launch_bounds__(256) void slice_extra_kernel(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ blocks,
                                                          int nblocks, int32_t* __restrict__ list,
                                                          int32_t* __restrict__ row_extra) {
  const int t = (int)(((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= nblocks) return;
  const int32_t* blk = blocks + (int64_t)kSliceBlockInts * t;
  const int64_t row0 = blk[0];
  const int rows = blk[1], base = blk[2], piece = blk[6];
  int at = 0;
  for (int r0 = 0; r0 < rows; r0 += 64) {
    const int r = r0 + lane;
    const int len = r < rows ? (int)(rowptr[row0 + r + 1] - rowptr[row0 + r]) : 0;
    const int x = len > piece ? (len - 1) / piece : 0;
    int incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    const int mine = at + incl - x;
    if (r < rows) row_extra[row0 + r] = mine << 16 | x;
    for (int q = 0; q < x; ++q) list[base + mine + q] = (int32_t)(row0 + r);
    at += __shfl(incl, 63, 64);
  }
}

// Deals a sliced block's slices to the waves: a workgroup per block, blocks[kSliceBlockInts t ..].  For every slot (wave, place)
// of the block, from slot0 on: desc = the slice in it (or none), slice_len = its longest row (at least 1), slice_first = its
// first row within the block / its first extra row, slice_entries = what it takes in the copy, whole groups of four rounds.
// slice_entries[nslots] = 0: the scan's last output is the copy's size.
__global__ __launch_bounds__(256) void slice_layout_kernel(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ blocks,
                                                           const int32_t* __restrict__ list,
                                                           const int32_t* __restrict__ row_extra, int nslots,
                                                           SliceDesc* __restrict__ desc, int32_t* __restrict__ slice_len,
                                                           int32_t* __restrict__ slice_first,
                                                           int64_t* __restrict__ slice_entries) {
  constexpr int MAXN = (kSliceOwn + kSliceExtra) * kSliceWaves;
  __shared__ int length[MAXN], slot_of[MAXN];
  const int32_t* blk = blocks + (int64_t)kSliceBlockInts * blockIdx.x;
  const int row0 = blk[0], nr = blk[1], extra0 = blk[2], nx = blk[3], cols = blk[4], slot0 = blk[5], piece = blk[6];
  const int rs = 256 / cols, xs = sliced_slices(nx, cols), rsl = sliced_slices(nr, cols);
  const int xslots = sliced_extra_slots(nx, cols), rslots = sliced_slots(nr, cols), slots = xslots + rslots;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (blockIdx.x == 0 && threadIdx.x == 0) slice_entries[nslots] = 0;
  auto describe = [&](int q) __attribute__((always_inline)) -> SliceDesc {  // slice q: the extra rows' first
    const bool x = q < xs;
    const int at = rs * (x ? q : q - xs), left = (x ? nx : nr) - at;
    return SliceDesc{(x ? extra0 : row0) + at, left < rs ? left : rs, row0, nr, cols, x ? 1 : 0, extra0, piece};
  };
  for (int q = wave; q < xs + rsl; q += 4) {
    const SliceDesc sd = describe(q);
    int64_t from;
    int len = slice_row(sd, lane, rowptr, list, row_extra, &from);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const int other = __shfl_xor(len, o, 64);
      len = len > other ? len : other;
    }
    if (lane == 0) length[q] = len < 1 ? 1 : len;
  }
  for (int q = threadIdx.x; q < slots * kSliceWaves; q += 256) {  // no slice, unless one is dealt
    desc[slot0 + q] = SliceDesc{0, 0, row0, nr, cols, 0, extra0, piece};
    slice_len[slot0 + q] = 0;
    slice_first[slot0 + q] = 0;
    slice_entries[slot0 + q] = 0;
  }
  __syncthreads();
  if (wave == 0) {
    int busy = 0, taken = 0;  // of wave `lane`, lane < 16: rounds, slices of the kind that is being dealt
    for (int q = 0; q < xs + rsl; ++q) {
      if (q == xs) taken = 0;
      const int len = (length[q] + 3) / 4 * 4;
      int key = lane < kSliceWaves && taken < (q < xs ? xslots : rslots) ? busy << 4 | lane : INT32_MAX;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        const int other = __shfl_xor(key, o, 16);
        key = other < key ? other : key;
      }
      if (lane == (key & 15)) {
        slot_of[q] = lane * slots + (q < xs ? 0 : xslots) + taken;
        busy += len;
        ++taken;
      }
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < xs + rsl; q += 256) {
    const int at = slot0 + slot_of[q];
    desc[at] = describe(q);
    slice_len[at] = length[q];
    slice_first[at] = rs * (q < xs ? q : q - xs);
    slice_entries[at] = (int64_t)rs * ((length[q] + 3) / 4 * 4);
  }
}

// Fills the copy; a workgroup per slice, half a wave per row, RS = 256 / cols rows.  Round k of row j sits in group k / 4: column number
// at group * 4 RS + 4 j + k % 4, value at group * 4 RS + (k % 4) / 2 * 2 RS + 2 j + k % 2.  Column numbers count the operand's
// 32-byte pieces inside the block; rounds past a row's end, and rows past the block's end, have value 0.
//
// The order of a row's entries is chosen for the LDS banks.  In a round the 16 lanes of a pass read 16 bytes each of
// 256 / (8 cols) = NC different operand rows at a time without a conflict if these rows differ mod NC (cols 4, 8, 16: NC 8, 4,
// 2), half of the pass's rows one piece and half the other (rows j of the same parity).  Row j therefore wants in round k an
// entry whose column is (j / 2 + k) mod NC; the r-th entry of a class goes into the r-th such round.  Entries for which a
// row has too few such rounds take, in order, the rounds that other classes leave free.  The order depends on the matrix
// alone, so the sums stay reproducible.
__global__ __launch_bounds__(256) void slice_fill_kernel(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                                         const double* __restrict__ val, const SliceDesc* __restrict__ desc,
                                                         const int32_t* __restrict__ list,
                                                         const int32_t* __restrict__ row_extra, const int64_t* __restrict__ slice_base,
                                                         const int64_t* __restrict__ slice_entries,
                                                         uint16_t* __restrict__ scol, double* __restrict__ sval) {
  const int lane = threadIdx.x & 31, half = (threadIdx.x & 32);
  const int64_t sidx = blockIdx.x;
  const SliceDesc sd = desc[sidx];
  const int rs = 256 / sd.cols, lpr = sd.cols / 4, lognc = sd.cols == 16 ? 1 : sd.cols == 8 ? 2 : 3, nc = 1 << lognc;
  if (sd.rows == 0) return;
  const int rounds = (int)(slice_entries[sidx] / rs);
  const int64_t base = slice_base[sidx];
  const unsigned last = (unsigned)(sd.blk_rows - 1);
  for (int j = threadIdx.x >> 5; j < rs; j += 8) {  // uniform over the wave: rs is a multiple of 16
  int64_t e0;
  const int len = slice_row(sd, j, rowptr, list, row_extra, &e0);
  const int turn = j >> 1;
  auto local = [&](int e) __attribute__((always_inline)) -> unsigned {
    const unsigned lc = (unsigned)(col[e0 + e] - sd.blk0);
    return lc < last ? lc : last;  // a column outside the block (there is none in a diagonal block) stays inside LDS
  };
  auto first_round = [&](int cls) __attribute__((always_inline)) -> int { return (cls - turn) & (nc - 1); };
  auto rounds_of = [&](int cls) __attribute__((always_inline)) -> int {
    const int f = first_round(cls);
    return f < len ? (len - f + nc - 1) >> lognc : 0;
  };
  auto put = [&](int k, unsigned lc, double av) __attribute__((always_inline)) {
    const int64_t at = base + (int64_t)(k >> 2) * (4 * rs);
    scol[at + 4 * j + (k & 3)] = (uint16_t)(lc * (unsigned)lpr);
    sval[at + ((k >> 1) & 1) * 2 * rs + 2 * j + (k & 1)] = av;
  };
  const int longest = max(len, __shfl_xor(len, 32, 64));  // of the wave's two rows: they go through the loops together
  // entries of every class, and how many before them have no round of their own / how many rounds are free before
  int count[8], over[8], gap[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) count[c] = 0;
  for (int b0 = 0; b0 < longest; b0 += 32) {
    const bool in = b0 + lane < len;
    const int cls = in ? (int)(local(b0 + lane) & (unsigned)(nc - 1)) : -1;
#pragma unroll
    for (int c = 0; c < 8; ++c) count[c] += __popc((unsigned)(__ballot(cls == c) >> half));
  }
  int so = 0, sg = 0;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int m = c < nc ? rounds_of(c) : 0;
    over[c] = so;
    gap[c] = sg;
    so += count[c] > m ? count[c] - m : 0;
    sg += m > count[c] ? m - count[c] : 0;
  }
  int seen[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) seen[c] = 0;
  for (int b0 = 0; b0 < longest; b0 += 32) {
    const bool in = b0 + lane < len;
    const unsigned lc = in ? local(b0 + lane) : 0u;
    const int cls = in ? (int)(lc & (unsigned)(nc - 1)) : -1;
    int rank = 0, before = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const unsigned m = (unsigned)(__ballot(cls == c) >> half);
      if (cls == c) {
        rank = seen[c] + __popc(m & ((1u << lane) - 1u));
        before = over[c];
      }
      seen[c] += __popc(m);
    }
    if (in) {
      const int own = rounds_of(cls);
      int k;
      if (rank < own) {
        k = first_round(cls) + (rank << lognc);
      } else {  // the (before + rank - own)-th free round
        int want = before + rank - own;
        k = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int m = c < nc ? rounds_of(c) : 0, free_here = m > count[c] ? m - count[c] : 0;
          const int at = want - gap[c];
          if (at >= 0 && at < free_here) k = first_round(c) + ((count[c] + at) << lognc);
        }
      }
      put(k, lc, val[e0 + b0 + lane]);
    }
  }
  for (int k = len + lane; k < rounds; k += 32) {  // padding: a row of the wanted class
    const unsigned want = (unsigned)((turn + k) & (nc - 1));
    put(k, want <= last ? want : 0u, 0.0);
  }
  }
}

// counts of diagonal block t, from extra[kBlockCounts t] on: chunks beyond the first, summed over its rows, for chunks of 32, 16
// and kSliceLong entries; its entries; what its rows' first kSliceLong entries take in slices of 16 rows, padding included (both
// INT32_MAX if more).  W waves per block: few blocks are large ones (one wave for each of 20 blocks of 5,000 rows took 35 us).
template <int W>
__global__ __launch_bounds__(W > 1 ? 64 * W : 256) void block_counts_kernel(const int64_t* __restrict__ rowptr,
                                                                          const int32_t* __restrict__ starts, int nblk,
                                                                          int64_t n, int32_t* __restrict__ extra) {
  __shared__ int64_t sums[W][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = W > 1 ? (int)blockIdx.x : (int)blockIdx.x * 4 + wave;
  if (t >= nblk) return;  // uniform over the workgroup where it meets below
  const int64_t r0 = starts[t], r1 = t + 1 < nblk ? (int64_t)starts[t + 1] : n;
  int64_t v[4] = {0, 0, 0, 0};  // chunks of 32, of 16, of kSliceLong; padded entries
  for (int64_t first = r0 + (W > 1 ? 64 * wave : 0); first < r1; first += 64 * W) {  // uniform over the wave
    const int64_t r = first + lane;
    const int len = r < r1 ? (int)(rowptr[r + 1] - rowptr[r]) : 0;
    int longest = len < kSliceLong ? len : kSliceLong;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
      const int other = __shfl_xor(longest, o, 16);
      longest = other > longest ? other : longest;
    }
    if ((lane & 15) == 0) v[3] += 16 * ((longest + 3) / 4 * 4);
    if (len > 32) v[0] += (len + 31) / 32 - 1;
    if (len > 16) v[1] += (len + 15) / 16 - 1;
    if (len > kSliceLong) v[2] += (len + kSliceLong - 1) / kSliceLong - 1;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
  if constexpr (W > 1) {
    if (lane == 0)
#pragma unroll
      for (int q = 0; q < 4; ++q) sums[wave][q] = v[q];
    __syncthreads();
    if (threadIdx.x) return;
    for (int w = 1; w < W; ++w)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += sums[w][q];
  } else if (lane) {
    return;
  }
  const int64_t entries = rowptr[r1] - rowptr[r0];
  auto put = [&](int q, int64_t c) { extra[kBlockCounts * (int64_t)t + q] = c < INT32_MAX ? (int32_t)c : INT32_MAX; };
  put(0, v[0]);
  put(1, v[1]);
  put(2, v[2]);
  put(3, entries);
  put(4, v[3]);
}

// ---- diagonal blocks of a CSR matrix -------------------------------------------------------------------------------
// reach[i] = max(i, largest column of row i)
__global__ __launch_bounds__(256) void row_reach_kernel(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                                        int64_t n, int32_t* __restrict__ reach) {
  const int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;
  const int lane = threadIdx.x & 15;
  if (row >= n) return;
  const int64_t e1 = rowptr[row + 1];
  int32_t m = (int32_t)row;
  for (int64_t e = rowptr[row] + lane; e < e1; e += 16) m = max(m, col[e]);
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 16));
  if (lane == 0) reach[row] = m;
}

// flag[p] = 1 if row p starts a diagonal block: no row before it reaches column p or beyond
__global__ __launch_bounds__(256) void block_start_kernel(const int32_t* __restrict__ reach_prefix_max, int64_t n,
                                                          unsigned char* __restrict__ flag) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= n) return;
  flag[p] = (p == 0 || (int64_t)reach_prefix_max[p - 1] < p) ? 1 : 0;
}

struct MaxOp {
  __host__ __device__ int32_t operator()(const int32_t& a, const int32_t& b) const { return a > b ? a : b; }
};

size_t up256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

size_t resident_item_lds_bytes(int nrows, int cl, int extra) { return resident_lds_bytes(nrows, cl, extra); }

int resident_max_chunks(int cl) { return kRS * (kRT / cl); }

int sliced_piece() { return kSliceLong; }

int sliced_shape(int cols) { return cols == 16 ? kShape16 : cols == 8 ? kShape8 : kShape4; }

size_t resident_sliced_lds_bytes(int nrows, int extra, int cols) {
  // more slices than the waves own, or more extra rows than their numbers hold: no item
  if (nrows > 65535 || extra > 32767 || sliced_slices(nrows, cols) > kSliceOwn * kSliceWaves ||
      sliced_slices(extra, cols) > kSliceExtra * kSliceWaves)
    return ~(size_t)0;
  return (size_t)(nrows + extra) * cols * sizeof(double) +
         (size_t)2 * kSliceWaves * (kSliceOwn + kSliceExtra) * sizeof(int32_t);
}

int sliced_block_slots(int nrows, int extra, int cols) {
  return (sliced_slots(nrows, cols) + sliced_extra_slots(extra, cols)) * kSliceWaves;
}

size_t sliced_desc_bytes(int nslots) { return (size_t)nslots * sizeof(SliceDesc); }

size_t sliced_scan_workspace(int nslices) {
  size_t t = 0;
  (void)rocprim::exclusive_scan(nullptr, t, (int64_t*)nullptr, (int64_t*)nullptr, (int64_t)0, (size_t)nslices + 1,
                                rocprim::plus<int64_t>());
  return up256(t) + 256;
}

hipError_t sliced_extra_rows(const int64_t* rowptr, const int32_t* blocks, int nblocks, int32_t* list, int32_t* row_extra,
                             hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(slice_extra_kernel, dim3((unsigned)(((int64_t)nblocks * 64 + 255) / 256)), dim3(256), 0, st, rowptr, blocks,
                     nblocks, list, row_extra);
  return hipGetLastError();
}

hipError_t sliced_copy_layout(const int64_t* rowptr, const int32_t* blocks, int nblocks, const int32_t* list,
                              const int32_t* row_extra, int nslots, void* desc, int32_t* slice_len, int32_t* slice_first,
                              int64_t* slice_entries, int64_t* slice_base, void* work, size_t work_bytes, hipStream_t st) {
  if (nslots <= 0 || nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(slice_layout_kernel, dim3((unsigned)nblocks), dim3(256), 0, st, rowptr, blocks, list, row_extra, nslots,
                     static_cast<SliceDesc*>(desc), slice_len, slice_first, slice_entries);
  const hipError_t e = rocprim::exclusive_scan(work, work_bytes, slice_entries, slice_base, (int64_t)0, (size_t)nslots + 1,
                                               rocprim::plus<int64_t>(), st);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

hipError_t sliced_copy_fill(const int64_t* rowptr, const int32_t* col, const double* val, const void* desc,
                            const int32_t* list, const int32_t* row_extra, int nslots, const int64_t* slice_base,
                            const int64_t* slice_entries, uint16_t* scol, double* sval, hipStream_t st) {
  if (nslots <= 0) return hipSuccess;
  hipLaunchKernelGGL(slice_fill_kernel, dim3((unsigned)nslots), dim3(256), 0, st, rowptr, col, val,
                     static_cast<const SliceDesc*>(desc), list, row_extra, slice_base, slice_entries, scol, sval);
  return hipGetLastError();
}

hipError_t launch_block_extra_chunks(const int64_t* rowptr, const int32_t* starts, int nblk, int64_t n, int32_t* extra,
                                     hipStream_t st) {
  if (nblk <= 0) return hipSuccess;
  if (nblk <= 1024)
    hipLaunchKernelGGL(block_counts_kernel<16>, dim3((unsigned)nblk), dim3(1024), 0, st, rowptr, starts, nblk, n, extra);
  else
    hipLaunchKernelGGL(block_counts_kernel<1>, dim3((unsigned)((nblk + 3) / 4)), dim3(256), 0, st, rowptr, starts, nblk, n, extra);
  return hipGetLastError();
}

size_t diagonal_blocks_workspace(int64_t n) {
  size_t t1 = 0, t2 = 0;
  (void)rocprim::inclusive_scan(nullptr, t1, (int32_t*)nullptr, (int32_t*)nullptr, (size_t)n, MaxOp());
  (void)rocprim::select(nullptr, t2, rocprim::counting_iterator<int32_t>(0), (unsigned char*)nullptr, (int32_t*)nullptr,
                        (int32_t*)nullptr, (size_t)n);
  return up256((size_t)n * 4) + up256((size_t)n) + up256(t1 > t2 ? t1 : t2) + 256;
}

hipError_t diagonal_blocks(const int64_t* rowptr, const int32_t* col, int64_t n, void* work, size_t work_bytes,
                           int32_t* starts, int32_t* count, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (work_bytes < diagonal_blocks_workspace(n)) return hipErrorInvalidValue;
  char* w = static_cast<char*>(work);
  int32_t* reach = reinterpret_cast<int32_t*>(w);
  unsigned char* flag = reinterpret_cast<unsigned char*>(w + up256((size_t)n * 4));
  void* temp = w + up256((size_t)n * 4) + up256((size_t)n);
  size_t temp_bytes = work_bytes - up256((size_t)n * 4) - up256((size_t)n);
  hipLaunchKernelGGL(row_reach_kernel, dim3((unsigned)((n * 16 + 255) / 256)), dim3(256), 0, st, rowptr, col, n, reach);
  hipError_t e = rocprim::inclusive_scan(temp, temp_bytes, reach, reach, (size_t)n, MaxOp(), st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(block_start_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, reach, n, flag);
  e = rocprim::select(temp, temp_bytes, rocprim::counting_iterator<int32_t>(0), flag, starts, count, (size_t)n, st);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

hipError_t launch_cheb_resident(const int64_t* rowptr, const int32_t* col, const double* val, const double* x, double* y,
                                int64_t ldy, int b, int d, double alpha_first, double alpha_rest, double shift, const int32_t* items,
                                int nitems, size_t lds_bytes, const uint16_t* scol, const double* sval,
                                const int64_t* slice_base, const int32_t* slice_len, const int32_t* slice_first,
                                const int32_t* row_extra, hipStream_t st, int d32, uint64_t rnd_key, int use_rnd,
                                int copies, uint64_t rnd_key2) {
  if (nitems <= 0 || d <= 0) return hipSuccess;
  if (copies < 1 || copies > 2 || (copies == 2 && (!use_rnd || ldy < 2 * b))) return hipErrorInvalidValue;
  if (d32 < 0 || d32 >= d) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&cheb_resident_kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  const unsigned grid = copies == 2 ? (unsigned)((nitems + 7) / 8 * 16) : (unsigned)nitems;
  hipLaunchKernelGGL(cheb_resident_kernel, dim3(grid), dim3(kRT), lds_bytes, st, rowptr, col, val, x, y, ldy, b, d,
                     alpha_first, alpha_rest, shift, items, scol, sval, slice_base, slice_len, slice_first, row_extra, d32, rnd_key, use_rnd, nitems,
                     copies, rnd_key2);
  return hipGetLastError();
}

}  // namespace sceig
