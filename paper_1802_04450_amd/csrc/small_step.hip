// One block step of a small solve as one launch (see launch_small_step in kernels.h).
#include "kernels.h"
#include "wave_chol.h"

namespace sceig {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
#define MFMA_F64(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64((a), (b), (c), 0, 0, 0)

constexpr int kB = kSmallStepBlock;
constexpr int kStepThreads = 512;  // the factorization's registers allow two waves a SIMD
constexpr int kStepWaves = kStepThreads / 64;
constexpr int kWP = kB + 1;  // row pitch of the block and of the coefficients in LDS

// What one workgroup tells the others goes through agent-scope atomics, which pass by the caches that are not shared.
__device__ __forceinline__ void put_shared(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_shared(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All workgroups meet.  Every wave waits until its own stores have arrived where the others read them, then the workgroup
// counts itself in and looks until all have.  The look is bounded: a workgroup that finds the others missing for `polls`
// looks raises sync[kSyncAbort] for good, and whoever sees that leaves the kernel, too.  False: leave.
__device__ __forceinline__ bool meet(uint32_t* sync, uint32_t target, uint32_t polls, int* ok) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(sync + kSyncCount, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int there = 0;
    for (uint32_t i = 0; i < polls && !there; ++i) {
      const uint32_t seen = __hip_atomic_load(sync + kSyncCount, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t stop = __hip_atomic_load(sync + kSyncAbort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (stop) break;
      there = (int32_t)(seen - target) >= 0;
    }
    if (!there) __hip_atomic_store(sync + kSyncAbort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *ok = there;
  }
  __syncthreads();
  return *ok != 0;
}

struct StepLds {
  double *q, *w, *h, *red, *gram, *rinv, *r;
  int* ok;
};
constexpr int kRinvDoubles = kB * kPartialPad;
__host__ __device__ inline int step_pitch(int j) { return (j + 15) / 16 * 16 + 1; }  // odd: columns and rows both without bank conflicts
inline size_t step_lds_bytes(int j, int rows) {
  return ((size_t)rows * (step_pitch(j) + kWP) + (size_t)step_pitch(j) * kWP + kStepThreads + kB * kB + 2 * kRinvDoubles + 2) *
         sizeof(double);
}

// What bounds a step of few rows is that its nine launches take 3 to 8 us each, whatever they do: 58 us together with the
// gaps.  Here it is the six meetings, 1.6 us each, and the two factorizations, 2 us each: 30 us (2,000 rows, 24 to 56 columns;
// 4,040 rows 36).  Solves of 2,000 and 4,040 rows: 1.51 -> 1.26 and 1.64 -> 1.50 ms.
// Workgroup w holds rows [w rows, w rows + rows) of the basis and of the block in LDS throughout; what the others need of it
// are its partial sums of the coefficients and of the Gram matrices.  The coefficients are added up in two goes: every
// workgroup adds its share of them over all workgroups, then all read the sums.
__global__ __launch_bounds__(kStepThreads) __attribute__((amdgpu_waves_per_eu(2))) void small_step_kernel(SmallStep a) {
  extern __shared__ double lds[];
  const int j = a.j, pitch = step_pitch(j), rows = a.rows, j16 = pitch - 1;
  StepLds s;
  s.q = lds;
  s.w = s.q + (size_t)rows * pitch;
  s.h = s.w + rows * kWP;
  s.red = s.h + pitch * kWP;
  s.gram = s.red + kStepThreads;
  s.rinv = s.gram + kB * kB;
  s.r = s.rinv + kRinvDoubles;
  s.ok = reinterpret_cast<int*>(s.r + kRinvDoubles);

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i = lane & 15, g = lane >> 4;
  const int nwg = gridDim.x, wg = blockIdx.x;
  const int64_t row0 = (int64_t)wg * rows;
  uint32_t target = a.base;

  if (wg == 0 && tid == 0 && a.done) __hip_atomic_store(a.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  for (int e = tid; e < kRinvDoubles; e += kStepThreads) s.r[e] = e / kPartialPad == e % kPartialPad ? 1.0 : 0.0;

  // the workgroup's rows of the basis: eight rows a wave requested at once
  for (int c0 = 0; c0 < j16; c0 += 64) {
    const int c = c0 + lane;
    for (int r0 = wave * 8; r0 < rows; r0 += kStepWaves * 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t row = row0 + r0 + u;
        v[u] = a.basis[(row < a.n ? row : a.n - 1) * a.ld + (c < j ? c : j - 1)];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c < j16) s.q[(r0 + u) * pitch + c] = c < j && row0 + r0 + u < a.n ? v[u] : 0.0;
    }
  }

  // the product, or the block as it is
  if (a.val) {
    constexpr int L = 8, CL = kB / 2, NS = L / CL;  // lanes a row; a lane carries two columns; entries at a time
    const int rl = lane % L, tl = rl % CL, sg = rl / CL;
    const double2* __restrict__ z2 = reinterpret_cast<const double2*>(a.z);
    for (int lr = tid / L; lr < rows; lr += kStepThreads / L) {
      const int64_t row = row0 + lr;
      const int64_t e0 = row < a.n ? a.rowptr[row] : 0, e1 = row < a.n ? a.rowptr[row + 1] : 0;
      double acc0 = 0.0, acc1 = 0.0;
      for (int64_t e = e0; e < e1; e += 2 * L) {  // 16 entries, eight gathers in flight; past the end the last one, times 0
        int32_t c[2];
        double v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int64_t el = e + h * L + rl;
          c[h] = a.col[el < e1 ? el : e1 - 1];
          v[h] = el < e1 ? a.val[el] : 0.0;
        }
        double2 x[2 * CL];
#pragma unroll
        for (int u = 0; u < 2 * CL; ++u) x[u] = z2[(int64_t)__shfl(c[u / CL], (u % CL) * NS + sg, L) * CL + tl];
#pragma unroll
        for (int u = 0; u < 2 * CL; ++u) {
          const double vu = __shfl(v[u / CL], (u % CL) * NS + sg, L);
          acc0 += vu * x[u].x;
          acc1 += vu * x[u].y;
        }
      }
      acc0 += __shfl_xor(acc0, CL, L);
      acc1 += __shfl_xor(acc1, CL, L);
      if (sg == 0) {
        s.w[lr * kWP + 2 * tl] = acc0;
        s.w[lr * kWP + 2 * tl + 1] = acc1;
      }
    }
  } else {
    for (int e = tid; e < rows * kB; e += kStepThreads) {
      const int64_t row = row0 + e / kB;
      s.w[e / kB * kWP + e % kB] = row < a.n ? a.basis[row * a.ld + j + e % kB] : 0.0;
    }
  }

  // ---- Gram-Schmidt against columns [from, j), twice at most
  double first_sum = 0.0;  // workgroup 0: the coefficient of the slot that this thread keeps
  for (int pass = 0; pass < 2; ++pass) {
    const int from = pass == 0 ? a.from1 : a.from2;
    if (from >= j) continue;  // uniform over the grid
    const int t0 = from / 16, total = (j - from) * kB;
    double* mine = a.part + (int64_t)wg * total;
    __syncthreads();
    for (int t = t0 + wave; t < j16 / 16; t += kStepWaves) {
      d4 acc = {0.0, 0.0, 0.0, 0.0};
      for (int k = 0; k < rows; k += 4) {
        const double x = s.q[(k + g) * pitch + 16 * t + i];
        const double y = i < kB ? s.w[(k + g) * kWP + i] : 0.0;
        acc = MFMA_F64(x, y, acc);
      }
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int c = 16 * t + 4 * rr + g;
        if (i < kB && c >= from && c < j) put_shared(mine + (c - from) * kB + i, acc[rr]);
      }
    }
    if (!meet(a.sync, target += nwg, a.polls, s.ok)) return;
    // this workgroup's share of the coefficients: `share` of them, `split` threads each
    const int share = (total + nwg - 1) / nwg;
    for (int first = 0; first < share; first += 64) {
      const int el = tid % 64, r = tid / 64, e = wg * share + first + el;
      const bool has = first + el < share && e < total;
      double acc = 0.0;
      if (has) {
        int q = r;
        for (; q + 3 * kStepWaves < nwg; q += 4 * kStepWaves) {
          double v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = get_shared(a.part + (int64_t)(q + u * kStepWaves) * total + e);
#pragma unroll
          for (int u = 0; u < 4; ++u) acc += v[u];
        }
        for (; q < nwg; q += kStepWaves) acc += get_shared(a.part + (int64_t)q * total + e);
      }
      s.red[tid] = acc;
      __syncthreads();
      if (r == 0 && has) {
        double sum = s.red[el];
#pragma unroll
        for (int x = 1; x < kStepWaves; ++x) sum += s.red[x * 64 + el];
        put_shared(a.h + e, sum);
      }
      __syncthreads();
    }
    if (!meet(a.sync, target += nwg, a.polls, s.ok)) return;
    // all coefficients: rows of columns that take no part are zero
    for (int base = 0; base < j16 * kB; base += 4 * kStepThreads) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = base + u * kStepThreads + tid - from * kB;
        v[u] = e >= 0 && e < total ? get_shared(a.h + e) : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = base + u * kStepThreads + tid;
        if (e < j16 * kB) s.h[e / kB * kWP + e % kB] = v[u];
      }
    }
    __syncthreads();
    if (a.slot_a && wg == 0 && tid < kB * kB) {
      const int r = tid / kB, t = tid % kB;
      first_sum += s.h[(j - kB + r) * kWP + t];
      a.slot_a[r * kPartialPad + t] = first_sum;
    }
    for (int t = wave; t < rows / 16; t += kStepWaves) {
      d4 acc = {0.0, 0.0, 0.0, 0.0};
      for (int k = from / 4 * 4; k < j16; k += 4) {
        const double x = s.q[(16 * t + i) * pitch + k + g];
        const double y = i < kB ? s.h[(k + g) * kWP + i] : 0.0;
        acc = MFMA_F64(x, y, acc);
      }
      if (i < kB)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) s.w[(16 * t + 4 * rr + g) * kWP + i] -= acc[rr];
    }
  }

  // ---- Cholesky QR, twice
  for (int pass = 0; pass < 2; ++pass) {
    double* parts = a.gpart + (size_t)pass * nwg * kB * kB;
    __syncthreads();
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k = 4 * wave; k < rows; k += 4 * kStepWaves) {
      const double x = i < kB ? s.w[(k + g) * kWP + i] : 0.0;
      acc = MFMA_F64(x, x, acc);
    }
    if (i < kB)
#pragma unroll
      for (int rr = 0; rr < 2; ++rr) s.red[wave * kB * kB + (4 * rr + g) * kB + i] = acc[rr];  // rows 8 and up vanish
    __syncthreads();
    if (tid < kB * kB) {
      double sum = s.red[tid];
#pragma unroll
      for (int x = 1; x < kStepWaves; ++x) sum += s.red[x * kB * kB + tid];
      put_shared(parts + wg * kB * kB + tid, sum);
    }
    if (!meet(a.sync, target += nwg, a.polls, s.ok)) return;
    {
      const int e = tid % (kB * kB), r = tid / (kB * kB);
      double sum = 0.0;
      int q = r;
      for (; q + 3 * kStepWaves < nwg; q += 4 * kStepWaves) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = get_shared(parts + (q + u * kStepWaves) * kB * kB + e);
#pragma unroll
        for (int u = 0; u < 4; ++u) sum += v[u];
      }
      for (; q < nwg; q += kStepWaves) sum += get_shared(parts + q * kB * kB + e);
      s.red[tid] = sum;
      __syncthreads();
      if (tid < kB * kB) {  // a wave
        double tot = s.red[tid];
#pragma unroll
        for (int x = 1; x < kStepWaves; ++x) tot += s.red[x * kB * kB + tid];
        s.gram[tid] = tot;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (pass == 0 && wg == 0) a.slot_g[tid / kB * kPartialPad + tid % kB] = tot;
        // the factor goes to where the one before it was; before the first that is the identity
        chol_wave<kB>(s.gram, kB, nullptr, s.rinv, s.r, s.r, a.abs_tol2[pass], a.rel_tol[pass]);
      }
      __syncthreads();
    }
    for (int t = wave; t < rows / 16; t += kStepWaves) {
      d4 acc2 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < kB; k += 4) {
        const double x = s.w[(16 * t + i) * kWP + k + g];
        const double y = i < kB ? s.rinv[(k + g) * kPartialPad + i] : 0.0;
        acc2 = MFMA_F64(x, y, acc2);
      }
      // the wave has read its rows; the matrix instruction's result is there only then
      if (i < kB)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) s.w[(16 * t + 4 * rr + g) * kWP + i] = acc2[rr];
    }
  }
  __syncthreads();
  if (wg == 0 && tid < kB * kB) a.slot_r[tid / kB * kPartialPad + tid % kB] = s.r[tid / kB * kPartialPad + tid % kB];
  for (int e = tid; e < rows * kB; e += kStepThreads) {
    const int64_t row = row0 + e / kB;
    if (row < a.n) {
      const double v = s.w[e / kB * kWP + e % kB];
      a.basis[row * a.ld + j + e % kB] = v;
      a.z[row * kB + e % kB] = v;
    }
  }
  if (a.done) {
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(a.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

}  // namespace

// 64 rows a workgroup, which four waves' tiles of 16 make quick work of, 128 where that would be too many workgroups (a meeting
// of 32 workgroups takes 1.0 us, of 128 2.0, of 256 3.7).
int small_step_rows(int64_t n, int j, size_t lds_limit) {
  for (int rows : {64, 128}) {
    if (n > (int64_t)rows * kSmallStepGroups || j > kSmallStepColumns) continue;
    return step_lds_bytes(j, rows) <= lds_limit ? rows : 0;
  }
  return 0;
}

hipError_t launch_small_step(const SmallStep& a, size_t lds_limit, hipStream_t st) {
  if (a.rows <= 0 || a.rows != small_step_rows(a.n, a.j, lds_limit) || a.j < 0 || (a.slot_a && a.j < kB) || a.from1 < 0 || a.from2 < 0)
    return hipErrorInvalidValue;
  const size_t lds = step_lds_bytes(a.j, a.rows);
  hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(small_step_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(small_step_kernel, dim3((unsigned)small_step_groups(a.n, a.rows)), dim3(kStepThreads), lds, st, a);
  return hipGetLastError();
}

}  // namespace sceig
