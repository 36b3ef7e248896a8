// The parts of a block step whose workgroups have to hear from one another, as one launch (see launch_fused_step in kernels.h).
#include <algorithm>

#include "exchange.h"
#include "kernels.h"
#include "wave_chol.h"

namespace sceig {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
#define MFMA_F64(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64((a), (b), (c), 0, 0, 0)

constexpr int kThreads = 512;  // the factorization's registers allow two waves a SIMD
constexpr int kWaves = kThreads / 64;

// The workgroup's share of the sums over all workgroups of `part` (workgroups x total, put there before) goes to sums.
// `share` entries (8 to 64, as many as all workgroups together need) by the whole workgroup, in a fixed order.
__device__ __forceinline__ void add_up(const double* part, double* sums, int total, int wg, int nwg, double* red, int* bad) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int share = 8;
  while (share < 64 && share * nwg < total) share *= 2;
  const int el = tid & (share - 1), r = tid / share, splits = kThreads / share;
  for (int e0 = wg * share; e0 < total; e0 += nwg * share) {  // uniform over the workgroup
    double acc = 0.0;
    if (e0 + el < total) {
      for (int q = r; q < nwg; q += 4 * splits) {
        double v[4];
        if (!get(part + (int64_t)q * total + e0 + el, (int64_t)splits * total, (nwg - q + splits - 1) / splits, v)) *bad = 1;
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += v[u];
      }
    }
    for (int o = share; o < 64; o <<= 1) acc += __shfl_xor(acc, o);
    if (lane < share) red[wave * 64 + lane] = acc;
    __syncthreads();
    if (tid < share && e0 + tid < total) {
      double sum = red[tid];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) sum += red[w * 64 + tid];
      put(sums + e0 + tid, sum);
    }
    __syncthreads();
  }
}

// ---- the launch --------------------------------------------------------------------------------------------------------
__host__ __device__ inline int basis_pitch(int j) { return (j + 15) / 16 * 16 + 1; }  // odd: no bank conflicts along rows or columns
template <int B>
constexpr int kGramParts = B > 16 ? kWaves / 2 : kWaves;  // Gram matrices of waves, or of pairs of them
template <int B>
constexpr int kRed = kGramParts<B> * B * B > kThreads ? kGramParts<B> * B * B : kThreads;  // partial sums of the waves
template <int B, bool STEP>
size_t fused_lds_bytes(int j, int rows) {
  size_t d = (size_t)rows * (B + 1) + kRed<B> + 2 * B * kCholPitch<B> + 2;
  if (STEP) d += (size_t)(rows + B + 1) * basis_pitch(j);
  return d * sizeof(double);
}

// A wait that should have ended did not.
__device__ __forceinline__ void failed(const FusedStep& a) {
  if (threadIdx.x == 0) put_host(a.done, -a.number);
}

// Workgroup w holds rows [w rows, w rows + rows) of the block in LDS throughout, and with STEP those of the basis.  What the
// others need of it are its partial sums of the coefficients and of the Gram matrices; each is added up in two goes: every
// workgroup adds its share of the entries over all workgroups, then all read the sums.
template <int B, bool STEP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void fused_step_kernel(FusedStep a) {
  extern __shared__ double lds[];
  constexpr int WP = B + 1;  // row pitch of the block and of the coefficients
  constexpr int NT = B > 16 ? 2 : 1;
  static_assert(!STEP || B == kFusedStepBlock, "a tile holds the block");
  const int rows = a.rows, j = a.j;
  const int pitch = STEP ? basis_pitch(j) : 0, j16 = pitch - 1;
  double* const w = lds;
  double* const red = w + rows * WP;
  double* const gram = red;  // there between sums
  double* const factor = red + kRed<B>;  // chol_rows' results of either pass
  int* const flag = reinterpret_cast<int*>(factor + 2 * B * kCholPitch<B>);  // [0] all there, [1] a wait that should have ended did not
  double* const q = factor + 2 * B * kCholPitch<B> + 2;
  double* const h = q + (size_t)rows * pitch;

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i = lane & 15, g = lane >> 4;
  const int nwg = gridDim.x, wg = blockIdx.x;
  const int64_t row0 = (int64_t)wg * rows;
  if (tid == 0) {
    arrive(a.sync + kSyncWord);
    flag[1] = 0;
  }

  if constexpr (STEP) {
    // the workgroup's rows of the basis: eight rows a wave requested at once
    for (int c0 = 0; c0 < j16; c0 += 64) {
      const int c = c0 + lane;
      for (int r0 = wave * 8; r0 < rows; r0 += kWaves * 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int64_t row = row0 + r0 + u;
          v[u] = a.basis[(row < a.n ? row : a.n - 1) * a.ld + (c < j ? c : j - 1)];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (c < j16) q[(r0 + u) * pitch + c] = c < j && row0 + r0 + u < a.n ? v[u] : 0.0;
      }
    }
    // the product
    constexpr int L = B, CL = B / 2, NS = L / CL;  // lanes a row; a lane carries two columns; entries at a time
    const int rl = lane % L, tl = rl % CL, sg = rl / CL;
    const double2* __restrict__ z2 = reinterpret_cast<const double2*>(a.z);
    for (int lr = tid / L; lr < rows; lr += kThreads / L) {
      const int64_t row = row0 + lr;
      const int64_t e0 = row < a.n ? a.rowptr[row] : 0, e1 = row < a.n ? a.rowptr[row + 1] : 0;
      double acc0 = 0.0, acc1 = 0.0;
      for (int64_t e = e0; e < e1; e += 2 * L) {  // 2 L entries, L gathers in flight; past the end the last one, times 0
        int32_t c[2];
        double v[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const int64_t el = e + x * L + rl;
          c[x] = a.col[el < e1 ? el : e1 - 1];
          v[x] = el < e1 ? a.val[el] : 0.0;
        }
        double2 zz[2 * CL];
#pragma unroll
        for (int u = 0; u < 2 * CL; ++u) zz[u] = z2[(int64_t)__shfl(c[u / CL], (u % CL) * NS + sg, L) * CL + tl];
#pragma unroll
        for (int u = 0; u < 2 * CL; ++u) {
          const double vu = __shfl(v[u / CL], (u % CL) * NS + sg, L);
          acc0 += vu * zz[u].x;
          acc1 += vu * zz[u].y;
        }
      }
      acc0 += __shfl_xor(acc0, CL, L);
      acc1 += __shfl_xor(acc1, CL, L);
      if (sg == 0) {
        w[lr * WP + 2 * tl] = acc0;
        w[lr * WP + 2 * tl + 1] = acc1;
      }
    }
  } else {
    // the block as it is, eight entries of a thread requested at once
    for (int base = 0; base < rows * B; base += 8 * kThreads) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = base + u * kThreads + tid;
        const int64_t row = row0 + e / B;
        v[u] = a.basis[(row < a.n ? row : a.n - 1) * a.ld + j + e % B];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = base + u * kThreads + tid;
        if (e < rows * B) w[e / B * WP + e % B] = row0 + e / B < a.n ? v[u] : 0.0;
      }
    }
  }
  if (tid == 0) flag[0] = all_arrived(a.sync + kSyncWord, a.base + nwg, a.polls);
  __syncthreads();
  if (!flag[0]) return;  // nothing has been written

  double* at = a.exchange;  // what the next sum goes through
  // ---- Gram-Schmidt against columns [from, j), twice at most
  if constexpr (STEP) {
    double slot_sum = 0.0;  // workgroup 0: the coefficient of the slot that this thread keeps
    for (int pass = 0; pass < 2; ++pass) {
      const int from = pass == 0 ? a.from1 : a.from2;
      if (from >= j) continue;  // uniform over the grid
      const int total = (j - from) * B;
      double* const part = at;
      double* const sums = part + (int64_t)nwg * total;
      at = sums + total;
      if (pass > 0) __syncthreads();
      for (int t = from / 16 + wave; t < j16 / 16; t += kWaves) {
        d4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k0 = 0; k0 < rows; k0 += 16)
#pragma unroll
          for (int k = k0 + g; k < k0 + 16 + g; k += 4) {
            const double x = q[k * pitch + 16 * t + i];
            const double y = i < B ? w[k * WP + i] : 0.0;
            acc = MFMA_F64(x, y, acc);
          }
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int c = 16 * t + 4 * rr + g;
          if (i < B && c >= from && c < j) put(part + (int64_t)wg * total + (c - from) * B + i, acc[rr]);
        }
      }
      add_up(part, sums, total, wg, nwg, red, flag + 1);
      // all coefficients; rows of columns that take no part are zero
      for (int e = tid; e < j16 * B; e += 4 * kThreads) {
        const int first = from * B;
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          double one[1];
          const int eu = e + u * kThreads - first;
          if (!get(sums + (eu >= 0 && eu < total ? eu : 0), 0, eu >= 0 && eu < total, one)) flag[1] = 1;
          v[u] = one[0];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int eu = e + u * kThreads;
          if (eu < j16 * B) h[eu / B * WP + eu % B] = v[u];
        }
      }
      __syncthreads();
      if (flag[1]) return failed(a);
      if (wg == 0 && tid < B * B) {
        slot_sum += h[(j - B + tid / B) * WP + tid % B];
        put_host(a.slot_a + tid / B * a.slot_ld + tid % B, slot_sum);
      }
      for (int t = wave; t < rows / 16; t += kWaves) {
        d4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k0 = from / 16 * 16; k0 < j16; k0 += 16)
#pragma unroll
          for (int k = k0 + g; k < k0 + 16 + g; k += 4) {
            const double x = q[(16 * t + i) * pitch + k];
            const double y = i < B ? h[k * WP + i] : 0.0;
            acc = MFMA_F64(x, y, acc);
          }
        if (i < B)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) w[(16 * t + 4 * rr + g) * WP + i] -= acc[rr];
      }
    }
    __syncthreads();
  }

  // ---- Cholesky QR, twice
  for (int pass = 0; pass < 2; ++pass) {
    double* const part = at;
    double* const sums = part + (int64_t)nwg * B * B;
    at = sums + B * B;
    d4 acc[NT][NT];
#pragma unroll
    for (int x = 0; x < NT; ++x)
#pragma unroll
      for (int y = 0; y < NT; ++y) acc[x][y] = (d4){0.0, 0.0, 0.0, 0.0};
    for (int k0 = 16 * wave; k0 < rows; k0 += 16 * kWaves)
#pragma unroll
      for (int k = k0 + g; k < k0 + 16 + g; k += 4) {
        double v[NT];
#pragma unroll
        for (int x = 0; x < NT; ++x) v[x] = i < B ? w[k * WP + 16 * x + i] : 0.0;
#pragma unroll
        for (int x = 0; x < NT; ++x)
#pragma unroll
          for (int y = 0; y < NT; ++y) acc[x][y] = MFMA_F64(v[x], v[y], acc[x][y]);
      }
#pragma unroll
    for (int turn = 0; turn < kWaves / kGramParts<B>; ++turn) {  // the second wave of a pair adds to what the first has left
      if (turn > 0) __syncthreads();
      if (i < B && wave / kGramParts<B> == turn)
#pragma unroll
        for (int x = 0; x < NT; ++x)
#pragma unroll
          for (int y = 0; y < NT; ++y)
#pragma unroll
            for (int rr = 0; rr < (B < 16 ? B / 4 : 4); ++rr) {  // rows from B on vanish
              double* const to = red + wave % kGramParts<B> * B * B + (16 * x + 4 * rr + g) * B + 16 * y + i;
              *to = (turn > 0 ? *to : 0.0) + acc[x][y][rr];
            }
    }
    __syncthreads();
    for (int e = tid; e < B * B; e += kThreads) {
      double sum = red[e];
#pragma unroll
      for (int x = 1; x < kGramParts<B>; ++x) sum += red[x * B * B + e];
      put(part + (int64_t)wg * B * B + e, sum);
    }
    __syncthreads();
    add_up(part, sums, B * B, wg, nwg, red, flag + 1);
    for (int e = tid; e < B * B; e += kThreads) {
      double one[1];
      if (!get(sums + e, 0, 1, one)) flag[1] = 1;
      gram[e] = one[0];
      if (pass == 0 && wg == 0 && a.slot_g) put_host(a.slot_g + e / B * a.slot_ld + e % B, one[0]);
    }
    __syncthreads();
    if (flag[1]) return failed(a);
    const double* const made = factor + pass * B * kCholPitch<B>;
    if (wave == 0) chol_rows<B>(gram, B, factor + pass * B * kCholPitch<B>, a.abs_tol2[pass], a.rel_tol[pass]);
    __syncthreads();
    for (int t = wave; t < rows / 16; t += kWaves) {
      d4 out[NT];
#pragma unroll
      for (int y = 0; y < NT; ++y) out[y] = (d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < B; k += 4) {
        const double x = w[(16 * t + i) * WP + k + g];
#pragma unroll
        for (int y = 0; y < NT; ++y)
          out[y] = MFMA_F64(x, i < B ? made[(16 * y + i) * kCholPitch<B> + B + k + g] : 0.0, out[y]);
      }
      // the wave alone reads these rows, and has
      if (i < B)
#pragma unroll
        for (int y = 0; y < NT; ++y)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) w[(16 * t + 4 * rr + g) * WP + 16 * y + i] = out[y][rr];
    }
    __syncthreads();
  }
  for (int e = tid; e < rows * B; e += kThreads) {
    const int64_t row = row0 + e / B;
    if (row < a.n) {
      const double v = w[e / B * WP + e % B];
      a.basis[row * a.ld + j + e % B] = v;
      if (a.z) a.z[row * B + e % B] = v;
    }
  }
  if (wg == 0 && a.slot_r) {  // the product of both factors
    for (int e = tid; e < B * B; e += kThreads) {
      const int r = e / B, t = e % B;
      double sum = 0.0;
#pragma unroll
      for (int x = 0; x < B; ++x) sum += factor[(B + r) * kCholPitch<B> + x] * factor[x * kCholPitch<B> + t];
      put_host(a.slot_r + r * a.slot_ld + t, sum);
    }
  }
  // the places that the launch before this one has written are for the next one
  for (int64_t e = (int64_t)wg * kThreads + tid; e < a.clear; e += (int64_t)nwg * kThreads)
    reinterpret_cast<long long*>(a.used)[e] = -1;
  if (wg == 0) {  // the slot, in host memory, before the word that says so
    host_written();
    __syncthreads();
  }
  if (tid == 0 && __hip_atomic_fetch_add(a.sync + kSyncDone, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == a.base + nwg)
    put_host(a.done, a.number);
}

// What a first launch finds: nothing exchanged, nobody arrived.
__global__ __launch_bounds__(kThreads) void fused_prepare_kernel(long long* __restrict__ exchange, int64_t len,
                                                                 uint32_t* __restrict__ sync, uint32_t word) {
  if (blockIdx.x == 0 && threadIdx.x >= kSyncWord && threadIdx.x < kSyncWords) sync[threadIdx.x] = threadIdx.x == kSyncWord ? word : 0;
  for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < len; e += (int64_t)gridDim.x * kThreads) exchange[e] = -1;
}

__global__ void fused_stop_kernel(uint32_t* __restrict__ sync) { atomicOr(sync + kSyncWord, kStopped); }

template <int B, bool STEP>
hipError_t launch(const FusedStep& a, hipStream_t st) {
  const size_t lds = fused_lds_bytes<B, STEP>(a.j, a.rows);
  const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(fused_step_kernel<B, STEP>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL((fused_step_kernel<B, STEP>), dim3((unsigned)fused_groups(a.n, a.rows)), dim3(kThreads), lds, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fused_prepare(double* exchange, int64_t len, uint32_t* sync, bool stopped, hipStream_t st) {
  const int64_t groups = std::min<int64_t>((len + 4 * kThreads - 1) / (4 * kThreads), 1024);
  hipLaunchKernelGGL(fused_prepare_kernel, dim3((unsigned)std::max<int64_t>(groups, 1)), dim3(kThreads), 0, st,
                     reinterpret_cast<long long*>(exchange), len, sync, stopped ? kStopped : 0u);
  return hipGetLastError();
}

hipError_t launch_fused_stop(uint32_t* sync, hipStream_t st) {
  hipLaunchKernelGGL(fused_stop_kernel, dim3(1), dim3(1), 0, st, sync);
  return hipGetLastError();
}

int fused_step_rows(int64_t n, int j, size_t lds_limit) {
  for (int rows : {64, 128})
    if (n <= (int64_t)rows * 128) return j <= kFusedColumns && fused_lds_bytes<kFusedStepBlock, true>(j, rows) <= lds_limit ? rows : 0;
  return 0;
}

int fused_qr_rows(int64_t n, int b, size_t lds_limit) {
  const int64_t rows = std::max<int64_t>(64, (n + 16 * kFusedGroups - 1) / (16 * kFusedGroups) * 16);
  if ((b != 8 && b != 16 && b != 32) || rows > 4096) return 0;
  const size_t lds = b == 8    ? fused_lds_bytes<8, false>(0, (int)rows)
                     : b == 16 ? fused_lds_bytes<16, false>(0, (int)rows)
                               : fused_lds_bytes<32, false>(0, (int)rows);
  return lds <= lds_limit ? (int)rows : 0;
}

hipError_t launch_fused_step(const FusedStep& a, size_t lds_limit, hipStream_t st) {
  if (a.rows <= 0 || a.rows != fused_step_rows(a.n, a.j, lds_limit) || a.j < kFusedStepBlock || a.from1 < 0 || a.from2 < 0)
    return hipErrorInvalidValue;
  return launch<kFusedStepBlock, true>(a, st);
}

hipError_t launch_fused_qr(const FusedStep& a, int b, size_t lds_limit, hipStream_t st) {
  if (a.rows <= 0 || a.rows != fused_qr_rows(a.n, b, lds_limit) || a.j < 0) return hipErrorInvalidValue;
  return b == 8 ? launch<8, false>(a, st) : b == 16 ? launch<16, false>(a, st) : launch<32, false>(a, st);
}

}  // namespace sceig
