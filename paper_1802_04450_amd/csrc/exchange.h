// What the workgroups of one running launch tell one another (device code).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sceig {
namespace {

constexpr uint32_t kStopped = 1u << 31;  // in the word that counts arrivals: no launch goes on

// Values go through agent-scope atomics, which pass by the caches that the workgroups do not share.  A place that nobody has
// written yet holds all ones: who needs it looks until it holds something else, so that a value takes one store and one
// load from one workgroup to the other (1.3 us; waiting for the store, counting oneself in and looking at the count before
// the load 2.5 us).  An all-ones NaN of the inputs goes as the ordinary one.
__device__ __forceinline__ void put(double* p, double v) {
  long long bits = __double_as_longlong(v);
  if (bits == -1) bits = 0x7ff8000000000000ll;
  __hip_atomic_store(reinterpret_cast<long long*>(p), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ long long look(const double* p) {
  return __hip_atomic_load(reinterpret_cast<const long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// K values at p[0], p[stride] ...; those from `count` on are zero.  Every workgroup has arrived when this is called, so the wait
// is for work under way; its bound is only there so that no wait is without one.
constexpr int kLooks = 1 << 20;
template <int K>
__device__ __forceinline__ bool get(const double* p, int64_t stride, int count, double (&v)[K]) {
  for (int i = 0; i < kLooks; ++i) {
    long long bits[K];
    bool all = true;
#pragma unroll
    for (int u = 0; u < K; ++u) bits[u] = u < count ? look(p + u * stride) : 0;
#pragma unroll
    for (int u = 0; u < K; ++u) {
      all = all && bits[u] != -1;
      v[u] = __longlong_as_double(bits[u]);
    }
    if (all) return true;
  }
  return false;
}

// Counts the workgroup in (one thread).
__device__ __forceinline__ void arrive(uint32_t* word) {
  __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Whether all workgroups of the launch have arrived (one thread): looked for `looks` times, then the word is stopped, unless
// they have by then.  All workgroups get the same answer, and after a true one all of them are running.
__device__ __forceinline__ bool all_arrived(uint32_t* word, uint32_t target, int looks) {
  uint32_t seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int i = 0; i < looks && seen != target && !(seen & kStopped); ++i)
    seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  while (seen != target && !(seen & kStopped)) {  // ends: the word changes at most once for every workgroup in between
    if (__hip_atomic_compare_exchange_strong(word, &seen, kStopped, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return false;
  }
  return seen == target;
}

// Stores to coherent host memory, and the wait that orders them: a release fence would write the whole L2 back first (5 to 10 us).
template <class T>
__device__ __forceinline__ void put_host(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void host_written() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

}  // namespace
}  // namespace sceig
