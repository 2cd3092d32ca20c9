// Stands in for <hip/hip_runtime.h> where device code of the library's headers is
// compiled for the CPU and run by one thread (a wave of one lane, a block of one
// thread).  Atomics are the host's; a sleep is nothing.
#pragma once
#include <stdint.h>

#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, order)
#define __hip_atomic_fetch_sub(p, v, order, scope) __atomic_fetch_sub(p, v, order)
#define __hip_atomic_fetch_or(p, v, order, scope) __atomic_fetch_or(p, v, order)
#define __hip_atomic_fetch_and(p, v, order, scope) __atomic_fetch_and(p, v, order)
#define __hip_atomic_exchange(p, v, order, scope) __atomic_exchange_n(p, v, order)
#define __hip_atomic_compare_exchange_strong(p, expected, desired, ok, fail, scope) \
  __atomic_compare_exchange_n(p, expected, desired, false, ok, fail)
#define __builtin_amdgcn_s_sleep(n) ((void)0)
#define __builtin_amdgcn_mbcnt_lo(m, x) 0u
#define __builtin_amdgcn_mbcnt_hi(m, x) 0u
#define __builtin_amdgcn_alignbit(hi, lo, n) ((uint32_t)((((uint64_t)(hi) << 32) | (lo)) >> (n)))

struct CpuDim3 {
  uint32_t x, y, z;
};
static const CpuDim3 threadIdx{0, 0, 0}, blockIdx{0, 0, 0}, blockDim{1, 1, 1};

inline int __clzll(uint64_t x) { return x ? __builtin_clzll(x) : 64; }
inline int __ffsll(unsigned long long x) { return __builtin_ffsll((long long)x); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline uint64_t __ballot(int p) { return p ? 1u : 0u; }
template <typename T>
inline T __shfl(T x, int, int) { return x; }
inline void __syncthreads() {}
