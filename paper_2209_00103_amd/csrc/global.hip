// Access by global index (the rw_g variant of Sec. VI-B).  Global element i is
// element i - P[v] of LFVector v, where P is the exclusive prefix of the
// LFVector sizes (Sec. IV) and v the last LFVector with P[v] <= i; an empty
// LFVector shares its offset with the next one, so this choice skips it.  Inside
// the LFVector the closed form gives bucket and offset.
//
// One thread per element, each with a search of P of its own, is the shortest path
// while every element can be in flight at once.  With more of them the searches'
// chains of dependent loads, not the elements' traffic, bound it (V = 512, 2^24
// u32 elements: an update of all 161 us, 0.83 TB/s; 2^22 random reads 99 us), so the
// update of a larger array searches once per wave and span of consecutive indices
// and streams the span's bucket runs (24-27 us, 5.0-5.6 TB/s), and a larger gather
// keeps P (or a sample of it) in LDS and runs several searches per thread side by
// side (84 us, bound by the 128-byte line that each random read fetches: 541 MB,
// 6.4 TB/s).
#include "gga_internal.h"

namespace gga {
namespace {

constexpr uint32_t kGlobalThreads = 256;
constexpr uint32_t kGlobalBlocks = 8192;  // 32 workgroups per CU, grid-stride

// Address of global element i < P[V], by a binary search of P.
template <typename T>
__device__ __forceinline__ gptr<T> element_at(const ArrRef& A, uint64_t i) {
  uint32_t lo = 0, hi = A.V;  // P[lo] <= i < P[hi]
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (A.prefix[mid] <= i) lo = mid;
    else hi = mid;
  }
  const uint64_t j = i - A.prefix[lo];
  const uint32_t b = bucket_of(A.log2F, j);
  return gmem(reinterpret_cast<T*>(A.bptr[(uint64_t)lo * kMaxBuckets + b])) + offset_in(A.log2F, j, b);
}

// One thread per element (small arrays, few reads).
template <typename T>
__device__ __forceinline__ void rw_elements(const ArrRef& A, uint32_t op, uint64_t n) {
  const uint64_t stride = (uint64_t)gridDim.x * kGlobalThreads;
  for (uint64_t i = (uint64_t)blockIdx.x * kGlobalThreads + threadIdx.x; i < n; i += stride) {
    const gptr<T> p = element_at<T>(A, i);
    *p = apply_op<T>(op, *p);
  }
}

template <typename T>
__global__ __launch_bounds__(kGlobalThreads) void rw_element_kernel(ArrRef A, uint32_t op) {
  rw_elements<T>(A, op, A.prefix[A.V]);
}

template <typename T>
__global__ __launch_bounds__(kGlobalThreads) void gather_element_kernel(ArrRef A, const uint64_t* idx, uint64_t n,
                                                                       T* out) {
  const uint64_t k = (uint64_t)blockIdx.x * kGlobalThreads + threadIdx.x;
  if (k >= n) return;
  const uint64_t i = idx[k];
  if (i < A.prefix[A.V]) out[k] = *element_at<T>(A, i);
  else set_error(A.err, kErrRange);
}

// x = op(x) over n elements from p on, by one wave, kU vectors per lane in flight
// (unconditional loads, clamped indices; only the lane that owns a vector stores it).
template <typename T, uint32_t kU>
__device__ __forceinline__ void wave_rw_run(gptr<T> p, uint32_t n, uint32_t op) {
  constexpr uint32_t VPL = 16 / sizeof(T);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t mis = (uint32_t)((reinterpret_cast<uintptr_t>((T*)p) / sizeof(T)) & (VPL - 1));
  uint32_t head = mis ? VPL - mis : 0u;
  if (head > n) head = n;
  const uint32_t nv = (n - head) / VPL, tail = head + nv * VPL;
  const gptr<u32x4> vp = reinterpret_cast<gptr<u32x4>>(p + head);
  for (uint32_t q0 = 0; q0 < nv; q0 += kU * 64) {
    u32x4 x[kU];
#pragma unroll
    for (uint32_t k = 0; k < kU; ++k) {
      const uint32_t q = q0 + 64u * k + lane;
      x[k] = vp[q < nv ? q : nv - 1];
    }
#pragma unroll
    for (uint32_t k = 0; k < kU; ++k) {
      const uint32_t q = q0 + 64u * k + lane;
      if (q < nv) __builtin_nontemporal_store(op_vec<T>(op, x[k]), vp + q);
    }
  }
  if (lane < head) p[lane] = apply_op<T>(op, p[lane]);
  if (tail + lane < n) p[tail + lane] = apply_op<T>(op, p[tail + lane]);
}

// One wave per span of kU KiB of consecutive global indices.  The span's first
// LFVector comes from one 64-way search of P; then, while the span reaches at
// most kRunVectors LFVectors, its bucket runs are streamed in order.  A span over
// more of them (short LFVectors) takes its elements one by one, kE per lane side by
// side, each search limited to the LFVectors that the span reaches.
constexpr uint32_t kRunVectors = 4;
template <typename T, uint32_t kU>
__device__ __forceinline__ void rw_spans(const ArrRef& A, uint32_t op, uint64_t n) {
  constexpr uint32_t kPer = kU * (16 / sizeof(T)), kSpan = 64 * kPer, kE = kPer < 8 ? kPer : 8;
  const uint64_t waves = (uint64_t)gridDim.x * (kGlobalThreads / 64);
  const uint32_t lane = threadIdx.x & 63u;
  for (uint64_t w = (uint64_t)blockIdx.x * (kGlobalThreads / 64) + (threadIdx.x >> 6); w * kSpan < n; w += waves) {
    const uint64_t i0 = w * kSpan, i1 = i0 + kSpan < n ? i0 + kSpan : n;
    uint32_t v = wave_search(A.prefix, A.V, i0);
    const uint32_t reach = A.prefix[v + 1] >= i1 ? 1u : wave_search(A.prefix + v, A.V - v, i1 - 1) + 1;
    if (reach <= kRunVectors) {
      uint64_t p0 = A.prefix[v], p1 = A.prefix[v + 1];
      for (uint64_t i = i0; i < i1;) {
        if (i >= p1) {  // the next LFVector (an empty one ends where it starts)
          ++v;
          p0 = p1;
          p1 = A.prefix[v + 1];
          continue;
        }
        const uint64_t j = i - p0;
        const uint32_t b = bucket_of(A.log2F, j);
        uint64_t end = p0 + bucket_start(A.log2F, b) + bucket_len(A.log2F, b);
        if (end > p1) end = p1;
        if (end > i1) end = i1;
        const gptr<T> p = gmem(reinterpret_cast<T*>(A.bptr[(uint64_t)v * kMaxBuckets + b])) + offset_in(A.log2F, j, b);
        wave_rw_run<T, kU>(p, (uint32_t)(end - i), op);
        i = end;
      }
      continue;
    }
    const uint64_t* P = A.prefix + v;
    uint32_t top = 1;
    while (2 * top < reach) top *= 2;
    for (uint64_t i = i0 + lane; i < i1; i += 64 * kE) {  // lanes past the end redo the span's last element, unstored
      uint32_t at[kE];
#pragma unroll
      for (uint32_t u = 0; u < kE; ++u) at[u] = 0;
      for (uint32_t step = top; step; step >>= 1) {  // the last P at or below the index
#pragma unroll
        for (uint32_t u = 0; u < kE; ++u) {
          const uint32_t m = at[u] + step;
          const uint64_t iu = i + 64 * u < i1 ? i + 64 * u : i1 - 1;
          if (m < reach && P[m] <= iu) at[u] = m;
        }
      }
      uint64_t row[kE], off[kE];
#pragma unroll
      for (uint32_t u = 0; u < kE; ++u) {
        const uint64_t j = (i + 64 * u < i1 ? i + 64 * u : i1 - 1) - P[at[u]];
        const uint32_t b = bucket_of(A.log2F, j);
        row[u] = A.bptr[(uint64_t)(v + at[u]) * kMaxBuckets + b];
        off[u] = offset_in(A.log2F, j, b);
      }
      T x[kE];
#pragma unroll
      for (uint32_t u = 0; u < kE; ++u) x[u] = gmem(reinterpret_cast<T*>(row[u]))[off[u]];
#pragma unroll
      for (uint32_t u = 0; u < kE; ++u)
        if (i + 64 * u < i1) gmem(reinterpret_cast<T*>(row[u]))[off[u]] = apply_op<T>(op, x[u]);
    }
  }
}

// Where one thread per element gives way to spans: at 4 MiB (us, element against span
// form: V = 512, 1.0e5 u32 elements 4.3 and 6.7, 3.0e6 27 and 14; V = 4096, 1.0e6 u32
// 14.6 and 16.0, 2.0e6 24 and 15.5, 6.0e5 u64 13.2 and 13.2).  Spans of 8 KiB once they
// fill the chip's 8192 wave slots (64 MiB of elements), 2 KiB below.
constexpr uint64_t kSpanMinBytes = 1ull << 22;
constexpr uint64_t kWideMinBytes = 1ull << 26;

// The host's bound of the size, which chooses the launch, may be far above it (rounds
// that inserted little, shrinks): the form follows the size itself (V = 512, 30000
// elements under a bound of 6e7: 32 us in spans of 8 KiB, 7 us as elements).
template <typename T, bool kWide>
__global__ __launch_bounds__(kGlobalThreads) void rw_global_kernel(ArrRef A, uint32_t op) {
  const uint64_t n = A.prefix[A.V];
  if (n * sizeof(T) < kSpanMinBytes)
    rw_elements<T>(A, op, n);
  else if (kWide && n * sizeof(T) >= kWideMinBytes)
    rw_spans<T, 8>(A, op, n);
  else
    rw_spans<T, 2>(A, op, n);
}

// Every workgroup keeps P[0], P[2^k], P[2 2^k], ... in LDS, k the smallest that
// leaves at most kSample entries (all of P up to 2048 LFVectors; 16 KiB keep eight
// workgroups on a CU).  A thread searches for kReads indices side by side, first
// there, then, for k > 0, in the 2^k entries of P after the one found.
constexpr uint32_t kSample = 2048;
constexpr uint32_t kReads = 4;
template <typename T>
__global__ __launch_bounds__(kGlobalThreads) void gather_kernel(ArrRef A, const uint64_t* idx, uint64_t n, T* out,
                                                               uint32_t k, uint32_t top) {
  __shared__ uint64_t s_p[kSample];
  const uint32_t tid = threadIdx.x;
  const uint64_t size = A.prefix[A.V];
  const uint32_t ns = (A.V + (1u << k) - 1) >> k;
  for (uint32_t q = tid; q < ns; q += kGlobalThreads) s_p[q] = A.prefix[(uint64_t)q << k];
  __syncthreads();
  bool bad = false;
  for (uint64_t c = (uint64_t)blockIdx.x * kGlobalThreads * kReads; c < n;
       c += (uint64_t)gridDim.x * kGlobalThreads * kReads) {
    uint64_t i[kReads];
    uint32_t v[kReads];
#pragma unroll
    for (uint32_t u = 0; u < kReads; ++u) {
      const uint64_t q = c + u * kGlobalThreads + tid;
      i[u] = idx[q < n ? q : n - 1];
      v[u] = 0;
    }
    for (uint32_t step = top; step; step >>= 1) {  // the last sample at or below i
#pragma unroll
      for (uint32_t u = 0; u < kReads; ++u) {
        const uint32_t m = v[u] + step;
        if (m < ns && s_p[m] <= i[u]) v[u] = m;
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < kReads; ++u) v[u] <<= k;
    for (uint32_t step = (1u << k) >> 1; step; step >>= 1) {
#pragma unroll
      for (uint32_t u = 0; u < kReads; ++u) {
        const uint32_t m = v[u] + step;
        if (m < A.V && A.prefix[m] <= i[u]) v[u] = m;
      }
    }
    uint64_t p[kReads], off[kReads];
#pragma unroll
    for (uint32_t u = 0; u < kReads; ++u) {  // an index past the size reads the table's first word, unused
      const bool in = i[u] < size;
      const uint64_t j = in ? i[u] - (k ? A.prefix[v[u]] : s_p[v[u]]) : 0;
      const uint32_t b = bucket_of(A.log2F, j);
      p[u] = A.bptr[in ? (uint64_t)v[u] * kMaxBuckets + b : 0];
      off[u] = offset_in(A.log2F, j, b);
    }
#pragma unroll
    for (uint32_t u = 0; u < kReads; ++u) {
      const uint64_t q = c + u * kGlobalThreads + tid;
      if (q >= n) continue;
      if (i[u] < size) out[q] = gmem(reinterpret_cast<T*>(p[u]))[off[u]];
      else bad = true;
    }
  }
  if (bad) set_error(A.err, kErrRange);
}

}  // namespace

// Where one thread per read gives way to the LDS form (us, element against LDS form): at
// V = 4096, 1.6e5 reads 7.8 against 10.7, 2.0e6 60 against 44, at V = 32, 2.0e6 40
// against 36.
constexpr uint64_t kGatherMinReads = 1ull << 20;

template <typename T>
static void queue_rw_global(const ggarray* a, uint32_t op, hipStream_t s) {
  const dim3 block(kGlobalThreads);
  if (a->size_ub < kSpanMinBytes >> a->elem_log2) {
    const uint64_t blocks = a->size_ub / kGlobalThreads + 1;
    hipLaunchKernelGGL(rw_element_kernel<T>, dim3((uint32_t)blocks), block, 0, s, a->ref, op);
    return;
  }
  // A wave per span of the host's bound of the size, looping beyond.
  const bool wide = a->size_ub >= kWideMinBytes >> a->elem_log2;
  const uint64_t spans = (a->size_ub >> ((wide ? 13u : 11u) - a->elem_log2)) + 1, per = kGlobalThreads / 64;
  const dim3 grid((uint32_t)(spans < kGlobalBlocks * per ? (spans + per - 1) / per : kGlobalBlocks));
  if (wide)
    hipLaunchKernelGGL((rw_global_kernel<T, true>), grid, block, 0, s, a->ref, op);
  else
    hipLaunchKernelGGL((rw_global_kernel<T, false>), grid, block, 0, s, a->ref, op);
}

int launch_rw_global(ggarray* a, uint32_t op, hipStream_t s) {
  if (a->elem_bytes == 4) queue_rw_global<uint32_t>(a, op, s);
  else queue_rw_global<uint64_t>(a, op, s);
  return hip_status(hipGetLastError());
}

template <typename T>
static void queue_gather(const ggarray* a, const uint64_t* idx, uint64_t n, T* out, hipStream_t s) {
  const dim3 block(kGlobalThreads);
  if (n < kGatherMinReads) {
    hipLaunchKernelGGL(gather_element_kernel<T>, dim3((uint32_t)((n + kGlobalThreads - 1) / kGlobalThreads)), block,
                       0, s, a->ref, idx, n, out);
    return;
  }
  constexpr uint64_t kPer = kGlobalThreads * kReads;
  uint64_t blocks = (n + kPer - 1) / kPer;
  if (blocks > kGlobalBlocks) blocks = kGlobalBlocks;
  uint32_t k = 0, top = 1;
  while (((a->V + (1u << k) - 1) >> k) > kSample) ++k;
  while (2 * top < ((a->V + (1u << k) - 1) >> k)) top *= 2;
  hipLaunchKernelGGL(gather_kernel<T>, dim3((uint32_t)blocks), block, 0, s, a->ref, idx, n, out, k, top);
}

int launch_gather(ggarray* a, const uint64_t* idx, uint64_t n, void* out, hipStream_t s) {
  if (n == 0) return GGA_OK;
  if (a->elem_bytes == 4) queue_gather<uint32_t>(a, idx, n, static_cast<uint32_t*>(out), s);
  else queue_gather<uint64_t>(a, idx, n, static_cast<uint64_t*>(out), s);
  return hip_status(hipGetLastError());
}

}  // namespace gga
