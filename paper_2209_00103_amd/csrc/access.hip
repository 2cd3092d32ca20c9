// Size/prefix scan, shrink, regular read/write, flatten and bucket release.
//
// Regular access walks the LFVectors bucket by bucket (the per-block access rw_b
// of Sec. VI-B), but the work is cut into bucket-aligned tiles of at most 16 KiB,
// so the number of LFVectors and their uneven sizes do not set the parallelism.
// A tile lies inside one bucket and streams 16-byte vectors.  For an array (or a
// batch) of at least 2048 tiles the tiles are listed once per state of the sizes
// in a tile table and workgroups take table entries; smaller arrays and served
// steps spread the tiles over a persistent grid that locates its share by a
// search of the tile prefix.
#include <hip/hip_ext.h>

#include "gga_internal.h"

namespace gga {
namespace {

constexpr uint32_t kScanThreads = 1024;
// Persistent grids of the batched and served streaming kernels (256-thread
// workgroups; 256 CUs).  Measured on configuration 2 with the search-located
// shares: r/w peaks at 4096-8192 workgroups, flatten keeps gaining up to 65536
// (4.47 TB/s at 2048, 4.70 at 16384, 5.13 at 32768, 5.27 at 65536).
constexpr uint32_t kRwBlocks = 8192;
constexpr uint32_t kFlattenBlocks = 65536;
// Table-driven r/w and flatten of one array: one workgroup per tile, up to this
// many workgroups, looping beyond (configuration 2: flatten 5.33 -> 5.7 TB/s
// against the search-located persistent grid).
constexpr uint32_t kTableBlocks = 131072;
// Largest tile table kept per array (128 MiB, arrays up to 128 GiB of elements);
// a larger array walks its buckets instead.  Arrays the host knows to hold fewer
// than kTableMinTiles tiles (32 MiB of elements) walk their buckets too: for them
// the table's extra launch costs more than it saves.
constexpr uint64_t kTableMaxTiles = 1ull << 23;
constexpr uint64_t kTableMinTiles = 2048;

// Workgroups are dispatched round robin over the 8 XCDs, each with its own L2
// and address-translation caches.  A streaming grid is therefore a multiple of
// 8, and the workgroups of XCD x (those with b % 8 == x) take the x-th
// contiguous eighth of the tiles, striding by the number of workgroups per XCD:
// each XCD's caches then see one region of the tile table and of the buckets it
// lists (measured: configuration 2's r/w 5.72 -> 6.00 TB/s after a flatten and
// 5.58 -> 5.72 after an r/w; configuration 3's 1-2% faster).
inline uint32_t xcd_grid(uint64_t g) {
  g = (g + 7) & ~7ull;
  return (uint32_t)(g < 8 ? 8 : g);
}

struct TileSpan {
  uint64_t t, end, step;
};

__device__ __forceinline__ TileSpan xcd_span(uint64_t total) {
  const uint64_t G = gridDim.x;
  if (G & 7u) return {blockIdx.x, total, G};
  const uint64_t part = (total + 7) >> 3, x = blockIdx.x & 7u;
  const uint64_t end = (x + 1) * part < total ? (x + 1) * part : total;
  return {x * part + (blockIdx.x >> 3), end, G >> 3};
}

// Workgroups for one array's r/w or flatten: enough for the tiles the array can
// hold (the host's upper bound of its size), at most `cap`, so a small array
// does not pay for dispatching a grid sized for the largest ones.
inline uint32_t stream_grid(const ggarray* a, uint32_t cap) {
  const uint32_t te_log2 = 14u - a->elem_log2;
  const uint64_t g = (a->size_ub >> te_log2) + 2ull * a->V;
  return xcd_grid(g > cap ? cap : g);
}

typedef u32x4 u32x4_a4 __attribute__((aligned(4)));

// Exclusive prefix sums of the LFVector sizes (element offsets, Sec. IV) and of
// their tile counts, by one workgroup of kScanThreads; entry V holds the totals.
__device__ __forceinline__ void scan_array(const ArrRef& A, uint32_t te_log2, uint64_t* copy = nullptr) {
  __shared__ uint64_t wsum_e[kScanThreads / 64], wsum_t[kScanThreads / 64];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const uint32_t V = A.V;
  const uint32_t per = (V + kScanThreads - 1) / kScanThreads;
  const uint32_t v0 = tid * per < V ? tid * per : V;
  const uint32_t v1 = v0 + per < V ? v0 + per : V;
  uint64_t e = 0, t = 0;
  for (uint32_t v = v0; v < v1; ++v) {
    const uint64_t s = A.size[v];
    e += s;
    t += tiles_for(A.log2F, s, te_log2);
  }
  const uint64_t ie = wave_incl_scan64(e), it = wave_incl_scan64(t);
  if (lane == 63) {
    wsum_e[w] = ie;
    wsum_t[w] = it;
  }
  __syncthreads();
  uint64_t be = 0, bt = 0, te = 0, tt = 0;
  for (uint32_t k = 0; k < kScanThreads / 64; ++k) {
    if (k < w) {
      be += wsum_e[k];
      bt += wsum_t[k];
    }
    te += wsum_e[k];
    tt += wsum_t[k];
  }
  uint64_t re = be + ie - e, rt = bt + it - t;
  for (uint32_t v = v0; v < v1; ++v) {
    const uint64_t s = A.size[v];
    A.prefix[v] = re;
    if (copy) copy[v] = re;
    A.tprefix[v] = rt;
    re += s;
    rt += tiles_for(A.log2F, s, te_log2);
  }
  if (tid == 0) {
    A.prefix[V] = te;
    if (copy) copy[V] = te;
    A.tprefix[V] = tt;
  }
}

// `copy`, if not null, receives the V + 1 prefix entries too (ggarray_prefix).
__global__ __launch_bounds__(kScanThreads) void scan_kernel(ArrRef A, uint32_t te_log2, uint64_t* copy) {
  scan_array(A, te_log2, copy);
}

// The same prefix sums for many LFVectors, over many workgroups in two passes.
// Pass 1: workgroup c scans LFVectors [1024 c, 1024 c + 1024) (one per thread,
// coalesced), writes their prefixes within the chunk and the chunk's totals.
__global__ __launch_bounds__(kScanThreads) void scan_chunks_kernel(ArrRef A, uint64_t* tot, uint32_t te_log2) {
  __shared__ uint64_t wsum_e[kScanThreads / 64], wsum_t[kScanThreads / 64];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const uint32_t v = blockIdx.x * kScanThreads + tid;
  const uint64_t e = v < A.V ? A.size[v] : 0;
  const uint64_t t = tiles_for(A.log2F, e, te_log2);
  const uint64_t ie = wave_incl_scan64(e), it = wave_incl_scan64(t);
  if (lane == 63) {
    wsum_e[w] = ie;
    wsum_t[w] = it;
  }
  __syncthreads();
  uint64_t be = 0, bt = 0, ce = 0, ct = 0;
  for (uint32_t k = 0; k < kScanThreads / 64; ++k) {
    if (k < w) {
      be += wsum_e[k];
      bt += wsum_t[k];
    }
    ce += wsum_e[k];
    ct += wsum_t[k];
  }
  if (v < A.V) {
    A.prefix[v] = be + ie - e;
    A.tprefix[v] = bt + it - t;
  }
  if (tid == 0) {
    tot[2 * blockIdx.x] = ce;
    tot[2 * blockIdx.x + 1] = ct;
  }
}

// Pass 2: workgroup c adds the totals of the chunks before it; the last chunk's
// workgroup writes entry V.
__global__ __launch_bounds__(kScanThreads) void scan_fix_kernel(ArrRef A, const uint64_t* tot, uint32_t nchunks,
                                                             uint64_t* copy) {
  __shared__ uint64_t red_e[kScanThreads / 64], red_t[kScanThreads / 64];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  uint64_t e = 0, t = 0;
  for (uint32_t c = tid; c < blockIdx.x; c += kScanThreads) {
    e += tot[2 * c];
    t += tot[2 * c + 1];
  }
  e = wave_incl_scan64(e);
  t = wave_incl_scan64(t);
  if (lane == 63) {
    red_e[w] = e;
    red_t[w] = t;
  }
  __syncthreads();
  uint64_t oe = 0, ot = 0;
  for (uint32_t k = 0; k < kScanThreads / 64; ++k) {
    oe += red_e[k];
    ot += red_t[k];
  }
  const uint32_t v = blockIdx.x * kScanThreads + tid;
  if (v < A.V) {
    A.prefix[v] += oe;
    if (copy) copy[v] = A.prefix[v];
    A.tprefix[v] += ot;
  }
  if (blockIdx.x == nchunks - 1 && tid == 0) {
    A.prefix[A.V] = oe + tot[2 * blockIdx.x];
    if (copy) copy[A.V] = oe + tot[2 * blockIdx.x];
    A.tprefix[A.V] = ot + tot[2 * blockIdx.x + 1];
  }
}

constexpr uint32_t kVecPerBlock = 4;  // one wave per LFVector: 256 threads = 4 LFVectors

// kLanes lanes per LFVector.  A clear is a chain of dependent atomics per bucket.
// While a wave per LFVector fits the chip's 8192 wave slots it is the shortest; a
// few thousand LFVectors more come in turns, and four of them share a wave (V =
// 8192, 13 buckets: 19.6 -> 16.6 us).  Many more would be in flight together with those
// that share their free lists and retry each other's swaps: they release chains (below).
inline bool shrink_shares_wave(uint64_t V) { return V >= 4096; }
template <uint32_t kLanes>
__global__ __launch_bounds__(256) void shrink_kernel(ArrRef A, uint32_t num, uint32_t den,
                                                     uint32_t elem_log2) {
  const uint32_t v = (blockIdx.x * 256 + threadIdx.x) / kLanes;
  if (v < A.V) shrink_vector<kLanes>(A, v, num, den, elem_log2);
}

// The shrink of many LFVectors (more than the pool has free lists per class).  Every
// 4096th LFVector's bucket b goes to the same free list, so 16 lanes take residue r:
// lane l links bucket l (then l + 16, ...) of LFVectors r, r + 4096, ..., 16 at a
// time, into one chain and pushes it with one swap of the list's head.  One swap per
// bucket makes the LFVectors of a list wait for each other (V = 65536, 2 and 4
// buckets, a wave per LFVector: 47 and 57 us; 24 and 31 us this way).  What is left
// is the serial chain: sizes, pointers, links, swap, each one trip to memory.  With
// fewer LFVectors there is little to link (V = 16384, 2 buckets: 21.8 us with 16 lanes
// per LFVector, 16.0 us this way; V = 8192, 6 buckets: 18.2 us either way).
constexpr uint32_t kChainLanes = 16;
constexpr uint64_t kChainStep = (uint64_t)kFreeShards * kChainLanes;

__device__ __forceinline__ uint64_t exchange_link(uint8_t* block, uint64_t next) {
  return __hip_atomic_exchange(gmem(reinterpret_cast<uint64_t*>(block)), next, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
}

// n > 0 linked blocks of class cls, the top one's index word `first`, go to free list
// f; every link but the last has landed.
__device__ __forceinline__ void push_chain(PoolHdr* H, uint32_t cls, uint32_t f, uint64_t first, uint8_t* last,
                                           uint32_t n) {
  uint64_t* const head = &H->heads[(uint64_t)cls * kFreeShards + f];
  uint64_t h = ld_rlx(head);
  for (;;) {
    asm volatile("" ::"v"(exchange_link(last, h & kIdxMask)) : "memory");
    if (cas_rlx(head, h, (((h >> 40) + 1) << 40) | first)) break;
  }
  if ((h & kIdxMask) == 0)
    __hip_atomic_fetch_or(&H->nonempty[cls][f >> 6], 1ull << (f & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  sub_nr(&free_stat(H)->in_use, (uint64_t)n << cls);
  add_nr(&free_stat(H)->n_free, (uint64_t)n);
}

// Buckets [lo, hi) of LFVector v are to go, as lo << 8 | hi (0: none, also for !in).
__device__ __forceinline__ uint32_t shrink_range(const ArrRef& A, uint64_t v, uint32_t num, uint32_t den, bool in) {
  uint32_t dead = A.dead[v];
  uint64_t s = A.size[v];
  asm volatile("" : "+v"(dead), "+v"(s));  // both loads in flight before either is looked at
  const uint32_t hi = dead ? (uint32_t)kMaxBuckets : nbuckets_for(A.log2F, s);
  const uint32_t lo = nbuckets_for(A.log2F, shrink_keep(s, num, den));
  return in ? lo << 8 | (hi < (uint32_t)kMaxBuckets ? hi : (uint32_t)kMaxBuckets) : 0;
}

__device__ __forceinline__ uint32_t shrink_range_at(const ArrRef& A, uint64_t v, uint32_t num, uint32_t den) {
  return shrink_range(A, v < A.V ? v : 0, num, den, v < A.V);
}

__global__ __launch_bounds__(256) void shrink_chain_kernel(ArrRef A, uint32_t num, uint32_t den, uint32_t elem_log2) {
  const uint32_t l = threadIdx.x & (kChainLanes - 1);
  const uint64_t r = ((uint64_t)blockIdx.x * 256 + threadIdx.x) / kChainLanes;
  if (r >= (uint64_t)kFreeShards || r >= A.V) return;
  uint32_t range = 0, most = 0;  // most: buckets of the residue's longest LFVector
  for (uint64_t v0 = r; v0 < A.V; v0 += kChainStep) {
    range = shrink_range_at(A, v0 + (uint64_t)l * kFreeShards, num, den);
    most = (range & 255u) > most ? range & 255u : most;
  }
#pragma unroll
  for (uint32_t d = 1; d < kChainLanes; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_xor((int)most, (int)d, (int)kChainLanes);
    most = o > most ? o : most;
  }
  for (uint32_t b0 = 0; b0 < most; b0 += kChainLanes) {
    const uint32_t b = b0 + l;
    uint64_t* const row = A.bptr + (b < (uint32_t)kMaxBuckets ? b : 0);
    uint64_t first = 0;  // index word of the chain's top block
    uint32_t n = 0;
    uint8_t* last = nullptr;
    for (uint64_t v0 = r; v0 < A.V; v0 += kChainStep) {
      if (A.V > kChainStep) range = shrink_range_at(A, v0 + (uint64_t)l * kFreeShards, num, den);
      uint64_t p[kChainLanes];
#pragma unroll
      for (uint32_t u = 0; u < kChainLanes; ++u) {
        const uint64_t v = v0 + u * kFreeShards;
        p[u] = row[(v < A.V ? v : r) * kMaxBuckets];
      }
#pragma unroll
      for (uint32_t u = 0; u < kChainLanes; ++u) {
        asm volatile("" : "+v"(p[u]));  // all of them in flight before the first is looked at
        const uint32_t g = (uint32_t)__shfl((int)range, (int)u, (int)kChainLanes);
        if (b < (g >> 8) || b >= (g & 255u)) p[u] = 0;
      }
      uint64_t landed[kChainLanes];  // what the links' exchanges returned
#pragma unroll
      for (uint32_t u = 0; u < kChainLanes; ++u) {
        landed[u] = 0;
        if (p[u] == 0) continue;
        row[(v0 + u * kFreeShards) * kMaxBuckets] = 0;
        if (p[u] <= kFailedPtr) continue;
        uint8_t* const block = reinterpret_cast<uint8_t*>(p[u]);
        const uint64_t idx = ((uint64_t)(block - A.pool.base) >> kMinClassLog2) + 1;
        if (n)
          landed[u] = exchange_link(last, idx);
        else
          first = idx;
        last = block;
        ++n;
      }
      // Consuming the results makes the wave wait until every link has landed before
      // the swap below can publish the chain.
#pragma unroll
      for (uint32_t u = 0; u < kChainLanes; ++u) asm volatile("" ::"v"(landed[u]) : "memory");
    }
    if (n == 0) continue;
    push_chain(A.pool.hdr, bucket_class(A.log2F, elem_log2, b), pool_shard((uint32_t)r, b, A.salt), first, last, n);
  }
  // Every lane of the residue has read the old sizes: one wave, program order.
  for (uint64_t v = r + (uint64_t)l * kFreeShards; v < A.V; v += kChainStep)
    A.size[v] = shrink_keep(A.size[v], num, den);
}
constexpr uint64_t kChainMinV = 16384;

// The same for a batch.  Arrays created in a row take consecutive free lists, so every
// 4096th LFVector of such a batch shares its lists too, as long as first bucket and
// element size agree; where sixteen of them do not (other first buckets, an array
// between them that is not in the batch, several pools) their blocks are released one by
// one (81224 LFVectors of 512 arrays: 101 us as a wave each, 42 us; 30 and 8 us when
// nothing is held).
struct ShrinkItem {  // LFVector w of the batch, held by one lane
  uint64_t* row;
  uint8_t* base;
  PoolHdr* hdr;
  uint32_t list;   // log2 of the first bucket's bytes << 12 | its free list
  uint32_t range;  // shrink_range
};
__device__ __forceinline__ ShrinkItem shrink_item(const BatchArr* items, const uint64_t* vbegin, const uint32_t* varr,
                                                  uint64_t w, uint64_t total, uint32_t num, uint32_t den) {
  const bool in = w < total;
  if (!in) w = 0;
  const uint32_t i = varr[w];
  const ArrRef& A = items[i].A;
  const uint32_t v = (uint32_t)(w - vbegin[i]);
  return ShrinkItem{A.bptr + (uint64_t)v * kMaxBuckets, A.pool.base, A.pool.hdr,
                    (A.log2F + items[i].elem_log2) << 12 | pool_shard(v, 0, A.salt),
                    shrink_range(A, v, num, den, in)};
}

__global__ __launch_bounds__(256) void batch_shrink_chain_kernel(const BatchArr* items, const uint64_t* vbegin,
                                                                 const uint32_t* varr, uint64_t total, uint32_t num,
                                                                 uint32_t den) {
  const uint32_t l = threadIdx.x & (kChainLanes - 1);
  const uint64_t r = ((uint64_t)blockIdx.x * 256 + threadIdx.x) / kChainLanes;
  if (r >= (uint64_t)kFreeShards || r >= total) return;
  ShrinkItem it{};
  uint32_t most = 0;
  for (uint64_t w0 = r; w0 < total; w0 += kChainStep) {
    it = shrink_item(items, vbegin, varr, w0 + (uint64_t)l * kFreeShards, total, num, den);
    most = (it.range & 255u) > most ? it.range & 255u : most;
  }
#pragma unroll
  for (uint32_t d = 1; d < kChainLanes; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_xor((int)most, (int)d, (int)kChainLanes);
    most = o > most ? o : most;
  }
  for (uint32_t b0 = 0; b0 < most; b0 += kChainLanes) {
    const uint32_t b = b0 + l, bb = b < (uint32_t)kMaxBuckets ? b : 0;
    uint64_t first = 0;
    uint32_t n = 0, list = 0;  // of the chain
    PoolHdr* hdr = nullptr;
    uint8_t* last = nullptr;
    for (uint64_t w0 = r; w0 < total; w0 += kChainStep) {
      if (total > kChainStep) it = shrink_item(items, vbegin, varr, w0 + (uint64_t)l * kFreeShards, total, num, den);
      uint64_t p[kChainLanes];
#pragma unroll
      for (uint32_t u = 0; u < kChainLanes; ++u)
        p[u] = reinterpret_cast<const uint64_t*>(__shfl((uint64_t)it.row, (int)u, (int)kChainLanes))[bb];
#pragma unroll
      for (uint32_t u = 0; u < kChainLanes; ++u) {
        asm volatile("" : "+v"(p[u]));
        uint64_t* const slot = reinterpret_cast<uint64_t*>(__shfl((uint64_t)it.row, (int)u, (int)kChainLanes)) + bb;
        const uint32_t g = (uint32_t)__shfl((int)it.range, (int)u, (int)kChainLanes);
        if (b < (g >> 8) || b >= (g & 255u)) p[u] = 0;
        if (p[u]) *slot = 0;
        if (p[u] <= kFailedPtr) p[u] = 0;
      }
      const uint32_t list0 = (uint32_t)__shfl((int)it.list, 0, (int)kChainLanes);
      uint8_t* const base = reinterpret_cast<uint8_t*>(__shfl((uint64_t)it.base, 0, (int)kChainLanes));
      PoolHdr* const hdr0 = reinterpret_cast<PoolHdr*>(__shfl((uint64_t)it.hdr, 0, (int)kChainLanes));
      const uint64_t odd = __ballot(it.range && (it.list != list0 || it.hdr != hdr0));
      const bool one = ((odd >> (threadIdx.x & 48u)) & 0xFFFFull) == 0;
      if (n && (!one || list != list0 || hdr != hdr0)) {
        push_chain(hdr, bucket_class(list >> 12, 0, b), pool_shard(list, b, 0), first, last, n);
        n = 0;
      }
      if (one) {
        list = list0;
        hdr = hdr0;
        uint64_t landed[kChainLanes];
#pragma unroll
        for (uint32_t u = 0; u < kChainLanes; ++u) {
          landed[u] = 0;
          if (p[u] == 0) continue;
          uint8_t* const block = reinterpret_cast<uint8_t*>(p[u]);
          const uint64_t idx = ((uint64_t)(block - base) >> kMinClassLog2) + 1;
          if (n)
            landed[u] = exchange_link(last, idx);
          else
            first = idx;
          last = block;
          ++n;
        }
#pragma unroll
        for (uint32_t u = 0; u < kChainLanes; ++u) asm volatile("" ::"v"(landed[u]) : "memory");
      } else {
#pragma unroll 1
        for (uint32_t u = 0; u < kChainLanes; ++u) {
          const uint64_t q = p[0];
#pragma unroll
          for (uint32_t k = 0; k + 1 < kChainLanes; ++k) p[k] = p[k + 1];
          const uint32_t lu = (uint32_t)__shfl((int)it.list, (int)u, (int)kChainLanes);
          PoolRef P{};
          P.base = reinterpret_cast<uint8_t*>(__shfl((uint64_t)it.base, (int)u, (int)kChainLanes));
          P.hdr = reinterpret_cast<PoolHdr*>(__shfl((uint64_t)it.hdr, (int)u, (int)kChainLanes));
          if (q)
            pool_free(P, reinterpret_cast<uint8_t*>(q), bucket_class(lu >> 12, 0, b), pool_shard(lu, b, 0));
        }
      }
    }
    if (n) push_chain(hdr, bucket_class(list >> 12, 0, b), pool_shard(list, b, 0), first, last, n);
  }
  for (uint64_t w = r + (uint64_t)l * kFreeShards; w < total; w += kChainStep) {
    const uint32_t i = varr[w];
    uint64_t* const size = items[i].A.size + (w - vbegin[i]);
    *size = shrink_keep(*size, num, den);
  }
}

// Returns every bucket of the array to the pool (destroy).
__global__ __launch_bounds__(256) void free_all_kernel(ArrRef A, uint32_t elem_log2) {
  const uint32_t v = blockIdx.x * kVecPerBlock + (threadIdx.x >> 6);
  const uint32_t b = threadIdx.x & 63u;
  if (v >= A.V || b >= (uint32_t)kMaxBuckets) return;
  uint64_t* slot = A.bptr + (uint64_t)v * kMaxBuckets + b;
  const uint64_t p = *slot;
  if (p > kFailedPtr)
    pool_free(A.pool, reinterpret_cast<uint8_t*>(p), bucket_class(A.log2F, elem_log2, b), pool_shard(v, b, A.salt));
  *slot = 0;
}

// Elements held by allocated buckets.
__global__ void capacity_kernel(ArrRef A, uint64_t* out) {
  const uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= A.V) return;
  const uint64_t* row = A.bptr + (uint64_t)v * kMaxBuckets;
  uint64_t c = 0;
  for (uint32_t b = 0; b < (uint32_t)kMaxBuckets; ++b)
    if (row[b] > kFailedPtr) c += bucket_len(A.log2F, b);
  if (c) fetch_add(out, c);
}

// The words that a synchronising call returns, straight into the array's pinned
// host memory: *word (if any) and the sticky error.
__global__ void report_kernel(const uint64_t* word, const uint32_t* err, uint64_t* host) {
  if (word) host[0] = *word;
  host[1] = *err;
}

// One tile: cnt (<= te) elements at src (16-byte aligned); rw in place, or copy
// to dst (element aligned) for flatten.  Lane i of slot k handles the 16 bytes
// at element k * (256 * VPL) + i * VPL.  Every byte is touched once, so stores
// are non-temporal; so are flatten's loads, while r/w loads through the cache,
// which lets its non-temporal stores find the lines they overwrite (measured:
// r/w 4.80 -> 5.31 TB/s, flatten slower with cached loads).  Neither carries the
// device-scope bit that the insertion's stores do: with it r/w measured 5.0
// TB/s, and flatten gained 1.5% on configuration 2 but slowed the batched step
// that follows it by 3%.
template <typename T, bool kFlatten, bool kNtLoad = kFlatten>
__device__ __forceinline__ void stream_tile(T* src_, T* dst_, uint32_t cnt, uint32_t op) {
  const gptr<T> src = gmem(src_), dst = gmem(dst_);
  constexpr uint32_t VPL = 16 / sizeof(T);
  constexpr uint32_t kSlots = 4;
  constexpr uint32_t kSpan = kRwThreads * VPL;
  const uint32_t tid = threadIdx.x;
  if (kFlatten) {
    // A destination that is not 128-byte aligned: stage the tile in LDS (aligned
    // loads), then write the destination in whole 128-byte lines, each store
    // instruction of a wave covering complete lines (flatten 4.51 -> 4.70 TB/s;
    // taking the misalignment on the global loads instead was slower).
    __shared__ u32x4 stage[kSlots * kRwThreads];
    const uint32_t mis = (uint32_t)((reinterpret_cast<uintptr_t>(dst_) & 127u) / sizeof(T));
    if (mis) {
      const uint32_t nsrc = (cnt + VPL - 1) / VPL;
      for (uint32_t k = 0; k < kSlots; ++k) {
        const uint32_t q = k * kRwThreads + tid;
        if (q < nsrc) {
          if ((q + 1) * VPL <= cnt)
            stage[q] = __builtin_nontemporal_load(reinterpret_cast<gptr<const u32x4>>(src + q * VPL));
          else {
            T tmp[VPL] = {};
            for (uint32_t e = 0; e < VPL && q * VPL + e < cnt; ++e) tmp[e] = src[q * VPL + e];
            u32x4 x;
            __builtin_memcpy(&x, tmp, 16);
            stage[q] = x;
          }
        }
      }
      __syncthreads();
      const T* st = reinterpret_cast<const T*>(stage);
      const gptr<T> dal = dst - mis;
      const uint32_t nvec = (cnt + mis + VPL - 1) / VPL;
      for (uint32_t j = tid; j < nvec; j += kRwThreads) {
        const int64_t e0 = (int64_t)j * VPL - (int64_t)mis;
        if (e0 >= 0 && e0 + (int64_t)VPL <= (int64_t)cnt) {
          T tmp[VPL];
          for (uint32_t e = 0; e < VPL; ++e) tmp[e] = st[e0 + e];
          u32x4 x;
          __builtin_memcpy(&x, tmp, 16);
          __builtin_nontemporal_store(x, reinterpret_cast<gptr<u32x4>>(dal + (uint64_t)j * VPL));
        } else {
          for (uint32_t e = 0; e < VPL; ++e) {
            const int64_t i = e0 + e;
            if (i >= 0 && i < (int64_t)cnt) dst[i] = st[i];
          }
        }
      }
      __syncthreads();
      return;
    }
  }
  if (cnt == kSlots * kSpan) {
    u32x4 r[kSlots];
#pragma unroll
    for (uint32_t k = 0; k < kSlots; ++k)
      r[k] = kNtLoad ? __builtin_nontemporal_load(reinterpret_cast<gptr<const u32x4>>(src + k * kSpan + tid * VPL))
                      : *reinterpret_cast<gptr<const u32x4>>(src + k * kSpan + tid * VPL);
#pragma unroll
    for (uint32_t k = 0; k < kSlots; ++k) {
      if (kFlatten)
        __builtin_nontemporal_store(r[k], reinterpret_cast<gptr<u32x4_a4>>(dst + k * kSpan + tid * VPL));
      else
        __builtin_nontemporal_store(op_vec<T>(op, r[k]), reinterpret_cast<gptr<u32x4>>(src + k * kSpan + tid * VPL));
    }
    return;
  }
  for (uint32_t k = 0; k < kSlots; ++k) {
    const uint32_t e = k * kSpan + tid * VPL;
    if (e + VPL <= cnt) {
      const u32x4 x = kNtLoad ? __builtin_nontemporal_load(reinterpret_cast<gptr<const u32x4>>(src + e))
                               : *reinterpret_cast<gptr<const u32x4>>(src + e);
      if (kFlatten)
        __builtin_nontemporal_store(x, reinterpret_cast<gptr<u32x4_a4>>(dst + e));
      else
        __builtin_nontemporal_store(op_vec<T>(op, x), reinterpret_cast<gptr<u32x4>>(src + e));
    } else {
      for (uint32_t q = e; q < cnt && q < e + VPL; ++q) {
        if (kFlatten)
          dst[q] = src[q];
        else
          src[q] = apply_op<T>(op, src[q]);
      }
    }
  }
}

// The LFVector of tile t < tprefix[V] (the last one whose tiles start at or before
// t).  LFVectors of one length put it at t's share of V, so that place is looked at
// first, and only then is one side of it searched: nine dependent loads of a binary search at V = 512 are most of a
// small array's r/w (2 MiB over 256 LFVectors: 6.5 -> 5.4 us).
__device__ __forceinline__ uint32_t vector_of_tile(const ArrRef& A, uint64_t t) {
  const uint32_t V = A.V;
  const uint64_t total = A.tprefix[V];
  const uint32_t g = (uint32_t)((float)t * ((float)V / (float)total));  // a guess: any rounding will do
  uint32_t lo = g < V ? g : V - 1, hi = lo + 1;
  const uint64_t a = A.tprefix[lo], b = A.tprefix[hi];
  if (a <= t && t < b) return lo;
  if (a > t) {
    hi = lo;
    lo = 0;
  } else {
    lo = hi;
    hi = V;
  }
  while (hi - lo > 1) {  // tprefix[lo] <= t < tprefix[hi]
    const uint32_t mid = (lo + hi) >> 1;
    if (A.tprefix[mid] <= t) lo = mid; else hi = mid;
  }
  return lo;
}

// Walk over the bucket-aligned tiles [t0, t1) of one array: find the first
// LFVector by binary search over the tile prefix, then walk forward; the bucket
// pointer and the destination offset are reloaded only when the walk enters a
// new bucket.
template <typename T, bool kFlatten>
__device__ __forceinline__ void stream_range(const ArrRef& A, uint64_t t0, uint64_t t1, uint32_t op,
                                             T* out, uint32_t te_log2) {
  const uint32_t V = A.V;
  if (t0 >= t1) return;
  uint32_t v = vector_of_tile(A, t0);
  uint64_t s = A.size[v];
  uint64_t k = t0 - A.tprefix[v];
  const uint32_t log2F = A.log2F;
  const uint64_t te = 1ull << te_log2;
  uint32_t b = 0;
  uint64_t live, nt;
  for (;;) {
    live = bucket_len(log2F, b);
    const uint64_t st = bucket_start(log2F, b);
    if (s - st < live) live = s - st;
    nt = (live + te - 1) >> te_log2;
    if (k < nt) break;
    k -= nt;
    ++b;
  }
  T* bucket = reinterpret_cast<T*>(A.bptr[(uint64_t)v * kMaxBuckets + b]);
  T* dbase = kFlatten ? out + A.prefix[v] + bucket_start(log2F, b) : nullptr;
  for (uint64_t t = t0;;) {
    const uint64_t e0 = k << te_log2;
    const uint64_t rem = live - e0;
    const uint32_t cnt = (uint32_t)(rem < te ? rem : te);
    stream_tile<T, kFlatten>(bucket + e0, kFlatten ? dbase + e0 : nullptr, cnt, op);
    if (++t >= t1) break;
    if (++k == nt) {
      k = 0;
      ++b;
      if (bucket_start(log2F, b) >= s) {
        b = 0;
        do {
          ++v;
          s = A.size[v];
        } while (s == 0);
      }
      live = bucket_len(log2F, b);
      const uint64_t st = bucket_start(log2F, b);
      if (s - st < live) live = s - st;
      nt = (live + te - 1) >> te_log2;
      bucket = reinterpret_cast<T*>(A.bptr[(uint64_t)v * kMaxBuckets + b]);
      if (kFlatten) dbase = out + A.prefix[v] + st;
    }
  }
}

// Tile table of one array, built once per state of the sizes (after the prefix
// scan): tile t, in the order of the tile prefix, gets the address of its first
// element and its destination offset in a flatten, with its element count in the
// top 16 bits.  kLanes lanes per LFVector, over the tiles of each bucket; they read the
// bucket table's first kLanes entries at once, beside the size and the prefixes.
// Entries from `cap` on are not written; the streaming kernels then walk the
// buckets instead.
template <uint32_t kLanes>
__device__ __forceinline__ uint64_t table_entry(const ArrRef& A, uint32_t v) {
  const uint32_t lane = threadIdx.x & (kLanes - 1);
  return A.bptr[(uint64_t)v * kMaxBuckets + (lane < (uint32_t)kMaxBuckets ? lane : 0)];
}
// LFVector v of s elements; its first tile is t, its first element's place pv, the lane's
// entry of its bucket table `mine`.
template <uint32_t kLanes>
__device__ __forceinline__ void vector_tiles(const ArrRef& A, uint32_t v, uint64_t s, uint64_t* tab, uint64_t cap,
                                             uint32_t te_log2, uint32_t elem_log2, uint64_t t, uint64_t pv,
                                             uint64_t mine) {
  const uint32_t lane = threadIdx.x & (kLanes - 1);
  const uint64_t* row = A.bptr + (uint64_t)v * kMaxBuckets;
  const uint32_t log2F = A.log2F;
  const uint64_t te = 1ull << te_log2;
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  for (uint32_t b = 0; b < (uint32_t)kMaxBuckets; ++b) {
    const uint64_t st = bucket_start(log2F, b);
    if (st >= s) break;
    uint64_t live = bucket_len(log2F, b);
    if (s - st < live) live = s - st;
    const uint64_t nt = (live + te - 1) >> te_log2;
    const uint64_t base = b < kLanes ? __shfl(mine, (int)b, (int)kLanes) : row[b];
    for (uint64_t i = lane; i < nt; i += kLanes) {
      const uint64_t e0 = i << te_log2;
      const uint64_t cnt = live - e0 < te ? live - e0 : te;
      if (t + i < cap) {
        const u64x2 d = {base + (e0 << elem_log2), (pv + st + e0) | (cnt << 48)};
        gmem(reinterpret_cast<u64x2*>(tab))[t + i] = d;
      }
    }
    t += nt;
  }
}

// An LFVector for the tile table: of array A, with the table's and the flatten's place
// of that array's first tile and element.
struct TableItem {
  const ArrRef* A;
  uint32_t v, elem_log2;
  uint64_t tile, elem;
};

// Tiles of LFVector w (of `total`) by kLanes lanes; item(w) says where it is.  One of
// more than kLongTiles tiles is left to its whole wave (with sixteen lanes of it for the
// one long LFVector of 16384, 2^28 u32 elements, table and r/w took 759 us, 495 this way).
constexpr uint64_t kLongTiles = 256;
template <uint32_t kLanes, class Item>
__device__ __forceinline__ void table_vector(Item item, uint64_t w, uint64_t total, uint64_t* tab, uint64_t cap,
                                             uint32_t te_log2) {
  const bool in = w < total;
  const TableItem it = item(in ? w : 0);
  const uint64_t s = it.A->size[it.v], t = it.tile + it.A->tprefix[it.v], e = it.elem + it.A->prefix[it.v];
  const uint64_t mine = table_entry<kLanes>(*it.A, it.v);
  const bool whole = kLanes < 64 && s >> te_log2 > kLongTiles;
  if (in && !whole) vector_tiles<kLanes>(*it.A, it.v, s, tab, cap, te_log2, it.elem_log2, t, e, mine);
  if constexpr (kLanes < 64) {
    for (uint64_t m = __ballot(in && whole && (threadIdx.x & (kLanes - 1)) == 0); m; m &= m - 1) {
      const int l = __ffsll((unsigned long long)m) - 1;
      const TableItem long_it = item(__shfl(w, l, 64));
      vector_tiles<64>(*long_it.A, long_it.v, __shfl(s, l, 64), tab, cap, te_log2, long_it.elem_log2,
                       __shfl(t, l, 64), __shfl(e, l, 64), table_entry<64>(*long_it.A, long_it.v));
    }
  }
}

// The prefix scan and the tile table in one launch (up to 4 * kScanThreads
// LFVectors): every workgroup sums the sizes and tiles of the LFVectors before its
// own, which the caches serve after the first, and writes the prefix entries and
// the tiles of its own (V = 512: 5.8 us, against 4.8 each as two launches).
__global__ __launch_bounds__(256) void scan_table_kernel(ArrRef A, uint64_t* copy, uint64_t* tab, uint64_t cap,
                                                         uint32_t te_log2, uint32_t elem_log2) {
  __shared__ uint64_t red_e[4], red_t[4];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const uint32_t v0 = blockIdx.x * kVecPerBlock;
  uint64_t e = 0, t = 0;
  for (uint32_t v = tid; v < v0; v += 256) {
    const uint64_t s = A.size[v];
    e += s;
    t += tiles_for(A.log2F, s, te_log2);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    e += __shfl_xor(e, d, 64);
    t += __shfl_xor(t, d, 64);
  }
  if (lane == 0) {
    red_e[w] = e;
    red_t[w] = t;
  }
  __syncthreads();
  e = red_e[0] + red_e[1] + red_e[2] + red_e[3];
  t = red_t[0] + red_t[1] + red_t[2] + red_t[3];
  const uint32_t v = v0 + w;
  for (uint32_t u = v0; u < v && u < A.V; ++u) {  // the workgroup's LFVectors before this wave's
    const uint64_t s = A.size[u];
    e += s;
    t += tiles_for(A.log2F, s, te_log2);
  }
  if (v >= A.V) return;
  const uint64_t s = A.size[v], mine = table_entry<64>(A, v);
  if (lane == 0) {
    A.prefix[v] = e;
    A.tprefix[v] = t;
    if (copy) copy[v] = e;
    if (v == A.V - 1) {
      A.prefix[A.V] = e + s;
      A.tprefix[A.V] = t + tiles_for(A.log2F, s, te_log2);
      if (copy) copy[A.V] = e + s;
    }
  }
  vector_tiles<64>(A, v, s, tab, cap, te_log2, elem_log2, t, e, mine);
}

// A wave per LFVector is as short while the waves fit the chip's wave slots at once; from
// 16384 LFVectors on sixteen lanes each are (us, 64 against 16 lanes: V = 16384 8-10 and
// 5, V = 65536 with 2 buckets 17 and 7, with 4 buckets 24 and 8.5, V = 131072 40 and
// 13; V = 12000 5.4 as a wave).
constexpr uint64_t kTableSharedMinV = 16384;
template <uint32_t kLanes>
__global__ __launch_bounds__(256) void tile_table_kernel(ArrRef A, uint64_t* tab, uint64_t cap, uint32_t te_log2,
                                                         uint32_t elem_log2) {
  const auto item = [&](uint64_t v) { return TableItem{&A, (uint32_t)v, elem_log2, 0, 0}; };
  table_vector<kLanes>(item, ((uint64_t)blockIdx.x * 256 + threadIdx.x) / kLanes, A.V, tab, cap, te_log2);
}

// The tile table of a batch: the tiles of array i follow those of arrays before
// it (tile_begin), and destination offsets are positions in the batch flatten
// (elem_begin).  Group w of kLanes lanes is LFVector w - vbegin[i] of array i = varr[w].
template <uint32_t kLanes>
__global__ __launch_bounds__(256) void batch_table_kernel(const BatchArr* items, const uint64_t* vbegin,
                                                          const uint32_t* varr, const uint64_t* tile_begin,
                                                          const uint64_t* elem_begin, uint64_t total, uint64_t* tab,
                                                          uint64_t cap, uint32_t te_log2) {
  const auto item = [&](uint64_t w) {
    const uint32_t i = varr[w];
    return TableItem{&items[i].A, (uint32_t)(w - vbegin[i]), items[i].elem_log2, tile_begin[i], elem_begin[i]};
  };
  table_vector<kLanes>(item, ((uint64_t)blockIdx.x * 256 + threadIdx.x) / kLanes, total, tab, cap, te_log2);
}

// Load policy of r/w.  Non-temporal loads (kNtLoad) serve an r/w that directly
// follows another r/w of the array (configuration 2: 5.3 against 4.9 TB/s) and
// every r/w of at least kNtLoadBytes of elements; a smaller array read after an
// insertion or a flatten loads through the cache.  Measured on single arrays
// (u32, V = 512, r/w after an insertion), cached against non-temporal loads:
// 6.07 against 5.27 TB/s at 0.54 GB, 5.74 against 5.59 at 1.07 GB, 5.68 against
// 5.78 at 2.15 GB and 5.41 against 5.56 at 4.29 GB; configuration 4's batch
// (3.84 GB of buckets of at most 64 KiB) 4.40 against 4.70 TB/s.
constexpr uint64_t kNtLoadBytes = 5ull << 28;  // 1.25 GiB

// Tiles [sp.t, sp.end) of a tile table, stride sp.step.
template <typename T, bool kFlatten, bool kNtLoad>
__device__ __forceinline__ void table_tiles(const uint64_t* __restrict__ tab, const TileSpan& sp, uint32_t op,
                                            T* out) {
  for (uint64_t t = sp.t; t < sp.end; t += sp.step) {
    const uint64_t src = tab[2 * t], w = tab[2 * t + 1];
    stream_tile<T, kFlatten, kNtLoad>(reinterpret_cast<T*>(src), kFlatten ? out + (w & 0xFFFFFFFFFFFFull) : nullptr,
                                      (uint32_t)(w >> 48), op);
  }
}

// r/w or flatten of one array through its tile table: each XCD's workgroups
// stride over their eighth of the tiles (one tile each when the grid covers the
// array).  Without a table for the current state (more tiles than it holds) the
// grid walks the buckets.
template <typename T, bool kFlatten, bool kNtLoad = kFlatten>
__global__ __launch_bounds__(kRwThreads) void stream_table_kernel(ArrRef A, const uint64_t* __restrict__ tab,
                                                                 uint64_t cap, uint32_t op, T* out,
                                                                 uint64_t out_cap, uint32_t te_log2) {
  const uint64_t total = A.tprefix[A.V];
  if (kFlatten && A.prefix[A.V] > out_cap) {
    if (blockIdx.x == 0 && threadIdx.x == 0) set_error(A.err, kErrRange);
    return;
  }
  const uint64_t G = gridDim.x;
  if (total > cap) {
    stream_range<T, kFlatten>(A, total * blockIdx.x / G, total * (blockIdx.x + 1) / G, op, out, te_log2);
    return;
  }
  const TileSpan sp = xcd_span(total);
  if (!kFlatten && !kNtLoad && A.prefix[A.V] * sizeof(T) >= kNtLoadBytes)
    table_tiles<T, false, true>(tab, sp, op, out);
  else
    table_tiles<T, kFlatten, kNtLoad>(tab, sp, op, out);
}

// Static / semi-static array r/w: the flat array cut into 16 KiB tiles, workgroup
// w streaming tiles w, w + G, ... (the GGArray's tile size and load policy
// without the bucket indirection).  A contiguous array streams faster in this
// plain order than with the GGArray's split of the tiles over the XCDs
// (configuration 2's static r/w 6.35 against 6.07 TB/s), so it keeps it.
template <typename T, bool kNtLoad>
__global__ __launch_bounds__(kRwThreads) void static_rw_kernel(T* data, const uint64_t* size,
                                                              uint64_t cap, uint32_t op, uint32_t te_log2) {
  uint64_t n = *size;
  if (n > cap) n = cap;
  const uint64_t te = 1ull << te_log2;
  const uint64_t total = (n + te - 1) >> te_log2;
  const TileSpan sp{blockIdx.x, total, gridDim.x};
  if (!kNtLoad && n * sizeof(T) >= kNtLoadBytes) {
    for (uint64_t t = sp.t; t < sp.end; t += sp.step) {
      const uint64_t e0 = t << te_log2;
      const uint64_t rem = n - e0;
      stream_tile<T, false, true>(data + e0, nullptr, (uint32_t)(rem < te ? rem : te), op);
    }
    return;
  }
  for (uint64_t t = sp.t; t < sp.end; t += sp.step) {
    const uint64_t e0 = t << te_log2;
    const uint64_t rem = n - e0;
    stream_tile<T, false, kNtLoad>(data + e0, nullptr, (uint32_t)(rem < te ? rem : te), op);
  }
}


// ----------------------------------------------------------------- batches --
// One workgroup per array of the batch: its own prefix sums.
__global__ __launch_bounds__(kScanThreads) void batch_scan_kernel(const BatchArr* items, uint32_t te_log2) {
  scan_array(items[blockIdx.x].A, te_log2);
}

// Exclusive prefix over the arrays of their tile counts and sizes (entry n holds
// the totals), by one workgroup.
template <class Item>
__global__ __launch_bounds__(kScanThreads) void batch_top_kernel(const Item* items, uint32_t n,
                                                                uint64_t* tile_begin, uint64_t* elem_begin) {
  __shared__ uint64_t wsum_e[kScanThreads / 64], wsum_t[kScanThreads / 64];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const uint32_t per = (n + kScanThreads - 1) / kScanThreads;
  const uint32_t i0 = tid * per < n ? tid * per : n;
  const uint32_t i1 = i0 + per < n ? i0 + per : n;
  uint64_t e = 0, t = 0;
  for (uint32_t i = i0; i < i1; ++i) {
    e += items[i].A.prefix[items[i].A.V];
    t += items[i].A.tprefix[items[i].A.V];
  }
  const uint64_t ie = wave_incl_scan64(e), it = wave_incl_scan64(t);
  if (lane == 63) {
    wsum_e[w] = ie;
    wsum_t[w] = it;
  }
  __syncthreads();
  uint64_t be = 0, bt = 0, te = 0, tt = 0;
  for (uint32_t k = 0; k < kScanThreads / 64; ++k) {
    if (k < w) {
      be += wsum_e[k];
      bt += wsum_t[k];
    }
    te += wsum_e[k];
    tt += wsum_t[k];
  }
  uint64_t re = be + ie - e, rt = bt + it - t;
  for (uint32_t i = i0; i < i1; ++i) {
    elem_begin[i] = re;
    tile_begin[i] = rt;
    re += items[i].A.prefix[items[i].A.V];
    rt += items[i].A.tprefix[items[i].A.V];
  }
  if (tid == 0) {
    elem_begin[n] = te;
    tile_begin[n] = tt;
  }
}

// Shrink of every array of the batch, kLanes lanes per LFVector as for one array;
// LFVector w of the batch is w - vbegin[i] of array i = varr[w].
template <uint32_t kLanes>
__global__ __launch_bounds__(256) void batch_shrink_kernel(const BatchArr* items, const uint64_t* vbegin,
                                                           const uint32_t* varr, uint64_t total, uint32_t num,
                                                           uint32_t den) {
  const uint64_t w = ((uint64_t)blockIdx.x * 256 + threadIdx.x) / kLanes;
  if (w >= total) return;
  const uint32_t i = varr[w];
  shrink_vector<kLanes>(items[i].A, (uint32_t)(w - vbegin[i]), num, den, items[i].elem_log2);
}

// r/w or flatten of every array of the batch.  With a tile table covering the
// batch, each XCD's workgroups stride over their eighth of it (r/w with
// non-temporal loads from kNtLoadBytes of elements on); otherwise a persistent
// grid: workgroup w takes the w-th contiguous share of the tiles and walks it
// array by array.  Flatten writes array i at out + elem_begin[i].
template <typename T, bool kFlatten>
__global__ __launch_bounds__(kRwThreads) void batch_stream_kernel(const BatchArr* items, const uint64_t* tile_begin,
                                                                 const uint64_t* elem_begin, uint32_t n,
                                                                 const uint64_t* __restrict__ tab, uint64_t tcap,
                                                                 uint32_t op, T* out, uint64_t cap,
                                                                 uint32_t* err, uint32_t te_log2) {
  const uint64_t total = tile_begin[n];
  if (kFlatten && elem_begin[n] > cap) {
    if (blockIdx.x == 0 && threadIdx.x == 0) set_error(err, kErrRange);
    return;
  }
  const uint64_t G = gridDim.x;
  if (total <= tcap) {
    const TileSpan sp = xcd_span(total);
    if (!kFlatten && elem_begin[n] * sizeof(T) >= kNtLoadBytes)
      table_tiles<T, false, true>(tab, sp, op, out);
    else
      table_tiles<T, kFlatten, kFlatten>(tab, sp, op, out);
    return;
  }
  uint64_t g0 = total * blockIdx.x / G;
  const uint64_t g1 = total * (blockIdx.x + 1) / G;
  if (g0 >= g1) return;
  uint32_t i = wave_search(tile_begin, n, g0);
  while (g0 < g1 && i < n) {
    const uint64_t b0 = tile_begin[i], b1 = tile_begin[i + 1];
    const uint64_t hi = b1 < g1 ? b1 : g1;
    if (hi > g0)
      stream_range<T, kFlatten>(items[i].A, g0 - b0, hi - b0, op, kFlatten ? out + elem_begin[i] : nullptr, te_log2);
    if (hi > g0) g0 = hi;
    ++i;
  }
}

// ---------------------------------------------------------- served steps --
// Tile offsets of the step's items (exclusive prefix of their tile totals, entry
// n the sum) into tb, by one workgroup.
__device__ __forceinline__ void block_tile_offsets(const ServeItem* items, uint32_t n, uint64_t* tb) {
  __shared__ uint64_t wsum[kRwThreads / 64];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const uint32_t per = (n + kRwThreads - 1) / kRwThreads;
  const uint32_t i0 = tid * per < n ? tid * per : n;
  const uint32_t i1 = i0 + per < n ? i0 + per : n;
  uint64_t t = 0;
  for (uint32_t i = i0; i < i1; ++i) t += items[i].A.tprefix[items[i].A.V];
  const uint64_t it = wave_incl_scan64(t);
  if (lane == 63) wsum[w] = it;
  __syncthreads();
  uint64_t r = it - t, total = 0;
  for (uint32_t k = 0; k < kRwThreads / 64; ++k) {
    if (k < w) r += wsum[k];
    total += wsum[k];
  }
  for (uint32_t i = i0; i < i1; ++i) {
    tb[i] = r;
    r += items[i].A.tprefix[items[i].A.V];
  }
  if (tid == 0) tb[n] = total;
  __syncthreads();
}

// The r/w and flatten requests of one served step in one persistent grid: item i
// is r/w'd in place, or flattened to its own destination (written only if its
// reservation holds it).  The step's front launch scanned the arrays.  With
// kFused every workgroup forms the items' tile offsets in LDS itself; otherwise
// they come from tile_begin (batch_top_kernel).  Workgroup 0 also reports each
// flatten's length.
template <typename T, bool kFused>
__global__ __launch_bounds__(kRwThreads) void serve_stream_kernel(const ServeItem* items, const uint64_t* tile_begin,
                                                                 uint32_t n, uint32_t* err, uint32_t te_log2) {
  extern __shared__ uint64_t lds_tb[];
  if (blockIdx.x == 0)
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x)
      if (items[i].len_out) items[i].len_out[0] = items[i].A.prefix[items[i].A.V];
  const uint64_t* tb = tile_begin;
  if (kFused) {
    block_tile_offsets(items, n, lds_tb);
    tb = lds_tb;
  }
  const uint64_t total = tb[n];
  const uint64_t G = gridDim.x;
  uint64_t g0 = total * blockIdx.x / G;
  const uint64_t g1 = total * (blockIdx.x + 1) / G;
  if (g0 >= g1) return;
  uint32_t i = wave_search(tb, n, g0);
  while (g0 < g1 && i < n) {
    const uint64_t b0 = tb[i], b1 = tb[i + 1];
    const uint64_t hi = b1 < g1 ? b1 : g1;
    if (hi > g0) {
      const ServeItem& it = items[i];
      if (it.op != kOpFlatten)
        stream_range<T, false>(it.A, g0 - b0, hi - b0, it.op, nullptr, te_log2);
      else if (it.A.prefix[it.A.V] <= it.cap)
        stream_range<T, true>(it.A, g0 - b0, hi - b0, 0u, static_cast<T*>(it.out), te_log2);
      else if (threadIdx.x == 0)
        set_error(err, kErrRange);
      g0 = hi;
    }
    ++i;
  }
}

// Sizes of the arrays of a server, one workgroup per array.
__global__ __launch_bounds__(256) void serve_sizes_kernel(const SizeItem* items, uint64_t* out) {
  __shared__ uint64_t red[4];
  const SizeItem it = items[blockIdx.x];
  uint64_t s = 0;
  for (uint32_t v = threadIdx.x; v < it.V; v += 256) s += it.size[v];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((threadIdx.x & 63u) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

}  // namespace

int launch_serve_sizes(const SizeItem* items, uint32_t n, uint64_t* out, hipStream_t s) {
  hipLaunchKernelGGL(serve_sizes_kernel, dim3(n), dim3(256), 0, s, items, out);
  return hip_status(hipGetLastError());
}

int launch_serve_stream(const ServeItem* items, uint32_t n, uint64_t* tile_begin, uint64_t* elem_begin,
                        uint32_t* err, uint32_t elem_bytes, uint32_t grid, hipStream_t s) {
  if (n == 0) return GGA_OK;
  const uint32_t te_log2 = elem_bytes == 4 ? 12u : 11u;
  if (grid < 1) grid = 1;
  if (grid > kRwBlocks) grid = kRwBlocks;
  const bool fused = n <= kServeFusedItems;
  const size_t lds = fused ? (n + 1) * sizeof(uint64_t) : 0;
  if (!fused)
    hipLaunchKernelGGL(batch_top_kernel<ServeItem>, dim3(1), dim3(kScanThreads), 0, s, items, n, tile_begin,
                       elem_begin);
  if (elem_bytes == 4) {
    if (fused)
      hipLaunchKernelGGL((serve_stream_kernel<uint32_t, true>), dim3(grid), dim3(kRwThreads), lds, s, items,
                         tile_begin, n, err, te_log2);
    else
      hipLaunchKernelGGL((serve_stream_kernel<uint32_t, false>), dim3(grid), dim3(kRwThreads), 0, s, items,
                         tile_begin, n, err, te_log2);
  } else {
    if (fused)
      hipLaunchKernelGGL((serve_stream_kernel<uint64_t, true>), dim3(grid), dim3(kRwThreads), lds, s, items,
                         tile_begin, n, err, te_log2);
    else
      hipLaunchKernelGGL((serve_stream_kernel<uint64_t, false>), dim3(grid), dim3(kRwThreads), 0, s, items,
                         tile_begin, n, err, te_log2);
  }
  return hip_status(hipGetLastError());
}

// Grows the tile table to what the array's sizes may need (not while the stream is
// capturing, nor with the sizes unknown to the host, after device-side pushes).
// Tiles of an LFVector of s elements: at most s / te + one partial tile per bucket.
static uint64_t table_need(const ggarray* a) {
  if (a->size_ub >= (1ull << 40)) return a->tab_cap;
  const uint64_t need = (a->size_ub >> (14u - a->elem_log2)) + (uint64_t)a->V * (nbuckets_for(a->log2F, a->size_ub) + 1);
  return need > kTableMaxTiles ? kTableMaxTiles : need;
}
static int grow_table(ggarray* a, bool capturing, hipStream_t s) {
  const uint64_t need = table_need(a);
  if (need <= a->tab_cap || capturing) return GGA_OK;
  uint64_t ncap = a->tab_cap * 2 > need ? a->tab_cap * 2 : need;
  if (ncap > kTableMaxTiles) ncap = kTableMaxTiles;
  void* p = nullptr;
  if (hipMallocAsync(&p, 16 * ncap, s) != hipSuccess) {
    (void)hipGetLastError();  // keep the smaller table; a larger array walks its buckets
    return GGA_OK;
  }
  if (retire_buffer(a, a->tile_tab, s) != GGA_OK) return GGA_EHIP;
  a->retired_tab_bytes += 16 * a->tab_cap;
  a->tile_tab = static_cast<uint64_t*>(p);
  a->tab_cap = ncap;
  return GGA_OK;
}

// Whether r/w and flatten of the array go through a tile table.
static bool streams_by_table(const ggarray* a) { return (a->size_ub >> (14u - a->elem_log2)) >= kTableMinTiles; }

int launch_scan(ggarray* a, hipStream_t s, uint64_t* copy, ScanTable table) {
  const uint32_t te_log2 = 14u - a->elem_log2;
  const uint64_t tag = stream_capture_tag(s);
  bool with_table = table != kScanOnly && a->V <= 4 * kScanThreads && streams_by_table(a) && capture_reuse(a, tag, tag);
  if (with_table && table == kScanGrowTable) {
    const int rc = grow_table(a, tag != 0, s);
    if (rc) return rc;
  }
  with_table = with_table && a->tab_cap && (table == kScanGrowTable || table_need(a) <= a->tab_cap);
  if (with_table) {
    hipLaunchKernelGGL(scan_table_kernel, dim3((a->V + kVecPerBlock - 1) / kVecPerBlock), dim3(256), 0, s, a->ref,
                       copy, a->tile_tab, a->tab_cap, te_log2, a->elem_log2);
  } else if (a->V <= 4 * kScanThreads) {  // one workgroup, a few LFVectors per thread
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(kScanThreads), 0, s, a->ref, te_log2, copy);
  } else {  // one workgroup per 1024 LFVectors, two passes
    const uint32_t chunks = (a->V + kScanThreads - 1) / kScanThreads;
    hipLaunchKernelGGL(scan_chunks_kernel, dim3(chunks), dim3(kScanThreads), 0, s, a->ref, a->scan_tot, te_log2);
    hipLaunchKernelGGL(scan_fix_kernel, dim3(chunks), dim3(kScanThreads), 0, s, a->ref, a->scan_tot, chunks, copy);
  }
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) {
    a->prefix_valid = true;
    a->scan_tag = tag;
    if (with_table) {
      a->tab_gen = a->sizes_gen;
      a->tab_tag = tag;
    }
  }
  return hip_status(e);
}

int launch_report(ggarray* a, const uint64_t* word, uint64_t* host, hipStream_t s) {
  hipLaunchKernelGGL(report_kernel, dim3(1), dim3(1), 0, s, word, a->ref.err, host);
  return hip_status(hipGetLastError());
}

int launch_shrink(ggarray* a, uint32_t num, uint32_t den, hipStream_t s) {
  if (num == den) a->size_ub = 0;
  if (a->V >= kChainMinV)
    hipLaunchKernelGGL(shrink_chain_kernel, dim3(kFreeShards * kChainLanes / 256), dim3(256), 0, s, a->ref, num, den,
                       a->elem_log2);
  else if (shrink_shares_wave(a->V))
    hipLaunchKernelGGL(shrink_kernel<16>, dim3((a->V + 15) / 16), dim3(256), 0, s, a->ref, num, den, a->elem_log2);
  else
    hipLaunchKernelGGL(shrink_kernel<64>, dim3((a->V + 3) / 4), dim3(256), 0, s, a->ref, num, den, a->elem_log2);
  sizes_changed(a, s);
  return hip_status(hipGetLastError());
}

int launch_free_all(ggarray* a, hipStream_t s) {
  const uint32_t blocks = (a->V + kVecPerBlock - 1) / kVecPerBlock;
  hipLaunchKernelGGL(free_all_kernel, dim3(blocks), dim3(256), 0, s, a->ref, a->elem_log2);
  return hip_status(hipGetLastError());
}

int launch_capacity(ggarray* a, uint64_t* d_out, hipStream_t s) {
  if (hipMemsetAsync(d_out, 0, sizeof(uint64_t), s) != hipSuccess) return GGA_EHIP;
  const uint32_t blocks = (a->V + 255) / 256;
  hipLaunchKernelGGL(capacity_kernel, dim3(blocks), dim3(256), 0, s, a->ref, d_out);
  return hip_status(hipGetLastError());
}

// Builds the tile table for the current sizes (the prefix must be current) unless
// the scan has.  Under graph capture it is always rebuilt, inside the graph, and
// never grown.
static int ensure_table(ggarray* a, hipStream_t s) {
  const uint64_t tag = stream_capture_tag(s);
  if (a->tab_gen == a->sizes_gen && capture_reuse(a, a->tab_tag, tag)) return GGA_OK;
  const int rc = grow_table(a, tag != 0, s);
  if (rc) return rc;
  if (a->tab_cap) {
    if (a->V >= kTableSharedMinV)
      hipLaunchKernelGGL(tile_table_kernel<16>, dim3((a->V + 15) / 16), dim3(256), 0, s, a->ref, a->tile_tab,
                         a->tab_cap, 14u - a->elem_log2, a->elem_log2);
    else
      hipLaunchKernelGGL(tile_table_kernel<64>, dim3((a->V + kVecPerBlock - 1) / kVecPerBlock), dim3(256), 0, s,
                         a->ref, a->tile_tab, a->tab_cap, 14u - a->elem_log2, a->elem_log2);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_status(e);
  }
  a->tab_gen = a->sizes_gen;
  a->tab_tag = tag;
  return GGA_OK;
}

// The table to stream through (its capacity 0: walk the buckets), built if needed.
static int stream_source(ggarray* a, hipStream_t s, const uint64_t** tab, uint64_t* cap) {
  *tab = nullptr;
  *cap = 0;
  if (a->prefix_gen == a->sizes_gen + 1) a->prefix_streamed = true;
  if (!streams_by_table(a)) return GGA_OK;
  const int rc = ensure_table(a, s);
  if (rc) return rc;
  *tab = a->tile_tab;
  *cap = a->tab_cap;
  return GGA_OK;
}

// Launches an r/w (kind 0) or flatten (kind 1) kernel.  With kernel timing on and
// the stream not capturing, the dispatch itself records the array's start and end
// events of that kind, so they bracket the kernel alone.
template <typename... Args, typename F>
static void launch_streaming(ggarray* a, uint32_t kind, F kernel, dim3 grid, dim3 block, hipStream_t s,
                             Args... args) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (a->tev[kind][0] && !stream_capturing(s)) {
    e0 = a->tev[kind][0];
    e1 = a->tev[kind][1];
    a->tev_set |= 1u << kind;
  }
  hipExtLaunchKernelGGL(kernel, grid, block, 0, s, e0, e1, 0, args...);
}

int launch_rw(ggarray* a, uint32_t op, hipStream_t s) {
  const uint64_t* tab;
  uint64_t tcap;
  const int rc = stream_source(a, s, &tab, &tcap);
  if (rc) return rc;
  const uint32_t te_log2 = 14u - a->elem_log2;
  const dim3 grid(stream_grid(a, tcap ? kTableBlocks : kRwBlocks)), block(kRwThreads);
  const bool nt = a->last_rw_gen == a->sizes_gen + 1;  // the array's previous streaming call was an r/w
  if (a->elem_bytes == 4) {
    if (nt)
      launch_streaming(a, 0, stream_table_kernel<uint32_t, false, true>, grid, block, s, a->ref, tab, tcap, op,
                       (uint32_t*)nullptr, (uint64_t)0, te_log2);
    else
      launch_streaming(a, 0, stream_table_kernel<uint32_t, false>, grid, block, s, a->ref, tab, tcap, op,
                       (uint32_t*)nullptr, (uint64_t)0, te_log2);
  } else {
    if (nt)
      launch_streaming(a, 0, stream_table_kernel<uint64_t, false, true>, grid, block, s, a->ref, tab, tcap, op,
                       (uint64_t*)nullptr, (uint64_t)0, te_log2);
    else
      launch_streaming(a, 0, stream_table_kernel<uint64_t, false>, grid, block, s, a->ref, tab, tcap, op,
                       (uint64_t*)nullptr, (uint64_t)0, te_log2);
  }
  a->last_rw_gen = a->sizes_gen + 1;
  return hip_status(hipGetLastError());
}

int launch_flatten(ggarray* a, void* out, uint64_t cap, hipStream_t s) {
  const uint64_t* tab;
  uint64_t tcap;
  const int rc = stream_source(a, s, &tab, &tcap);
  if (rc) return rc;
  a->last_rw_gen = 0;
  const uint32_t te_log2 = 14u - a->elem_log2;
  const dim3 grid(stream_grid(a, tcap ? kTableBlocks : kFlattenBlocks)), block(kRwThreads);
  if (a->elem_bytes == 4)
    launch_streaming(a, 1, stream_table_kernel<uint32_t, true>, grid, block, s, a->ref, tab, tcap, 0u,
                     static_cast<uint32_t*>(out), cap, te_log2);
  else
    launch_streaming(a, 1, stream_table_kernel<uint64_t, true>, grid, block, s, a->ref, tab, tcap, 0u,
                     static_cast<uint64_t*>(out), cap, te_log2);
  return hip_status(hipGetLastError());
}

// The static array's r/w in the GGArray's launch shape: one workgroup per 16 KiB
// tile of the host's bound of its size (up to kTableBlocks, looping beyond) and
// the same load policy, so that only the layout differs.  (A grid sized for the
// capacity dispatches a workgroup per empty tile: 2^30-element capacity holding
// 6.25e7 elements streamed at 5.0 TB/s against 6.35 for the same bytes sized to
// fit.)
int launch_static_rw(gga_static* st, uint32_t op, hipStream_t s) {
  const uint32_t te_log2 = st->elem_bytes == 4 ? 12u : 11u;
  const uint64_t ub = st->size_ub < st->cap ? st->size_ub : st->cap;
  const uint64_t tiles = (ub + (1ull << te_log2) - 1) >> te_log2;
  const dim3 grid(xcd_grid(tiles > kTableBlocks ? kTableBlocks : tiles)), block(kRwThreads);
  const bool nt = st->rw_last;
  if (st->elem_bytes == 4) {
    if (nt)
      hipLaunchKernelGGL((static_rw_kernel<uint32_t, true>), grid, block, 0, s, static_cast<uint32_t*>(st->data),
                         st->d_size, st->cap, op, te_log2);
    else
      hipLaunchKernelGGL((static_rw_kernel<uint32_t, false>), grid, block, 0, s, static_cast<uint32_t*>(st->data),
                         st->d_size, st->cap, op, te_log2);
  } else {
    if (nt)
      hipLaunchKernelGGL((static_rw_kernel<uint64_t, true>), grid, block, 0, s, static_cast<uint64_t*>(st->data),
                         st->d_size, st->cap, op, te_log2);
    else
      hipLaunchKernelGGL((static_rw_kernel<uint64_t, false>), grid, block, 0, s, static_cast<uint64_t*>(st->data),
                         st->d_size, st->cap, op, te_log2);
  }
  st->rw_last = true;
  return hip_status(hipGetLastError());
}


// Sum of the member arrays' size generations: unchanged exactly when no member's
// sizes can have changed since it was last taken.
static uint64_t batch_gen(const gga_batch* b) {
  uint64_t g = 0;
  for (uint32_t i = 0; i < b->n; ++i) g += b->arrays[i]->sizes_gen;
  return g;
}

// capture_reuse for a batch: eager reuse also needs that no graph changes the
// sizes of any member.
static bool batch_reuse(const gga_batch* b, uint64_t built, uint64_t now) {
  if (built != now || now == ~0ull) return false;
  if (now == 0)
    for (uint32_t i = 0; i < b->n; ++i)
      if (b->arrays[i]->graph_sized) return false;
  return true;
}

int launch_batch_scan(gga_batch* b, hipStream_t s) {
  const uint64_t gen = batch_gen(b);
  const uint64_t tag = stream_capture_tag(s);
  if (b->scan_valid && b->scan_gen == gen && batch_reuse(b, b->scan_tag, tag)) return GGA_OK;
  const uint32_t te_log2 = b->elem_bytes == 4 ? 12u : 11u;
  hipLaunchKernelGGL(batch_scan_kernel, dim3(b->n), dim3(kScanThreads), 0, s, b->d_arrays, te_log2);
  hipLaunchKernelGGL(batch_top_kernel<BatchArr>, dim3(1), dim3(kScanThreads), 0, s, b->d_arrays, b->n,
                     b->d_tile_begin, b->d_elem_begin);
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) {
    for (uint32_t i = 0; i < b->n; ++i) {
      b->arrays[i]->prefix_valid = true;
      b->arrays[i]->scan_tag = tag;
    }
    b->scan_valid = true;
    b->scan_gen = gen;
    b->scan_tag = tag;
  }
  return hip_status(e);
}

// The batch's tile table for the current sizes (after launch_batch_scan); like
// the single-array table it is grown only outside graph capture, retired rather
// than freed, and always rebuilt under capture.  *tab / *tcap: what to stream
// through (capacity 0: the persistent walk).
static int ensure_batch_table(gga_batch* b, hipStream_t s, const uint64_t** tab, uint64_t* tcap, uint64_t* bound) {
  const uint32_t te_log2 = b->elem_bytes == 4 ? 12u : 11u;
  uint64_t need = 0;
  bool known = true;
  for (uint32_t i = 0; i < b->n; ++i) {
    const ggarray* a = b->arrays[i];
    if (a->size_ub >= (1ull << 40)) known = false;
    else need += (a->size_ub >> te_log2) + (uint64_t)a->V * (nbuckets_for(a->log2F, a->size_ub) + 1);
  }
  *bound = known ? need : kTableMaxTiles;
  *tab = nullptr;
  *tcap = 0;
  if (known && need < kTableMinTiles) return GGA_OK;
  if (!known) need = b->tab_cap;
  if (need > kTableMaxTiles) need = kTableMaxTiles;
  const uint64_t tag = stream_capture_tag(s);
  const bool cap_mode = tag != 0;
  const uint64_t gen = batch_gen(b);
  if (!(b->tab_valid && b->tab_gen == gen && batch_reuse(b, b->tab_tag, tag))) {
    if (need > b->tab_cap && !cap_mode) {
      uint64_t ncap = b->tab_cap * 2 > need ? b->tab_cap * 2 : need;
      if (ncap > kTableMaxTiles) ncap = kTableMaxTiles;
      void* p = nullptr;
      if (hipMalloc(&p, 16 * ncap) == hipSuccess) {  // freed with hipFree when the batch is destroyed
        if (b->tile_tab) {
          if (b->n_retired < sizeof(b->retired) / sizeof(b->retired[0])) b->retired[b->n_retired++] = b->tile_tab;
          else if (hipFree(b->tile_tab) != hipSuccess) return GGA_EHIP;  // waits for the device
        }
        b->tile_tab = static_cast<uint64_t*>(p);
        b->tab_cap = ncap;
      } else {
        (void)hipGetLastError();
      }
    }
    if (b->tab_cap) {
      const uint64_t V = b->total_vectors;
      if (V >= kTableSharedMinV)
        hipLaunchKernelGGL(batch_table_kernel<16>, dim3((uint32_t)((V + 15) / 16)), dim3(256), 0, s, b->d_arrays,
                           b->d_vbegin, b->d_varr, b->d_tile_begin, b->d_elem_begin, V, b->tile_tab, b->tab_cap,
                           te_log2);
      else
        hipLaunchKernelGGL(batch_table_kernel<64>, dim3((uint32_t)((V + kVecPerBlock - 1) / kVecPerBlock)), dim3(256),
                           0, s, b->d_arrays, b->d_vbegin, b->d_varr, b->d_tile_begin, b->d_elem_begin, V,
                           b->tile_tab, b->tab_cap, te_log2);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return hip_status(e);
    }
    b->tab_valid = true;
    b->tab_gen = gen;
    b->tab_tag = tag;
  }
  *tab = b->tile_tab;
  *tcap = b->tab_cap;
  return GGA_OK;
}

// Whether a batch's clears and shrinks run as chains: from 32768 LFVectors on, where the 16
// of a residue and pass share their lists in at least half of the batch (arrays created in a
// row with one first bucket, or long arrays).  Where they differ the chain kernel releases
// bucket by bucket, and an LFVector each for 16 lanes is faster (16 arrays of 5001
// LFVectors with others created between: 69 us, 48 that way; 4 of 20000 in a row: 31, 50).
constexpr uint64_t kBatchChainMinV = 32768;
bool batch_chains_suit(ggarray* const* arrays, const uint64_t* vbegin, const uint32_t* varr, uint64_t total) {
  if (total < kBatchChainMinV) return false;
  const auto same = [&](uint64_t w, uint64_t x) {
    const ggarray *a = arrays[varr[w]], *b = arrays[varr[x]];
    const uint64_t d = (w - vbegin[varr[w]] + a->ref.salt) - (x - vbegin[varr[x]] + b->ref.salt);
    return a->ref.pool.hdr == b->ref.pool.hdr && a->ref.log2F == b->ref.log2F && d % kFreeShards == 0;
  };
  uint64_t alike = 0;
  for (uint64_t w0 = 0; w0 < total; w0 += kChainStep)
    for (uint64_t w = w0; w < w0 + kFreeShards && w < total; ++w) {
      uint64_t n = 1;
      for (uint64_t x = w + kFreeShards; n && x < w0 + kChainStep && x < total; x += kFreeShards)
        n = same(w, x) ? n + 1 : 0;
      alike += n;
    }
  return 2 * alike >= total;
}

int launch_batch_shrink(gga_batch* b, uint32_t num, uint32_t den, hipStream_t s) {
  if (num == den)
    for (uint32_t i = 0; i < b->n; ++i) b->arrays[i]->size_ub = 0;
  const uint64_t V = b->total_vectors;
  if (b->chains)
    hipLaunchKernelGGL(batch_shrink_chain_kernel, dim3(kFreeShards * kChainLanes / 256), dim3(256), 0, s,
                       b->d_arrays, b->d_vbegin, b->d_varr, V, num, den);
  else if (shrink_shares_wave(V))
    hipLaunchKernelGGL(batch_shrink_kernel<16>, dim3((uint32_t)((V + 15) / 16)), dim3(256), 0, s, b->d_arrays,
                       b->d_vbegin, b->d_varr, V, num, den);
  else
    hipLaunchKernelGGL(batch_shrink_kernel<64>, dim3((uint32_t)((V + 3) / 4)), dim3(256), 0, s, b->d_arrays,
                       b->d_vbegin, b->d_varr, V, num, den);
  for (uint32_t i = 0; i < b->n; ++i) sizes_changed(b->arrays[i], s);
  return hip_status(hipGetLastError());
}

int launch_batch_stream(gga_batch* b, uint32_t op, void* out, uint64_t cap, bool flatten, hipStream_t s) {
  const uint32_t te_log2 = b->elem_bytes == 4 ? 12u : 11u;
  const uint64_t* tab;
  uint64_t tcap, bound;
  const int rc = ensure_batch_table(b, s, &tab, &tcap, &bound);
  if (rc) return rc;
  uint64_t g = b->stream_blocks;
  if (!g) g = tcap ? (bound < kTableBlocks ? bound : kTableBlocks) : (flatten ? kFlattenBlocks : kRwBlocks);
  const dim3 grid(tcap ? xcd_grid(g) : (uint32_t)g), block(kRwThreads);
  if (b->elem_bytes == 4) {
    if (flatten)
      hipLaunchKernelGGL((batch_stream_kernel<uint32_t, true>), grid, block, 0, s, b->d_arrays, b->d_tile_begin,
                         b->d_elem_begin, b->n, tab, tcap, 0u, static_cast<uint32_t*>(out), cap, b->d_err, te_log2);
    else
      hipLaunchKernelGGL((batch_stream_kernel<uint32_t, false>), grid, block, 0, s, b->d_arrays, b->d_tile_begin,
                         b->d_elem_begin, b->n, tab, tcap, op, (uint32_t*)nullptr, (uint64_t)0, b->d_err, te_log2);
  } else {
    if (flatten)
      hipLaunchKernelGGL((batch_stream_kernel<uint64_t, true>), grid, block, 0, s, b->d_arrays, b->d_tile_begin,
                         b->d_elem_begin, b->n, tab, tcap, 0u, static_cast<uint64_t*>(out), cap, b->d_err, te_log2);
    else
      hipLaunchKernelGGL((batch_stream_kernel<uint64_t, false>), grid, block, 0, s, b->d_arrays, b->d_tile_begin,
                         b->d_elem_begin, b->n, tab, tcap, op, (uint64_t*)nullptr, (uint64_t)0, b->d_err, te_log2);
  }
  return hip_status(hipGetLastError());
}

}  // namespace gga
