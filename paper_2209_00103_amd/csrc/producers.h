// Producers of insertion rounds: how logical thread gid decides whether it
// inserts and what (the synthetic workloads of the benchmark configurations and
// the buffer inputs of the C ABI).  Shared by the round kernels and the
// persistent step kernel, so every path produces the same elements.
//
// run(g0, n) gives the elements of the n consecutive threads from g0 on by their
// distance from g0 (K's argument grows by 256 per thread, seed and round occupying
// the bits above and below the thread's, so xor and sum agree).
#pragma once

#include "gga_internal.h"

namespace gga {

// Thread gid inserts values[gid] iff flags[gid] != 0.  Without flags (every
// thread inserts) only the dense kernels run, and they read values alone, so
// flag() reads flags unconditionally (a test per slot would keep each flag load
// under a branch, which costs a memory round trip per slot).
template <typename T>
struct ProdBuffer {
  static constexpr bool kMulti = false;
  static constexpr bool kDense = false;
  static constexpr bool kLoads = true;  // flags and payloads come from memory
  const T* values;
  const uint8_t* flags;
  __device__ __forceinline__ bool flag(uint64_t g) const { return flags[g] != 0; }
  __device__ __forceinline__ T value(uint64_t g) const { return values[g]; }
  struct Run {
    const T* p;
    __device__ __forceinline__ T operator()(uint64_t d) const { return p[d]; }
  };
  __device__ __forceinline__ Run run(uint64_t g0, uint64_t) const { return {values + g0}; }
};
// A payload buffer larger than the cache, copied by dense_store: its lines are not kept.
template <typename T>
struct ProdBufferOnce {
  static constexpr bool kDense = false;
  const T* values;
  using Run = typename ProdBuffer<T>::Run;
  __device__ __forceinline__ Run run(uint64_t g0, uint64_t) const { return {values + g0}; }
};
template <typename T>
struct ProdBernoulli {  // h = K(seed, gid, round); insert (T)h iff top bit
  static constexpr bool kMulti = false;
  static constexpr bool kDense = false;
  static constexpr bool kLoads = false;
  uint64_t seed;
  uint32_t round;
  __device__ __forceinline__ bool flag(uint64_t g) const { return (K(seed, g, round) >> 63) != 0; }
  __device__ __forceinline__ T value(uint64_t g) const { return (T)K(seed, g, round); }
  __device__ __forceinline__ bool take(uint64_t g, T& v) const {  // flag and value from one hash
    const uint64_t h = K(seed, g, round);
    v = (T)h;
    return (h >> 63) != 0;
  }
  struct Run {
    MixRun mix;
    __device__ __forceinline__ T operator()(uint32_t d) const { return (T)mix((uint64_t)d << 8); }
    __device__ __forceinline__ bool take(uint32_t d, T& v) const {
      const uint64_t h = mix((uint64_t)d << 8);
      v = (T)h;
      return (h >> 63) != 0;
    }
  };
  __device__ __forceinline__ Run run(uint64_t g0, uint64_t n) const {
    return {MixRun((seed << 56) + (g0 << 8) + round, n << 8)};
  }
  __device__ __forceinline__ void bind(const BatchArr&) {}
};
template <typename T>
struct ProdRoundTag {  // insert (round << shift) | gid
  static constexpr bool kMulti = false;
  static constexpr bool kDense = true;  // every thread inserts
  static constexpr bool kLoads = false;
  static constexpr bool kMixed = false;
  uint32_t round;
  uint32_t shift;
  __device__ __forceinline__ bool flag(uint64_t) const { return true; }
  __device__ __forceinline__ T value(uint64_t g) const { return (T)(((uint64_t)round << shift) | g); }
  __device__ __forceinline__ bool take(uint64_t g, T& v) const {
    v = value(g);
    return true;
  }
  struct Run {
    ProdRoundTag prod;
    uint64_t g0;
    __device__ __forceinline__ T operator()(uint32_t d) const { return prod.value(g0 + d); }
    __device__ __forceinline__ bool take(uint32_t d, T& v) const { return prod.take(g0 + d, v); }
  };
  __device__ __forceinline__ Run run(uint64_t g0, uint64_t) const { return {*this, g0}; }
  __device__ __forceinline__ void bind(const BatchArr&) {}
};
template <typename T>
struct ProdKeyed {  // every thread inserts K(seed, (tag << shift) | gid, round)
  static constexpr bool kMulti = false;
  static constexpr bool kDense = true;
  static constexpr bool kLoads = false;
  static constexpr bool kMixed = true;  // Run holds a MixRun
  uint64_t seed;
  uint32_t round;
  uint32_t shift;
  uint64_t tag;
  __device__ __forceinline__ bool flag(uint64_t) const { return true; }
  __device__ __forceinline__ T value(uint64_t g) const { return (T)K(seed, (tag << shift) | g, round); }
  __device__ __forceinline__ bool take(uint64_t g, T& v) const {
    v = value(g);
    return true;
  }
  struct Run {
    MixRun mix;
    __device__ __forceinline__ T operator()(uint32_t d) const { return (T)mix((uint64_t)d << 8); }
    template <bool kFlat>
    __device__ __forceinline__ T at(uint32_t d) const { return (T)mix.template at<kFlat>((uint64_t)d << 8); }
    __device__ __forceinline__ bool take(uint32_t d, T& v) const {
      v = (T)mix((uint64_t)d << 8);
      return true;
    }
  };
  __device__ __forceinline__ Run run(uint64_t g0, uint64_t n) const {
    return {MixRun((seed << 56) + (((tag << shift) | g0) << 8) + round, n << 8)};
  }
  __device__ __forceinline__ void bind(const BatchArr& it) { tag = it.tag; }  // each array its own key
};
template <typename T>
struct ProdCounts {  // insert values[gid * max + j], j < counts[gid]
  static constexpr bool kMulti = true;
  static constexpr bool kRuns = false;  // RunTile is Tile
  const T* values;
  const uint8_t* counts;
  uint32_t max_count;
  __device__ __forceinline__ uint32_t count(uint64_t g) const {
    const uint32_t c = counts[g];
    return c < max_count ? c : max_count;
  }
  // The counts and elements of a tile's threads by their distance from its first
  // thread g0 (at most 1024 of them).
  struct Tile {
    ProdCounts prod;
    uint64_t g0;
    __device__ __forceinline__ uint32_t count(uint32_t d) const { return prod.count(g0 + d); }
    __device__ __forceinline__ T value(uint32_t d, uint32_t r) const {
      return prod.values[(g0 + d) * prod.max_count + r];
    }
  };
  __device__ __forceinline__ Tile tile(uint64_t g0) const { return {*this, g0}; }
  typedef Tile RunTile;
  __device__ __forceinline__ RunTile run_tile(uint64_t g0) const { return tile(g0); }
};
template <typename T>
struct ProdPoisson {  // c = #{k : K(seed,gid,0x80|round) >= thr[k]}; insert K(seed,gid,16 round + j)
  static constexpr bool kMulti = true;
  static constexpr bool kRuns = true;
  uint64_t seed;
  uint32_t round;
  uint32_t max_count;
  uint64_t thr[16];
  // How many of the thresholds a draw reaches.
  __device__ __forceinline__ uint32_t reached(uint64_t u) const {
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) c += (k < (int)max_count && u >= thr[k]) ? 1u : 0u;
    return c;
  }
  // With the whole hash for each draw and element: in a round of few tiles each one's
  // chain hides the product that a run of states saves, and fetching both forms of the
  // hash costs more than it gains (1000 threads 13.2 us with runs, 12.4 us so).
  struct Tile {
    const ProdPoisson* prod;
    uint64_t g0;
    __device__ __forceinline__ uint32_t count(uint32_t d) const {
      return prod->reached(K(prod->seed, g0 + d, 0x80u | prod->round));
    }
    __device__ __forceinline__ T value(uint32_t d, uint32_t r) const {
      return (T)K(prod->seed, g0 + d, 16u * prod->round + r);
    }
  };
  __device__ __forceinline__ Tile tile(uint64_t g0) const { return {this, g0}; }
  // For rounds bound by issuing: a wave per LFVector (65536 of them 2% shorter), many tiles
  // (16384 of them 180 us as above, 174 so).
  struct RunTile {
    const ProdPoisson* prod;
    MixRun draws, mix;
    __device__ __forceinline__ uint32_t count(uint32_t d) const { return prod->reached(draws((uint64_t)d << 8)); }
    __device__ __forceinline__ T value(uint32_t d, uint32_t r) const { return (T)mix(((uint64_t)d << 8) + r); }
  };
  __device__ __forceinline__ RunTile run_tile(uint64_t g0) const {
    const uint64_t first = (seed << 56) + (g0 << 8);
    return {this, MixRun(first + (0x80u | round), 1024u << 8), MixRun(first + 16u * round, 1024u << 8)};
  }
};

}  // namespace gga
