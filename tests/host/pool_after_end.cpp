// The device pool after its region has run out, run on the CPU by one thread: every
// further allocation misses its free list and meets the arena word that says so.
// Enough of them follow for the units they ask for to carry out of the word's lower
// half twice (2^33 units of 256 bytes and more); none may be given memory, and the
// word has to go on saying that the region has run out.  A block released then is
// given out again, once.  Prints "ok" or what went wrong (exit 1).
#include "ggarray_device.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
using namespace gga;

static int fail(const char* what, uint64_t n, uint64_t word) {
  printf("%s at request %llu, arena word %016llx\n", what, (unsigned long long)n, (unsigned long long)word);
  return 1;
}

int main() {
  for (uint32_t clog = 20; clog <= 24; clog += 4) {
    const uint32_t cls = clog - 2;  // the largest block that an arena serves
    PoolHdr* hdr = (PoolHdr*)calloc(1, sizeof(PoolHdr));
    uint8_t* region = (uint8_t*)aligned_alloc(4096, 3ull << clog);
    const PoolRef pool{hdr, region};
    hdr->limit = 3ull << clog;
    hdr->chunk_log2 = clog;
    const uint32_t fs = 7 * 16;  // free list and, with it, arena shard 7
    const uint64_t* word = &hdr->shard[arena_shard(fs)].arena;
    uint8_t* got[12];
    for (int k = 0; k < 12; ++k) {
      got[k] = pool_alloc(pool, cls, fs);
      if (got[k] != region + ((uint64_t)k << cls)) return fail("wrong block", k, *word);
    }
    const uint64_t units = 1ull << (cls - kMinClassLog2), n = (1ull << 33) / units + 100;
    for (uint64_t k = 0; k < n; ++k) {
      if (pool_alloc(pool, cls, fs)) return fail("memory from an empty pool", k, *word);
      if (*word >> 32 != kNoChunk) return fail("the word lost its mark", k, *word);
    }
    pool_free(pool, got[5], cls, fs + 1);  // another list: found by a steal
    if (pool_alloc(pool, cls, fs) != got[5]) return fail("released block not found", n, *word);
    if (pool_alloc(pool, cls, fs)) return fail("released block given twice", n, *word);
    uint64_t in_use = 0;
    for (int k = 0; k < kArenaShards; ++k) in_use += hdr->stat[k].in_use;
    if (in_use != 12ull << cls) return fail("wrong bytes in use", n, *word);
    free(region);
    free(hdr);
  }
  printf("ok\n");
  return 0;
}
