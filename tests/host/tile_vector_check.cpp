// Host check of where the flagged rounds' vector loads of a tile start: inside the
// buffers always; a lane whose vector holds a thread of the tile reads that vector, or,
// where it would run past the buffers, their last one; every other lane reads what a lane
// of the tile reads too.  All tile lengths at several distances to the end of the
// buffers.  Prints "ok <cases>" or the first mismatch (exit 1).
#include "gga_internal.h"
#include <cstdio>
using namespace gga;

template <uint32_t E>
static uint64_t check() {
  uint64_t cases = 0;
  for (uint32_t len = 1; len <= kInsertTile; ++len)
    for (uint64_t after : {0ull, 1ull, (unsigned long long)E - 1, (unsigned long long)E, 4095ull, 4096ull, 1ull << 33}) {
      const uint64_t g0 = 3 * kInsertTile + 1, te = g0 + len, n = te + after;
      const int32_t room = tile_room(g0, n);
      for (uint32_t d = 0; d < kInsertTile; d += E, ++cases) {
        const uint64_t at = g0 + tile_vector<E>(d, len, room);
        const uint64_t want = g0 + d < te ? (g0 + d + E <= n ? g0 + d : n - E) : (g0 + E <= n ? g0 : n - E);
        if (at != want || at + E > n) {
          printf("mismatch E=%u len=%u after=%llu d=%u: %llu, not %llu\n", E, len, (unsigned long long)after, d,
                 (unsigned long long)at, (unsigned long long)want);
          return 0;
        }
      }
    }
  return cases;
}

int main() {
  const uint64_t a = check<4>(), b = a ? check<2>() : 0;
  if (!a || !b) return 1;
  printf("ok %llu\n", (unsigned long long)(a + b));
  return 0;
}
