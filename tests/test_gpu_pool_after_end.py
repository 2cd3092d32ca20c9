"""Arrays on a pool whose region has run out once: the blocks an earlier array gave back
are found on other free lists, also while the arena words have counted up to where a
few more requests would carry into their chunk id; sizes, contents and capacity against
the CPU oracle, and the words themselves."""
import numpy as np
import pytest
import torch

from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg

pytestmark = pytest.mark.gpu
# struct PoolHdr: eight words, the hint masks, the list heads, then one arena word per 128 bytes
ARENA_AT, ARENA_STEP, SHARDS = 64 + 41 * 64 * 8 + 41 * 4096 * 8, 128, 256
NO_CHUNK = 0xFFFFFFFF


def _arena_words(pool):
    mem = pool.mem[ARENA_AT:ARENA_AT + SHARDS * ARENA_STEP]
    return mem.view(torch.int64)[::ARENA_STEP // 8]


def test_arrays_after_the_region_has_run_out():
    G = gg()
    rng = np.random.default_rng(8)
    pool = G.Pool(8 << 20)
    V, F = 48, 64
    used = G.GGArray(pool, 4, V, F)
    while used.last_error() == 0:  # until the region is carved up and some LFVectors are frozen
        vals, _ = wl.random_round(rng, V * 3000, 1.0, 4)
        used.insert(dev(vals))
    assert used.last_error() == G.ENOMEM
    used.close()
    for r in range(4):  # each new array has free lists of its own, all empty at first
        a, o = both(4, V, F, pool)
        for k in range(3):
            words = _arena_words(pool)
            ended = (words >> 32 & NO_CHUNK) == NO_CHUNK
            assert r == 0 or bool(ended.any())
            near = torch.full_like(words, (NO_CHUNK << 32 | 0xFFFFFFFF - 40 * (k + 1)) - (1 << 64))
            words.copy_(torch.where(ended, near, words))
            vals, flags = wl.random_round(rng, V * 1500, 0.5, 4)
            a.insert(dev(vals), dev(flags))
            o.insert(vals, flags)
            a.insert(dev(vals))
            o.insert(vals)
            assert_same(a, o, f"array {r} round {k}")
            assert bool(((_arena_words(pool)[ended] >> 32 & NO_CHUNK) == NO_CHUNK).all())
        a.close()
        o.close()
    st = pool.stats()
    assert st["in_use"] == 0 and st["allocs"] == st["frees"]
    pool.close()
