"""Clears and partial shrinks at the edges of the release kernel's forms (a wave per
LFVector below 4096 LFVectors and from 32768 on, 16 lanes each between), single array
and batch, with more buckets than a group has lanes; sizes, contents, capacity and the
pool's counts against the CPU oracle."""
import numpy as np
import pytest

import oracle
from oracle import Oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg, gpu_sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elem,V,F,n", [
    (4, 4095, 16, 4095 * 90), (4, 4096, 16, 4096 * 90 - 50), (8, 32767, 64, 32767 * 5), (4, 32768, 64, 32768 * 5),
])
def test_shrink_group_edges(elem, V, F, n):
    rng = np.random.default_rng(V)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    for num, den in ((1, 3), (1, 1), (9, 10)):
        vals, flags = wl.random_round(rng, n, 0.7, elem)
        a.insert(dev(vals), dev(flags))
        o.insert(vals, flags)
        a.shrink(num, den)
        o.shrink(num, den)
        assert_same(a, o, f"shrink {num}/{den}")
    st = pool.stats()
    assert st["in_use"] == sum(max(256, elem * F << b) * int((o.vector_nbuckets() > b).sum()) for b in range(40))
    a.close()
    st = pool.stats()
    assert st["in_use"] == 0 and st["allocs"] == st["frees"]
    pool.close()


def test_shrink_group_many_buckets_and_batch():
    """F = 1 (up to 19 buckets, more than a group's 16 lanes) in a batch of 5000 LFVectors."""
    G = gg()
    pool = G.Pool(1 << 30)
    arrays = [G.GGArray(pool, 4, v, 1) for v in (4999, 1)]
    orcs = [Oracle(4, v, 1) for v in (4999, 1)]
    batch = G.Batch(arrays)
    threads = [4999 * 3, 400_000]
    for r in range(2):
        batch.insert_gen(G.make_gen(G.GEN_KEYED, seed=3, round=r, tag_shift=20), threads)
        for i, o in enumerate(orcs):
            o.insert_gen(oracle.GEN_KEYED, threads[i], seed=3, round=r, tag_shift=20, tag=i)
        batch.shrink(1, 4 - 3 * r)
        for a, o in zip(arrays, orcs):
            o.shrink(1, 4 - 3 * r)
            assert_same(a, o, f"round {r}")
    assert all(gpu_sizes(a).sum() == 0 for a in arrays)
    st = pool.stats()
    assert st["in_use"] == 0 and st["allocs"] == st["frees"]
    batch.close()
    for a in arrays:
        a.close()
    pool.close()
