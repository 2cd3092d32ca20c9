"""Clears and partial shrinks at the edges of the release kernel's forms (a wave per
LFVector below 4096 LFVectors, 16 lanes each up to 16383, from there on one chain per
free list; batches: chains from 32768), single array and batch, with more buckets than a group has lanes; sizes, contents, capacity and the
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


@pytest.mark.parametrize("elem,V,F", [(4, 16383, 2), (4, 16384, 1), (8, 40001, 2), (4, 70001, 1)])
def test_shrink_chains_uneven(elem, V, F):
    """Uneven LFVectors (empty ones, one of 17 or more buckets), partial shrinks and clears;
    the next rounds take the released blocks again."""
    rng = np.random.default_rng(V + elem)
    G = gg()
    pool = G.Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    a2, o2 = both(elem, V, F, pool)
    dt = np.uint32 if elem == 4 else np.uint64
    for k, (num, den) in enumerate(((1, 3), (1, 1), (2, 3), (1, 1))):
        for g, q in ((a, o), (a2, o2)):
            n = rng.integers(0, 9, V) * (rng.random(V) < 0.8)
            n[(k * 7919) % V] += 200_000
            pre = np.concatenate([[0], np.cumsum(n)]).astype(np.uint64)
            vals = rng.integers(0, 1 << 31, int(pre[-1])).astype(dt)
            g.insert_segments(dev(vals), dev(pre))
            q.insert_segments(vals, pre)
        for g, q in ((a, o), (a2, o2)):
            g.shrink(num, den)
            q.shrink(num, den)
            assert_same(g, q, f"shrink {num}/{den}")
    st = pool.stats()
    assert st["in_use"] == 0 and st["allocs"] == st["frees"]
    a.close()
    a2.close()
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


@pytest.mark.parametrize("kind", ["row", "below", "mixed", "pools", "many"])
def test_shrink_batch_chains(kind):
    """Batches around the chain form's first LFVector count (32768): arrays created in a
    row, mixed first buckets, one left out of the batch, two pools, more LFVectors than
    one pass of a residue takes; uneven and empty LFVectors, partial shrinks and clears.
    The pools' counts say that every block went back once."""
    G = gg()
    rng = np.random.default_rng(len(kind))
    pools = [G.Pool(1 << 30) for _ in range(2 if kind == "pools" else 1)]
    shapes = {"row": [(30000, 2), (2768, 2)], "below": [(30000, 2), (2767, 2)], "many": [(40000, 64), (33333, 64)],
              "mixed": [(20000, 1), (7000, 64), (9000, 2)], "pools": [(20000, 2), (20000, 2)]}[kind]
    arrays, orcs = [], []
    for k, (V, F) in enumerate(shapes):
        arrays.append(G.GGArray(pools[k % len(pools)], 4, V, F))
        orcs.append(Oracle(4, V, F))
        if kind == "mixed":
            G.GGArray(pools[0], 4, 77, 4).close()  # shifts the next array's free lists
    batch = G.Batch(arrays)
    for r, (num, den) in enumerate(((1, 3), (1, 1), (2, 3), (1, 1))):
        for a, o, (V, F) in zip(arrays, orcs, shapes):
            n = rng.integers(0, 9, V) * (rng.random(V) < 0.7)
            n[(r * 7919) % V] += 150_000
            pre = np.concatenate([[0], np.cumsum(n)]).astype(np.uint64)
            vals = rng.integers(0, 1 << 31, int(pre[-1])).astype(np.uint32)
            a.insert_segments(dev(vals), dev(pre))
            o.insert_segments(vals, pre)
        batch.shrink(num, den)
        for a, o in zip(arrays, orcs):
            o.shrink(num, den)
            assert_same(a, o, f"{kind} round {r}")
    for p in pools:
        st = p.stats()
        assert st["in_use"] == 0 and st["allocs"] == st["frees"]
    batch.close()
    for a in arrays:
        a.close()
    for p in pools:
        p.close()
