"""Generated payloads where a run of threads crosses into the next upper half of the
generator's state (a wave then leaves the shared product of the first step): keyed
rounds placed on the crossing, single array in the one-launch, two-launch and
several-rounds forms, batch and persistent step; Bernoulli and Poisson rounds of
enough threads to reach it; against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from oracle import Oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, gg

pytestmark = pytest.mark.gpu
# (tag << 20) | g with tag = 8: the state's lower half, golden ratio added, wraps at g = 46468
KEY = dict(seed=5, tag_shift=20, tag=8)


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("V,n", [(1, 100001), (1, 30000), (8, 400003), (600, 100003), (513, 47000)])
def test_keyed_rounds_across_the_wrap(elem, V, n):
    G = gg()
    pool = G.Pool(512 << 20)
    a, o = both(elem, V, 64, pool)
    for r in range(2):
        a.insert_gen(G.make_gen(G.GEN_KEYED, round=r, **KEY), n)
        o.insert_gen(oracle.GEN_KEYED, n, round=r, **KEY)
        assert_same(a, o, f"round {r}")
    a.insert_gen_rounds([G.make_gen(G.GEN_KEYED, round=r, **KEY) for r in (2, 3)], [n, n // 2])
    for r, m in ((2, n), (3, n // 2)):
        o.insert_gen(oracle.GEN_KEYED, m, round=r, **KEY)
    assert_same(a, o, "rounds in one call")
    a.close()
    pool.close()


def test_keyed_batch_and_step_across_the_wrap():
    G = gg()
    pool = G.Pool(512 << 20)
    vecs, threads = [1, 4, 70], [60000, 90000, 200000]
    arrays = [G.GGArray(pool, 4, v, 64) for v in vecs]
    orcs = [Oracle(4, v, 64) for v in vecs]
    batch = G.Batch(arrays)
    g = G.make_gen(G.GEN_KEYED, round=1, seed=5, tag_shift=20, tag=7)  # array 1 holds tag 8
    batch.insert_gen(g, threads)
    batch.step([g], [threads], G.RW_NONE)
    for i, (a, o) in enumerate(zip(arrays, orcs)):
        for _ in range(2):
            o.insert_gen(oracle.GEN_KEYED, threads[i], round=1, seed=5, tag_shift=20, tag=7 + i)
        assert_same(a, o, f"array {i}")
    batch.close()
    for a in arrays:
        a.close()
    pool.close()


@pytest.mark.parametrize("kind,V", [("bernoulli", 4096), ("bernoulli", 16), ("poisson", 16400), ("poisson", 64)])
def test_drawn_rounds_across_the_wrap(kind, V):
    """Thread 8435076 is the first past the wrap of seed 0's states (and a little before it for a round's)."""
    G = gg()
    n = 8435076 + 5000
    pool = G.Pool(2 << 30)
    a, o = G.GGArray(pool, 4, V, 1024), Oracle(4, V, 1024, forms=oracle.FORM_LIST)
    if kind == "bernoulli":
        a.insert_gen(G.make_gen(G.GEN_BERNOULLI, seed=3, round=7), n)
        o.insert_gen(oracle.GEN_BERNOULLI, n, seed=3, round=7)
    else:
        thr = wl.poisson_thresholds(3, 16)
        a.insert_gen(G.make_gen(G.GEN_POISSON, seed=3, round=5, max_count=16, thresholds=thr), n)
        o.insert_gen(oracle.GEN_POISSON, n, seed=3, round=5, max_count=16, thresholds=thr)
    np.testing.assert_array_equal(G.as_unsigned(a.flatten()), o.flatten())
    assert a.last_error() == 0
    a.close()
    o.close()
    pool.close()
