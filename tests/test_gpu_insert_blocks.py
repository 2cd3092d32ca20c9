"""GPU parity of 0/1 rounds of one tile per LFVector (a workgroup per LFVector): shares
at the edges of each workgroup shape (256, 1024 and 4096 threads, 2048 LFVectors),
ragged and empty last LFVectors, tiny first buckets, flags from buffers off their
alignment and drawn by the producer, and an allocation failure; against the CPU
oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg, gpu_flat, gpu_sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("V,F,chunk,short", [
    (1, 1, 1, 0), (3, 1, 4096, 5), (40, 64, 4095, 4000), (7, 1024, 1025, 0), (512, 16, 1024, 1030),
    (2047, 16, 256, 3), (2048, 16, 256, 0), (2048, 1, 257, 300), (2049, 64, 1025, 1), (2048, 1024, 700, 0),
])
def test_block_rounds(elem, V, F, chunk, short):
    print(f"case block rounds elem={elem} V={V} F={F} chunk={chunk} short={short}", flush=True)
    G = gg()
    rng = np.random.default_rng(V + chunk)
    pool = G.Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    n = V * chunk - short
    for r, (p, so, fo) in enumerate([(0.5, 0, 0), (0.02, 1, 3), (1.0, 0, 1)]):
        vals, flags = wl.random_round(rng, n, p, elem)
        dv = dev(np.concatenate([vals[:1], vals]))[1:] if so else dev(vals)
        a.insert(dv, dev(np.concatenate([np.ones(fo, np.uint8), flags]))[fo:])
        o.insert(vals, flags)
        assert_same(a, o, f"flags {r}")
        a.insert_gen(G.make_gen(G.GEN_BERNOULLI, seed=9, round=r), n)
        o.insert_gen(oracle.GEN_BERNOULLI, n, seed=9, round=r)
        assert_same(a, o, f"bernoulli {r}")
    a.close()
    pool.close()


@pytest.mark.parametrize("V,chunk", [(4, 4000), (2048, 100)])
def test_block_rounds_failed_growth_freezes_one_lfvector(V, chunk):
    G = gg()
    rng = np.random.default_rng(V)
    pool = G.Pool(256 << 20)
    a = G.GGArray(pool, 4, V, 64)
    n = V * chunk
    vals, flags = wl.random_round(rng, n, 0.5, 4)
    pool.set_fault(V + 2)
    a.insert(dev(vals), dev(flags))
    assert a.last_error() == G.ENOMEM
    want = flags.reshape(V, chunk).sum(1)
    sizes = gpu_sizes(a)
    lost = np.nonzero(sizes != want)[0]
    assert lost.size == 1 and sizes[lost[0]] == 0
    keep = flags.astype(bool).reshape(V, chunk)
    keep[lost[0]] = False
    np.testing.assert_array_equal(gpu_flat(a), vals[keep.ravel()])
    a.close()
    pool.set_fault(0)
    assert pool.stats()["in_use"] == 0
    pool.close()
