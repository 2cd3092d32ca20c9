"""GPU parity of multi-element rounds that run one wave per LFVector (many LFVectors
of at most 512 logical threads): shares at the edges of the lanes' 4 and 8 threads and
just past the form's range, ragged and empty last LFVectors, counts that fill several
owner-map passes, tiny first buckets, and an allocation failure; against the CPU
oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg, gpu_flat, gpu_sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elem,V,F,chunk,short,mc", [
    (8, 2048, 1024, 1, 0, 16),
    (4, 2048, 1, 256, 3, 5),
    (8, 2048, 1, 257, 300, 5),     # the last LFVector gets nothing, the one before a part
    (4, 2048, 1024, 512, 1, 16),   # up to 8192 outputs: several passes
    (4, 2048, 16, 513, 0, 3),      # the workgroup form
    (4, 2047, 16, 200, 7, 3),
    (8, 4100, 64, 63, 100, 16),
])
def test_count_rounds(elem, V, F, chunk, short, mc):
    print(f"case count waves elem={elem} V={V} F={F} chunk={chunk} max={mc}", flush=True)
    rng = np.random.default_rng(V + chunk)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    n = V * chunk - short
    for r in range(2):
        counts = rng.integers(0, mc + 1, size=n, dtype=np.uint8)
        if r:
            counts[: n // 2] = mc
        vals, _ = wl.random_round(rng, n * mc, 1.0, elem)
        a.insert_counts(dev(vals), dev(counts), mc)
        o.insert_counts(vals, counts, mc)
        assert_same(a, o, f"counts {r}")
    thr = wl.poisson_thresholds(3, 16)
    g = gg().make_gen(gg().GEN_POISSON, seed=7, round=3, max_count=16, thresholds=thr)
    a.insert_gen(g, n)
    o.insert_gen(oracle.GEN_POISSON, n, seed=7, round=3, max_count=16, thresholds=thr)
    assert_same(a, o, "poisson")
    a.close()
    pool.close()


def test_count_waves_failed_growth_freezes_one_lfvector():
    G = gg()
    rng = np.random.default_rng(3)
    pool = G.Pool(256 << 20)
    V, chunk = 2048, 100
    a = G.GGArray(pool, 4, V, 64)
    counts = np.full(V * chunk, 2, np.uint8)
    vals, _ = wl.random_round(rng, 2 * V * chunk, 1.0, 4)
    pool.set_fault(777)
    a.insert_counts(dev(vals), dev(counts), 2)
    assert a.last_error() == G.ENOMEM
    sizes = gpu_sizes(a)
    assert sizes.max() == 2 * chunk and (sizes == 0).sum() == 1 and sizes.sum() == 2 * chunk * (V - 1)
    keep = np.repeat(sizes > 0, 2 * chunk)
    np.testing.assert_array_equal(gpu_flat(a), vals[keep])
    a.close()
    pool.set_fault(0)
    assert pool.stats()["in_use"] == 0
    pool.close()
