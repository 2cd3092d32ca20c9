"""GPU parity of packed rounds at the edges of their short-tile forms: one wave per
LFVector (2048 LFVectors or more, up to 8 KiB of values each on average) and just past
it, tiles of 1 to 33 and of 1008 to 1024 logical threads at every alignment of the
counts (the totals are read 16 bytes at a time), ragged and empty last tiles, runs
across tiny buckets, and an allocation failure; against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg, gpu_flat, gpu_sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elem,V,F,chunk,short,mc", [
    (8, 2048, 1024, 1, 0, 255),
    (4, 2048, 1, 17, 5, 9),
    (8, 2048, 4, 100, 333, 20),    # three runs or more per LFVector
    (8, 2048, 1024, 256, 1, 8),    # 8 KiB of values on average: the wave form's largest
    (8, 2048, 1024, 256, 0, 9),    # past it: the workgroup form
    (4, 2047, 64, 200, 0, 6),
    (4, 4096, 256, 300, 301, 12),
])
def test_packed_waves(elem, V, F, chunk, short, mc):
    print(f"case packed waves elem={elem} V={V} F={F} chunk={chunk} max={mc}", flush=True)
    rng = np.random.default_rng(V + chunk + mc)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    n = V * chunk - short
    for r in range(3):
        counts = rng.integers(0, mc + 1, size=n, dtype=np.uint8)
        if chunk == 256 and r == 0:
            counts[:] = mc // 2  # the average at the form's edge exactly (mc = 8)
        total = int(counts.sum(dtype=np.uint64))
        vals, _ = wl.random_round(rng, total + 1, 1.0, elem)
        a.insert_packed(dev(vals), dev(counts), total)
        assert o.insert_packed(vals, counts) == oracle.OK
        assert_same(a, o, f"round {r}")
    a.close()
    pool.close()


@pytest.mark.parametrize("chunk", [1, 2, 15, 16, 17, 31, 32, 33, 1008, 1009, 1023, 1024, 1025, 2047])
def test_packed_totals_at_every_alignment(chunk):
    rng = np.random.default_rng(chunk)
    pool = gg().Pool(256 << 20)
    V = 18  # more than one group of 16 tiles
    n = V * chunk
    raw = rng.integers(0, 256, size=n + 16, dtype=np.uint8)
    draw = dev(raw)
    for shift in (0, 1, 7, 13):
        a, o = both(4, V, 16, pool)
        counts = raw[shift: shift + n]
        vals, _ = wl.random_round(rng, int(counts.sum(dtype=np.uint64)), 1.0, 4)
        a.insert_packed(dev(vals), draw[shift: shift + n])
        assert o.insert_packed(vals, np.ascontiguousarray(counts)) == oracle.OK
        assert_same(a, o, f"chunk {chunk} shift {shift}")
        a.close()
        o.close()
    pool.close()


def test_packed_waves_failed_growth_freezes_one_lfvector():
    G = gg()
    rng = np.random.default_rng(3)
    pool = G.Pool(256 << 20)
    V, chunk = 2048, 30
    a = G.GGArray(pool, 4, V, 64)
    counts = np.full(V * chunk, 3, np.uint8)
    vals, _ = wl.random_round(rng, 3 * V * chunk, 1.0, 4)
    pool.set_fault(1000)
    a.insert_packed(dev(vals), dev(counts))
    assert a.last_error() == G.ENOMEM
    sizes = gpu_sizes(a)
    assert (sizes == 0).sum() == 1 and sizes.sum() == 3 * chunk * (V - 1)
    np.testing.assert_array_equal(gpu_flat(a), vals[np.repeat(sizes > 0, 3 * chunk)])
    a.close()
    pool.set_fault(0)
    assert pool.stats()["in_use"] == 0
    pool.close()
