"""GPU parity of packed rounds in which some of many short tiles are long (the whole
workgroup copies those of its four waves): several in one workgroup and in the last,
which has fewer than four LFVectors, small and large first buckets, lengths around the
line (32 KiB), rounds on top of each other, a failed allocation and a refused round;
against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg, gpu_flat, gpu_sizes

pytestmark = pytest.mark.gpu
LINE = 32768  # bytes


def _counts(rng, V, chunk, full, elem):
    c = rng.integers(0, 2, size=(V, chunk), dtype=np.uint8)
    c[full] = rng.integers(200, 256, size=(len(full), chunk), dtype=np.uint8)
    per = LINE // elem  # three tiles of exactly the line, one more and one fewer
    for k, extra in ((9, 0), (10, 1), (14, -1)):
        c[k] = 0
        c[k, :per // 200] = 200
        c[k, per // 200] = per % 200 + extra
    return c.ravel()


@pytest.mark.parametrize("elem,V,F,chunk,short", [(4, 2049, 64, 1000, 0), (8, 2050, 1, 300, 7), (4, 4096, 1024, 500, 0)])
def test_packed_long_tiles(elem, V, F, chunk, short):
    print(f"case packed long elem={elem} V={V} F={F} chunk={chunk}", flush=True)
    rng = np.random.default_rng(V + chunk)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    full = np.array([0, 4, 5, 6, 7, V - 1])
    for r in range(3):
        counts = _counts(rng, V, chunk, full, elem)[: V * chunk - short]
        total = int(counts.sum(dtype=np.uint64))
        vals, _ = wl.random_round(rng, total + 3, 1.0, elem)
        a.insert_packed(dev(vals), dev(counts), total)
        assert o.insert_packed(vals, counts) == oracle.OK
        assert_same(a, o, f"round {r}")
    a.insert_packed(dev(vals), dev(counts), total - 1)  # one value too few: nothing is inserted
    assert a.last_error() == gg().ERANGE
    np.testing.assert_array_equal(gpu_sizes(a), o.vector_sizes())
    a.close()
    o.close()
    pool.close()


@pytest.mark.parametrize("fault", [1, 9, 30])
def test_packed_long_tiles_failed_growth(fault):
    """One allocation fails; its LFVector, long or short, keeps nothing, the others their rounds."""
    G = gg()
    rng = np.random.default_rng(fault)
    pool = G.Pool(256 << 20)
    V, chunk = 2048, 700
    a = G.GGArray(pool, 4, V, 64)
    counts = _counts(rng, V, chunk, np.arange(8), 4)
    vals, _ = wl.random_round(rng, int(counts.sum(dtype=np.uint64)), 1.0, 4)
    pool.set_fault(fault)
    a.insert_packed(dev(vals), dev(counts))
    assert a.last_error() == G.ENOMEM
    want = counts.reshape(V, chunk).sum(1, dtype=np.uint64)
    sizes = gpu_sizes(a)
    lost = np.nonzero(sizes != want)[0]
    assert lost.size == 1 and sizes[lost[0]] == 0
    keep = np.repeat(np.arange(V) != lost[0], want.astype(np.int64))
    np.testing.assert_array_equal(gpu_flat(a), vals[keep])
    a.close()
    pool.set_fault(0)
    assert pool.stats()["in_use"] == 0
    pool.close()
