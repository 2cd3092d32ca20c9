"""GPU parity of the segment append with segments long enough for several
workgroups per LFVector: segments that start and end off lines and vectors, one
segment of most of the values, empty segments, a pair that decreases, small first
buckets (pieces across several buckets), and LFVectors frozen by an allocation
failure; against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg, gpu_flat, gpu_sizes

pytestmark = pytest.mark.gpu


def _lens(rng, V, total, shape):
    if shape == "even":
        lens = np.full(V, total // V)
    elif shape == "one":  # one LFVector takes nearly everything
        lens = rng.integers(0, 7, size=V)
        lens[V // 2] = total
    else:  # uneven, some empty
        w = np.exp(1.5 * rng.standard_normal(V))
        lens = (w / w.sum() * total).astype(np.int64)
        lens[::3] = 0
    return lens


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("V,F,total,shape", [
    (1, 1024, 1024, "even"),            # the last size of the one-launch form
    (1, 1024, 2049, "even"),            # just past it
    (1, 16, 8 * 1024, "even"),          # u32: the last size of the workgroup form, u64: past it
    (1, 16, 9 * 1024, "even"),
    (40, 1024, 40 * 4 * 1024, "one"),
    (1030, 64, 1030 * 1500, "uneven"),  # too many LFVectors for it
    (6, 1, 70001, "uneven"),
    (32, 1024, 300007, "uneven"),
    (64, 16, 200003, "one"),
    (700, 256, 1500001, "uneven"),
])
def test_long_segments(elem, V, F, total, shape):
    print(f"case segments elem={elem} V={V} F={F} total={total} {shape}", flush=True)
    G = gg()
    rng = np.random.default_rng(V + total)
    pool = G.Pool(512 << 20)
    a, o = both(elem, V, F, pool)
    vals, flags = wl.random_round(rng, 3 * V + 1, 0.5, elem)  # sizes off every alignment
    a.insert(dev(vals), dev(flags))
    o.insert(vals, flags)
    for r in range(2):
        lens = _lens(rng, V, total, shape)
        lead = r * 3  # the first segment does not start at the buffer's start
        prefix = (lead + np.concatenate([[0], np.cumsum(lens)])).astype(np.uint64)
        seg, _ = wl.random_round(rng, int(prefix[-1]) + 5, 1.0, elem)
        a.insert_segments(dev(seg), dev(prefix))
        assert o.insert_segments(seg, prefix) == oracle.OK
        assert_same(a, o, f"segments {r}")
    a.close()
    pool.close()


def test_long_segments_bad_pair_and_overlap():
    G = gg()
    rng = np.random.default_rng(5)
    pool = G.Pool(256 << 20)
    a, o = both(4, 5, 8, pool)
    prefix = np.array([0, 9000, 5000, 40000, 40000, 90000], dtype=np.uint64)  # pair 1 decreases, 0 and 2 overlap
    seg, _ = wl.random_round(rng, 60000, 1.0, 4)  # the last segment runs past the values
    a.insert_segments(dev(seg), dev(prefix))
    assert o.insert_segments(seg, prefix) == oracle.ERANGE
    assert a.last_error() == G.ERANGE
    assert gpu_sizes(a).tolist() == o.vector_sizes().tolist() == [9000, 0, 35000, 0, 0]
    np.testing.assert_array_equal(gpu_flat(a), o.flatten())
    a.close()
    pool.close()


def test_long_segments_failed_growth_freezes_one_lfvector():
    """The allocation that fails leaves its LFVector as it was; the others hold their segments."""
    G = gg()
    rng = np.random.default_rng(6)
    pool = G.Pool(256 << 20)
    V, per = 4, 30000
    a = G.GGArray(pool, 4, V, 1024)
    prefix = (np.arange(V + 1) * per).astype(np.uint64)
    seg, _ = wl.random_round(rng, V * per, 1.0, 4)
    pool.set_fault(3)
    a.insert_segments(dev(seg), dev(prefix))
    assert a.last_error() == G.ENOMEM
    sizes = gpu_sizes(a)
    assert sorted(sizes.tolist()) == [0] + [per] * (V - 1)
    want = np.concatenate([seg[v * per:(v + 1) * per] for v in range(V) if sizes[v]])
    np.testing.assert_array_equal(gpu_flat(a), want)
    a.close()
    pool.set_fault(0)
    assert pool.stats()["in_use"] == 0
    pool.close()
