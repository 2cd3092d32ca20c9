"""GPU parity of buffer rounds on either side of the lines between their kernels' forms
for many LFVectors; against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elem,V,F,share", [
    (4, 600, 256, 1025), (8, 1024, 16, 2049),                      # eight waves per LFVector
    (4, 2048, 64, 1025), (4, 2049, 64, 3072), (8, 2049, 64, 1537),  # four; one up to 12 KiB; four past it
])
def test_dense_buffer_lines(elem, V, F, share):
    print(f"case dense lines elem={elem} V={V} F={F} share={share}", flush=True)
    rng = np.random.default_rng(V + share)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    n = V * share - 11  # a ragged last share
    for r in range(2):
        vals, _ = wl.random_round(rng, n, 1.0, elem)
        a.insert(dev(vals))
        o.insert(vals)
        assert_same(a, o, f"round {r}")
    a.close()
    o.close()
    pool.close()


@pytest.mark.parametrize("elem,V,F,kb", [
    (4, 700, 64, 9), (8, 1500, 16, 9), (4, 1500, 1, 20),              # eight waves per LFVector; four; eight
    (4, 2049, 64, 8), (8, 2049, 64, 9), (4, 2049, 64, 21), (8, 300, 256, 40),  # one; four; two launches
])
def test_segment_lines(elem, V, F, kb):
    print(f"case segment lines elem={elem} V={V} F={F} KiB={kb}", flush=True)
    rng = np.random.default_rng(V + kb)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    n = V * kb * 1024 // elem
    for r in range(2):
        w = np.exp(rng.standard_normal(V))
        lens = (w / w.sum() * n).astype(np.int64)
        lens[::7] = 0
        prefix = (3 * r + np.concatenate([[0], np.cumsum(lens)])).astype(np.uint64)
        vals, _ = wl.random_round(rng, n + 8, 1.0, elem)
        a.insert_segments(dev(vals), dev(prefix))
        o.insert_segments(vals, prefix)
        assert_same(a, o, f"segments {r}")
    a.close()
    o.close()
    pool.close()


@pytest.mark.parametrize("V,chunk,mc", [(8192, 256, 16), (8192, 512, 8), (2048, 257, 4)])
def test_counts_lines(V, chunk, mc):
    """A wave's largest shares (two owner-map passes), and the workgroup form just past the line."""
    print(f"case counts lines V={V} chunk={chunk} max={mc}", flush=True)
    rng = np.random.default_rng(V + chunk)
    pool = gg().Pool(1 << 30)
    a, o = both(4, V, 16, pool)
    n = V * chunk - 5
    counts = rng.integers(0, 2, size=n, dtype=np.uint8)
    counts.reshape(-1)[: 3 * chunk] = mc  # three full shares, the rest sparse
    counts[n // 2: n // 2 + chunk] = mc
    vals, _ = wl.random_round(rng, n * mc, 1.0, 4)
    a.insert_counts(dev(vals), dev(counts), mc)
    o.insert_counts(vals, counts, mc)
    assert_same(a, o, "counts")
    thr = [0] * 15 + [1 << 63]  # fifteen or sixteen elements a thread
    g = gg().make_gen(gg().GEN_POISSON, seed=7, round=3, max_count=16, thresholds=thr)
    m = V * min(chunk, 100)
    a.insert_gen(g, m)
    o.insert_gen(oracle.GEN_POISSON, m, seed=7, round=3, max_count=16, thresholds=thr)
    assert_same(a, o, "generated")
    a.close()
    o.close()
    pool.close()
