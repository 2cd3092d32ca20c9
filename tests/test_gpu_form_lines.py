"""GPU parity of buffer rounds on either side of the lines between their kernels' forms
for many LFVectors; against the CPU oracle, bit for bit."""
import numpy as np
import pytest

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
