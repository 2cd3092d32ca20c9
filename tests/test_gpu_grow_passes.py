"""GPU parity of counts rounds over LFVectors of so many tiles that their words are summed in
passes: the last round of one pass of 4096 tiles, one and four passes of 16384 with a
remainder, each with a round before it; against the CPU oracle, bit for bit."""
import numpy as np
import pytest

from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg

pytestmark = pytest.mark.gpu
TILE = 1024


@pytest.mark.parametrize("elem,V,F,n", [
    (4, 1, 64, 4096 * TILE),
    (8, 2, 1024, 2 * (4096 * TILE + 1)),
    (4, 1, 1024, 16384 * TILE),
    (4, 1, 1024, 16385 * TILE - 3),
    (4, 2, 16, 2 * (16384 * TILE + 65 * TILE + 9)),
])
def test_growth_in_passes(elem, V, F, n):
    print(f"case growth passes elem={elem} V={V} F={F} n={n}", flush=True)
    rng = np.random.default_rng(V + elem)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    vals, _ = wl.random_round(rng, n, 1.0, elem)
    dv = dev(vals)
    for r in range(2):
        counts = (rng.random(n, dtype=np.float32) < (0.5, 0.02)[r]).astype(np.uint8)
        a.insert_counts(dv, dev(counts), 1)
        o.insert_counts(vals, counts, 1)
        assert_same(a, o, f"round {r}")
    a.close()
    o.close()
    pool.close()
