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
