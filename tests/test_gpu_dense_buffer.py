"""GPU parity of rounds from a buffer without flags, one workgroup per LFVector:
shares at the edge of the one-wave form (4 KiB), off lines and vectors, ragged and
empty last LFVectors, pieces across small buckets, payloads off 16-byte alignment,
both workgroup sizes, and an allocation failure; against the CPU oracle, bit for
bit."""
import numpy as np
import pytest

from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg, gpu_flat, gpu_sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("V,F,n", [
    (1, 1024, 1024),             # u32: the one-wave form's largest share
    (1, 1024, 1025),
    (3, 1, 3 * 9000 - 7),        # a piece over several buckets, a ragged last LFVector
    (40, 64, 40 * 4096 + 13),
    (512, 1024, 512 * 5001 - 1),
    (1024, 16, 1024 * 1500 - 2999),   # the last LFVectors get nothing or little
    (1025, 256, 1025 * 1100 + 17),    # the smaller workgroup
])
def test_dense_buffer_rounds(elem, V, F, n):
    print(f"case dense buffer elem={elem} V={V} F={F} n={n}", flush=True)
    rng = np.random.default_rng(V + n)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    for r in range(3):
        vals, _ = wl.random_round(rng, n + r, 1.0, elem)
        t = dev(np.concatenate([vals[:1], vals]))[1:] if r == 1 else dev(vals)  # element-aligned only
        a.insert(t)
        o.insert(vals, None)
        assert_same(a, o, f"round {r}")
    a.close()
    pool.close()


def test_dense_buffer_failed_growth_freezes_one_lfvector():
    G = gg()
    rng = np.random.default_rng(9)
    pool = G.Pool(256 << 20)
    V, per = 4, 20000
    a = G.GGArray(pool, 4, V, 1024)
    vals, _ = wl.random_round(rng, V * per, 1.0, 4)
    pool.set_fault(5)
    a.insert(dev(vals))
    assert a.last_error() == G.ENOMEM
    sizes = gpu_sizes(a)
    assert sorted(sizes.tolist()) == [0] + [per] * (V - 1)
    want = np.concatenate([vals[v * per:(v + 1) * per] for v in range(V) if sizes[v]])
    np.testing.assert_array_equal(gpu_flat(a), want)
    a.close()
    pool.set_fault(0)
    assert pool.stats()["in_use"] == 0
    pool.close()
