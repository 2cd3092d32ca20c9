"""GPU parity of flagged rounds from buffers over LFVectors of several tiles, at every
way a share can sit on the 16-byte vectors: thread counts of every residue (the last
vector of the buffers is loaded before its place and shifted), shares that start
anywhere, payloads and flags off their alignment, ragged and empty last LFVectors,
tiles across small buckets, and LFVectors of more tiles than a wave's pass (256) and a
workgroup's (4096); against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from oracle import Oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg

pytestmark = pytest.mark.gpu
TILE = 4096


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("V,F,n", [
    (1, 1024, TILE + 1), (1, 1024, 2 * TILE - 1), (1, 64, 2 * TILE), (2, 16, 2 * TILE + 2), (2, 1, 2 * TILE + 3),
    (3, 1024, 3 * (TILE + 2) - 2), (5, 256, 5 * 9001), (7, 1, 7 * 5003 - 4), (16, 1024, 16 * 6001 - 6050),
    (1, 1024, 256 * TILE), (1, 1024, 256 * TILE + 5),
])
def test_flag_rounds_any_share(elem, V, F, n):
    print(f"case flag rounds elem={elem} V={V} F={F} n={n}", flush=True)
    rng = np.random.default_rng(V + n)
    pool = gg().Pool(512 << 20)
    a, o = both(elem, V, F, pool)
    for r, (p, so, fo) in enumerate([(0.5, 0, 0), (1.0, 1, 3), (0.03, 0, 1), (0.9, 1, 2)]):
        vals, flags = wl.random_round(rng, n, p, elem)
        dv = dev(np.concatenate([vals[:1], vals]))[1:] if so else dev(vals)  # element-aligned only
        df = dev(np.concatenate([np.ones(fo, np.uint8), flags * np.uint8(r + 1)]))[fo:]  # any byte, any value but 0
        a.insert(dv, df)
        o.insert(vals, flags)
        assert_same(a, o, f"round {r}")
    a.close()
    o.close()
    pool.close()


def test_flag_rounds_more_tiles_than_a_workgroup_pass():
    n = 4097 * TILE + 77
    rng = np.random.default_rng(2)
    pool = gg().Pool(1 << 30)
    a, o = gg().GGArray(pool, 4, 1, 1024), Oracle(4, 1, 1024, forms=oracle.FORM_LIST)
    for p in (0.3, 0.01):
        vals, flags = wl.random_round(rng, n, p, 4)
        a.insert(dev(vals), dev(flags))
        o.insert(vals, flags)
    np.testing.assert_array_equal(gg().as_unsigned(a.flatten()), o.flatten())
    assert a.last_error() == 0
    a.close()
    o.close()
    pool.close()
