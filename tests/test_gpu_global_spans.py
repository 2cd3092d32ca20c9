"""GPU parity of access by global index at the edges of its search: spans that reach
one, eight, nine and hundreds of LFVectors, empty LFVectors between long ones, spans
across several small buckets, more LFVectors than a workgroup keeps offsets for (one
and two levels of samples), and read counts around a workgroup's share; against the
CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("V,F,n", [
    (1, 1024, 8192),
    (5, 1, 40001),
    (64, 1024, 64 * 256),      # u32: a span of 2048 reaches 8 LFVectors
    (64, 1024, 64 * 230),      # and 9 or 10
    (2048, 16, 2048 * 9 + 5),  # the whole offset array in LDS
    (2049, 16, 2049 * 9),      # every second offset
    (70000, 4, 70000 * 3),     # every 64th
    (600, 1024, 700000),       # the span form from here on (2 KiB spans)
    (20000, 16, 600000),       # short LFVectors: elements one by one within a span
    (300, 1024, 18000000),     # 8 KiB spans
])
def test_global_access(elem, V, F, n):
    print(f"case global elem={elem} V={V} F={F} n={n}", flush=True)
    G = gg()
    rng = np.random.default_rng(V + n)
    pool = G.Pool(512 << 20)
    a, o = G.GGArray(pool, elem, V, F), Oracle(elem, V, F)
    for r in range(2):
        vals, flags = wl.random_round(rng, n, 0.8, elem)
        if r:  # a run of LFVectors gets nothing more, and the last ones too
            flags[n // 3: n // 2] = 0
            flags[-n // 7:] = 0
        a.insert(G.to_device(vals), G.to_device(flags))
        o.insert(vals, flags)
        if r == 0 and V > 1:
            a.shrink(1, 1)  # only the second round's elements stay: LFVectors in the middle are empty
            o.shrink(1, 1)
    a.rw_global(G.MUL3ADD1)
    o.rw(oracle.OP_MUL3ADD1)
    assert_same(a, o, "rw by global index")
    size = o.size()
    flat = o.flatten()
    for reads in (1, 1023, 1025, 30000, (1 << 20) - 1, (1 << 20) + 5):
        idx = rng.integers(0, size, reads, dtype=np.uint64)
        idx[0], idx[-1] = 0, size - 1
        got = G.as_unsigned(a.gather(torch.from_numpy(idx.view(np.int64)).cuda()))
        np.testing.assert_array_equal(got, flat[idx])
    got = G.as_unsigned(a.gather(torch.arange(size, dtype=torch.int64, device="cuda")))
    np.testing.assert_array_equal(got, flat)
    assert a.last_error() == 0
    a.close()
    o.close()
    pool.close()
