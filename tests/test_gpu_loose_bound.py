"""Access by global index when the host's bound of the size is far above it (rounds that
inserted nothing): the form follows the size itself.  Contents on either side of the
sizes where the form changes, against the CPU oracle, bit for bit; and the time, against
the same array under a close bound."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import dev, gg, gpu_flat

pytestmark = pytest.mark.gpu
EMPTY_ROUND = 17_000_000  # threads; past 64 MiB of either element


def _loosen(a, elem):
    v = torch.zeros(EMPTY_ROUND, dtype=torch.int32 if elem == 4 else torch.int64, device="cuda")
    a.insert(v, torch.zeros(EMPTY_ROUND, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("elem,V,n", [
    (4, 300, 1), (8, 5, 2000), (4, 300, (1 << 20) - 1), (8, 2000, (1 << 19) - 1), (8, 2000, 1 << 19), (4, 40000, (1 << 20) + 7),
    (8, 300, (1 << 23) - 1), (8, 300, 1 << 23), (4, 300, (1 << 24) - 1), (4, 9, (1 << 24) + 5),
])
def test_rw_global_under_a_loose_bound(elem, V, n):
    print(f"case loose bound elem={elem} V={V} n={n}", flush=True)
    G = gg()
    rng = np.random.default_rng(n)
    pool = G.Pool(1 << 30)
    a, o = G.GGArray(pool, elem, V, 64), Oracle(elem, V, 64, forms=oracle.FORM_LIST)
    vals, _ = wl.random_round(rng, n, 1.0, elem)
    a.insert(dev(vals))
    o.insert(vals)
    _loosen(a, elem)
    for _ in range(2):
        a.rw_global(G.MUL3ADD1)
        o.rw(oracle.OP_MUL3ADD1)
    assert a.size() == n and a.last_error() == 0
    np.testing.assert_array_equal(gpu_flat(a), o.flatten())
    a.close()
    o.close()
    pool.close()


def _us(call, fill, reps=20):
    best = float("inf")
    for i in range(reps):
        fill.fill_(i)  # the host is done with the launch before the GPU comes to it
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        call()
        e1.record()
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1) * 1e3)
    return best


def test_rw_global_time_follows_the_size():
    """7 against 5 us here; 32 us where the form followed the bound."""
    G = gg()
    pool = G.Pool(1 << 30)
    fill = torch.empty(48 << 20, dtype=torch.int32, device="cuda")
    a = G.GGArray(pool, 4, 512, 64)
    a.insert(torch.arange(30000, dtype=torch.int32, device="cuda"))
    close = _us(lambda: a.rw_global(G.ADD1), fill)
    _loosen(a, 4)
    loose = _us(lambda: a.rw_global(G.ADD1), fill)
    print(f"close {close:.1f} us, loose {loose:.1f} us", flush=True)
    assert loose < 2.5 * close
    a.close()
    pool.close()
