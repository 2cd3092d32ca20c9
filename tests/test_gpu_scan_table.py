"""GPU parity of the prefix scan that writes the tile table in its launch: LFVector
counts around a workgroup's four and the form's last (4096), uneven and empty
LFVectors, the prefix asked for before and after a table exists, and the place of a
tile found from uneven lengths in arrays below the table's size; against the CPU
oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, gg

pytestmark = pytest.mark.gpu
BIG = 2048 * 4096 + 5  # u32 elements of the smallest array with a table


@pytest.mark.parametrize("V,F", [(1, 1024), (5, 4096), (511, 1024), (4096, 256), (4097, 256)])
def test_scan_with_table(V, F):
    print(f"case scan table V={V} F={F}", flush=True)
    G = gg()
    rng = np.random.default_rng(V)
    pool = G.Pool(1 << 30)
    a, o = G.GGArray(pool, 4, V, F), Oracle(4, V, F, forms=oracle.FORM_LIST)
    for r, n in enumerate([BIG, BIG // 5, 3 * V]):
        lens = rng.integers(0, 3, size=V) * (n // V) if V > 1 else np.array([n])
        if r == 0:
            lens[V // 3] += n - min(n, int(lens.sum()))
        prefix = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
        seg, _ = wl.random_round(rng, int(prefix[-1]), 1.0, 4)
        a.insert_segments(G.to_device(seg), G.to_device(prefix))
        assert o.insert_segments(seg, prefix) == oracle.OK
        if r != 1:  # the offsets first: without a table, then with one large enough or not
            np.testing.assert_array_equal(a.prefix().cpu().numpy().astype(np.uint64), o.prefix())
        a.rw(G.MUL3ADD1)
        o.rw(oracle.OP_MUL3ADD1)
        np.testing.assert_array_equal(a.prefix().cpu().numpy().astype(np.uint64), o.prefix())
        np.testing.assert_array_equal(G.as_unsigned(a.flatten()), o.flatten())
        assert a.size() == o.size() and a.last_error() == 0
    a.close()
    o.close()
    pool.close()


@pytest.mark.parametrize("V,lens", [
    (300, "even"), (300, "rising"), (300, "one"), (300, "holes"), (1, "even"), (3000, "rising"),
])
def test_walk_of_uneven_small_arrays(V, lens):
    G = gg()
    rng = np.random.default_rng(V)
    pool = G.Pool(512 << 20)
    a, o = G.GGArray(pool, 8, V, 64), Oracle(8, V, 64)
    n = {"even": np.full(V, 3000), "rising": np.arange(V) * (6000 // V + 1), "one": np.zeros(V, int),
         "holes": rng.integers(0, 2, V) * rng.integers(0, 6000, V)}[lens]
    if lens == "one":
        n[-1] = 900_000
    prefix = np.concatenate([[0], np.cumsum(n)]).astype(np.uint64)
    seg, _ = wl.random_round(rng, int(prefix[-1]), 1.0, 8)
    a.insert_segments(G.to_device(seg), G.to_device(prefix))
    assert o.insert_segments(seg, prefix) == oracle.OK
    a.rw(G.MUL3ADD1)
    o.rw(oracle.OP_MUL3ADD1)
    assert_same(a, o, lens)
    a.close()
    pool.close()


@pytest.mark.parametrize("V,F", [((16383,), 64), ((16384,), 1), ((16000, 383), 64), ((383, 16001), 1)])
def test_table_of_many_lfvectors(V, F):
    """The last LFVector count with a wave each and the first with sixteen lanes, one
    array and a batch; empty LFVectors and one of 17 or more buckets of F = 1."""
    print(f"case table of many V={V} F={F}", flush=True)
    G = gg()
    rng = np.random.default_rng(sum(V))
    pool = G.Pool(1 << 30)
    arrays, orcs = [G.GGArray(pool, 4, v, F) for v in V], [Oracle(4, v, F) for v in V]
    batch = G.Batch(arrays) if len(V) > 1 else None
    for r in range(2):
        for a, o, v in zip(arrays, orcs, V):
            lens = rng.integers(0, 3, size=v) * (BIG // v // (2 * r + 1))
            lens[v // 2] += 300_000
            prefix = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
            seg, _ = wl.random_round(rng, int(prefix[-1]), 1.0, 4)
            a.insert_segments(G.to_device(seg), G.to_device(prefix))
            assert o.insert_segments(seg, prefix) == oracle.OK
            o.rw(oracle.OP_MUL3ADD1)
        if batch:
            batch.rw(G.MUL3ADD1)
            out = torch.empty(sum(o.size() for o in orcs), dtype=torch.int32, device="cuda")
            batch.flatten_into(out)
            flat = G.as_unsigned(out)
        else:
            arrays[0].rw(G.MUL3ADD1)
            flat = G.as_unsigned(arrays[0].flatten())
        np.testing.assert_array_equal(flat, np.concatenate([o.flatten() for o in orcs]))
    if batch:
        batch.close()
    for a, o in zip(arrays, orcs):
        assert a.last_error() == 0
        a.close()
        o.close()
    pool.close()
