"""Served appends at the edges of their forms (a workgroup per LFVector for at most 8
tiles each and at most 64 LFVectors, else a wave per tile), mixed in one step with each
other and with r/w and flatten requests, from tiny first buckets and off every
alignment; and an append whose allocation fails.  Against the CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, gg, gpu_sizes

pytestmark = pytest.mark.gpu
TILE = 4096
SHIFT = 20
KEYS = dict(seed=3, append_round=7, append_shift=SHIFT)


def _serve(arrays, kind, target, length):
    G = gg()
    arena = torch.zeros(16 << 20, dtype=torch.uint8, device="cuda")
    sv = G.Server(arrays, arena, 1 << 40, mode=G.SERVE_BATCHED, lanes=1, **KEYS)
    res = sv.run(np.zeros(len(kind), np.uint64), np.array(kind, np.uint8), np.array(target, np.uint32),
                 np.array(length, np.uint32))
    sv.close()
    torch.cuda.synchronize()
    return res


def _append(o, n, r):
    return o.insert_gen(oracle.GEN_KEYED, n, seed=KEYS["seed"], round=KEYS["append_round"], tag_shift=SHIFT, tag=r)


@pytest.mark.parametrize("elem", [4, 8])
def test_served_append_forms(elem):
    G = gg()
    shapes = [(1, 1, 1), (1, 64, 8 * TILE), (1, 64, 8 * TILE + 1), (1, 1024, 200_001), (3, 16, 3 * 8 * TILE),
              (3, 16, 3 * 8 * TILE + 1), (64, 16, 64 * 700 - 13), (65, 16, 65 * 700 - 13), (64, 1, 3), (65, 1, 70),
              (7, 1, 7 * 5000)]
    pool = G.Pool(1 << 30)
    arrays = [G.GGArray(pool, elem, V, F) for V, F, _ in shapes]
    orcs = [Oracle(elem, V, F) for V, F, _ in shapes]
    kind, target, length = [], [], []
    for k in (wl.REQ_APPEND, wl.REQ_RW, wl.REQ_APPEND, wl.REQ_FLATTEN, wl.REQ_APPEND):
        # request j of a pass goes to array j, so that every step mixes all shapes
        for a, (_, _, n) in enumerate(shapes):
            kind.append(k)
            target.append(a)
            length.append(max(1, n - len(kind) % 3) if k == wl.REQ_APPEND else 0)
            if k == wl.REQ_APPEND:
                _append(orcs[a], length[-1], len(kind) - 1)
            elif k == wl.REQ_RW:
                orcs[a].rw(oracle.OP_ADD1)
    res = _serve(arrays, kind, target, length)
    assert (res["status"] == 0).all()
    for a, (arr, o) in enumerate(zip(arrays, orcs)):
        assert_same(arr, o, f"array {a} {shapes[a]}")
        arr.close()
        o.close()
    pool.close()


@pytest.mark.parametrize("n", [3 * 5000, 3 * 9 * TILE])  # a workgroup per LFVector; a wave per tile
def test_served_append_that_cannot_allocate(n):
    G = gg()
    pool = G.Pool(256 << 20)
    a = G.GGArray(pool, 4, 3, 64)
    pool.set_fault(5)
    _serve([a], [wl.REQ_APPEND], [0], [n])
    assert a.last_error() == G.ENOMEM
    sizes = gpu_sizes(a)
    assert (sizes == 0).sum() == 1 and sizes.sum() == n - n // 3
    a.close()
    pool.set_fault(0)
    assert pool.stats()["in_use"] == 0
    pool.close()
