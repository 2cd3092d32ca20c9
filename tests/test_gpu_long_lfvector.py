"""The tile table of many LFVectors when a few of them hold most elements (sixteen lanes
write a short LFVector's tiles, a whole wave a long one's): lengths on either side of
that line, several long ones in one wave, one array and a batch, against the CPU oracle,
bit for bit; and the time against the count of LFVectors that has a wave each."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Oracle
from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import gg
from tests.test_gpu_loose_bound import _us

pytestmark = pytest.mark.gpu
LINE = 256 * 4096  # u32 elements of 256 tiles


def _prefix(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)


@pytest.mark.parametrize("V", [(16384,), (16000, 385)])
def test_table_with_long_lfvectors(V):
    print(f"case long lfvectors V={V}", flush=True)
    G = gg()
    rng = np.random.default_rng(len(V))
    pool = G.Pool(2 << 30)
    arrays = [G.GGArray(pool, 4, v, 64) for v in V]
    orcs = [Oracle(4, v, 64, forms=oracle.FORM_LIST) for v in V]
    for k, (a, o, v) in enumerate(zip(arrays, orcs, V)):
        lens = rng.integers(0, 400, size=v)
        if k == len(V) - 1:
            lens[:4] = LINE + 4095, LINE + 4096, 2 * LINE + 1, 7  # one wave's four: short, long, long, short
            lens[v - 1] = 3 * LINE
        prefix = _prefix(lens)
        seg, _ = wl.random_round(rng, int(prefix[-1]), 1.0, 4)
        a.insert_segments(G.to_device(seg), G.to_device(prefix))
        assert o.insert_segments(seg, prefix) == oracle.OK
        o.rw(oracle.OP_MUL3ADD1)
    if len(V) > 1:
        batch = G.Batch(arrays)
        batch.rw(G.MUL3ADD1)
        out = torch.empty(sum(o.size() for o in orcs), dtype=torch.int32, device="cuda")
        batch.flatten_into(out)
        flat = G.as_unsigned(out)
        batch.close()
    else:
        arrays[0].rw(G.MUL3ADD1)
        flat = G.as_unsigned(arrays[0].flatten())
    np.testing.assert_array_equal(flat, np.concatenate([o.flatten() for o in orcs]))
    for a, o in zip(arrays, orcs):
        assert a.last_error() == 0
        a.close()
        o.close()
    pool.close()


def test_table_time_of_one_long_lfvector():
    """The table of 2^28 elements in one LFVector, as the time by which an r/w after a change of the sizes
    exceeds one without: some 150 us of a wave either side of the count; 420 us with sixteen lanes."""
    G = gg()
    fill = torch.empty(48 << 20, dtype=torch.int32, device="cuda")
    took = []
    for V in (16383, 16384):
        n = 1 << 28
        pool = G.Pool(5 << 30)
        a = G.GGArray(pool, 4, V, 64)
        lens = np.full(V, 3)
        lens[V // 2] = n - 3 * V
        a.insert_segments(torch.empty(n, dtype=torch.int32, device="cuda"), G.to_device(_prefix(lens)))
        one = torch.zeros(V, dtype=torch.int32, device="cuda")

        def changed():
            a.insert(one)
            return _us(lambda: a.rw(G.ADD1), fill, reps=1)
        a.rw(G.ADD1)
        took.append(min(changed() for _ in range(12)) - _us(lambda: a.rw(G.ADD1), fill))
        a.close()
        pool.close()
    print(f"a wave {took[0]:.0f} us, {took[1]:.0f} us", flush=True)
    assert took[1] < 1.7 * took[0]
