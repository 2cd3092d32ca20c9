"""GPU parity of a batch's shrinks where most LFVectors of a free list line up and the rest of
the pass does not (an array longer than a pass, and one created after a gap); sizes, contents
and the pool's counts against the CPU oracle."""
import numpy as np
import pytest

from oracle import Oracle
from tests.gpu_util import assert_same, dev, gg

pytestmark = pytest.mark.gpu


def test_batch_chains_over_lists_that_partly_line_up():
    G = gg()
    rng = np.random.default_rng(11)
    pool = G.Pool(1 << 30)
    shapes = [(70000, 2), (20000, 2), (100, 16)]
    arrays, orcs = [], []
    for V, F in shapes:
        arrays.append(G.GGArray(pool, 4, V, F))
        orcs.append(Oracle(4, V, F))
        G.GGArray(pool, 4, 77, 4).close()  # shifts the next array's free lists
    batch = G.Batch(arrays)
    for r, (num, den) in enumerate(((1, 3), (1, 1), (2, 3), (1, 1))):
        print(f"case batch chains round {r}", flush=True)
        for a, o, (V, F) in zip(arrays, orcs, shapes):
            n = rng.integers(0, 9, V) * (rng.random(V) < 0.7)
            n[(r * 7919) % V] += 150_000
            pre = np.concatenate([[0], np.cumsum(n)]).astype(np.uint64)
            vals = rng.integers(0, 1 << 31, int(pre[-1])).astype(np.uint32)
            a.insert_segments(dev(vals), dev(pre))
            o.insert_segments(vals, pre)
        batch.shrink(num, den)
        for a, o in zip(arrays, orcs):
            o.shrink(num, den)
            assert_same(a, o, f"round {r}")
    st = pool.stats()
    assert st["in_use"] == 0 and st["allocs"] == st["frees"]
    batch.close()
    for a in arrays:
        a.close()
    pool.close()
