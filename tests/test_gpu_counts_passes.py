"""GPU parity of counts rounds over a padded buffer in two passes (more than 2048
tiles): the last tile count of the one-launch form and the next, counts above the
round's largest, sums at every alignment, tiny first buckets, more tiles per LFVector
than a wave's pass, and an allocation failure; against the CPU oracle, bit for bit."""
import numpy as np
import pytest

from paper_2209_00103_amd import workloads as wl
from tests.gpu_util import assert_same, both, dev, gg, gpu_flat, gpu_sizes

pytestmark = pytest.mark.gpu
TILE = 1024


@pytest.mark.parametrize("elem,V,F,n,mc", [
    (4, 1024, 16, 1024 * 2 * TILE, 1),            # 2048 tiles: one launch
    (4, 683, 1, 683 * (2 * TILE + 1) - 500, 3),   # 2049 tiles: two passes
    (8, 683, 1024, 683 * 2500 - 2600, 2),         # the last LFVector gets nothing
    (4, 1, 1024, 2100 * TILE + 7, 2),
    (8, 130, 64, 130 * (16 * TILE + 333), 4),
])
def test_counts_passes(elem, V, F, n, mc):
    print(f"case counts passes elem={elem} V={V} F={F} n={n} max={mc}", flush=True)
    rng = np.random.default_rng(V + mc)
    pool = gg().Pool(1 << 30)
    a, o = both(elem, V, F, pool)
    for r in range(2):
        counts = rng.integers(0, mc + 3, size=n, dtype=np.uint8)  # above the largest: clamped
        if r:
            counts[rng.random(n) < 0.8] = 0
        vals, _ = wl.random_round(rng, n * mc, 1.0, elem)
        dc = dev(np.concatenate([np.ones(r, np.uint8), counts]))[r:]
        a.insert_counts(dev(vals), dc, mc)
        o.insert_counts(vals, counts, mc)
        assert_same(a, o, f"round {r}")
    a.close()
    o.close()
    pool.close()


def test_counts_passes_failed_growth_freezes_one_lfvector():
    G = gg()
    rng = np.random.default_rng(3)
    pool = G.Pool(512 << 20)
    V, chunk = 300, 8 * TILE
    a = G.GGArray(pool, 4, V, 1024)
    vals, _ = wl.random_round(rng, V * chunk, 1.0, 4)
    pool.set_fault(500)
    a.insert_counts(dev(vals), dev(np.ones(V * chunk, np.uint8)), 1)
    assert a.last_error() == G.ENOMEM
    sizes = gpu_sizes(a)
    assert (sizes == 0).sum() == 1 and sizes.sum() == (V - 1) * chunk
    np.testing.assert_array_equal(gpu_flat(a), vals[np.repeat(sizes > 0, chunk)])
    a.close()
    pool.set_fault(0)
    assert pool.stats()["in_use"] == 0
    pool.close()


def test_smaller_counts_and_generated_rounds_in_a_graph_after_one_in_two_passes():
    """Only the eager two-pass round came before: the captured rounds' look-back words are there."""
    import torch

    import oracle

    G = gg()
    rng = np.random.default_rng(9)
    pool = G.Pool(1 << 30)
    V, mc = 300, 2
    a, o = both(4, V, 64, pool)
    big, small = V * 8 * TILE, V * 3 * TILE - 11
    vals, _ = wl.random_round(rng, big * mc, 1.0, 4)
    counts = rng.integers(0, mc + 1, size=big, dtype=np.uint8)
    dv, dc = dev(vals), dev(counts)
    a.insert_counts(dv, dc, mc)
    o.insert_counts(vals, counts, mc)
    gen = G.make_gen(G.GEN_BERNOULLI, seed=5, round=1)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        a.insert_counts(dv[:small * mc], dc[:small], mc)
        a.insert_gen(gen, big)
        a.insert_counts(dv, dc, mc)
        a.shrink(3, 4)
    for k in range(3):
        graph.replay()
        o.insert_counts(vals[:small * mc], counts[:small], mc)
        o.insert_gen(oracle.GEN_BERNOULLI, big, seed=5, round=1)
        o.insert_counts(vals, counts, mc)
        o.shrink(3, 4)
        assert_same(a, o, f"replay {k}")
    a.close()
    o.close()
    pool.close()
