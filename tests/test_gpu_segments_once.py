"""GPU parity of segment appends whose payloads are larger than the cache, from buffers at
every alignment of their type, with the last size of the other form; against torch."""
import pytest

from tests.gpu_util import gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elem,V,more,skip", [(4, 7, 0, 0), (4, 7, 1, 1), (4, 600, 12345, 3), (8, 600, 1, 1), (8, 3, 5, 0)])
def test_segments_larger_than_the_cache(elem, V, more, skip):
    import torch

    print(f"case segments once elem={elem} V={V} more={more} skip={skip}", flush=True)
    n = (256 << 20) // elem + more
    t = torch.int32 if elem == 4 else torch.int64
    buf = torch.arange(n + skip, device="cuda", dtype=t) * 7919 + 13
    vals = buf[skip:]
    g = torch.Generator(device="cuda").manual_seed(V)
    cuts = torch.randint(0, n, (V - 1,), device="cuda", generator=g).sort().values
    prefix = torch.cat([cuts.new_zeros(1), cuts, cuts.new_full((1,), n)])
    pool = gg().Pool(2 << 30)
    a = gg().GGArray(pool, elem, V, 1024)
    head = torch.arange(V, device="cuda", dtype=t)  # the segments start at odd places of their LFVectors
    a.insert_segments(head, torch.arange(V + 1, device="cuda", dtype=torch.int64))
    a.insert_segments(vals, prefix)
    out = a.flatten()
    assert a.last_error() == 0 and out.numel() == n + V
    at = prefix[:-1] + torch.arange(V, device="cuda")
    assert torch.equal(out[at], head)
    rest = torch.ones(n + V, dtype=torch.bool, device="cuda")
    rest[at] = False
    assert torch.equal(out[rest], vals)
    a.close()
    pool.close()
