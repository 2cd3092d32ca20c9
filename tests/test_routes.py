"""Which kernels a call launches, by size and state: the library's host side on the CPU
with its launches recorded."""
import os
import shutil

import pytest

from tests import hip_routes

pytestmark = pytest.mark.skipif(not shutil.which("gcc") or not shutil.which("c++filt")
                                or not os.path.exists(hip_routes.LIB), reason="needs gcc and the built library")


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    return hip_routes.build_record(tmp_path_factory.mktemp("record"))


def test_dense_buffer_rounds_by_share_and_count(record):
    """A wave per LFVector while the share is short or the waves alone fill the chip, else a workgroup of as many
    waves as leave every workgroup room on the chip at once."""
    out = hip_routes.run("""
p, out = R.pool(), []
for V, kb in ((1, 4), (1, 5), (512, 5), (513, 5), (1024, 5), (1024, 128), (1024, 129), (1025, 5), (2048, 5),
              (2049, 5), (2049, 12), (2049, 13), (65536, 12), (65536, 13)):
    for elem in (4, 8):
        a = R.array(p, elem, V)
        R.insert(a, V * (kb * 1024 // elem))
        out += R.launches()
""", record)
    want = {(1, 4): 1, (1, 5): 16, (512, 5): 16, (513, 5): 8, (1024, 5): 8, (1024, 128): 8, (1024, 129): 16,
            (1025, 5): 4, (2048, 5): 4, (2049, 5): 1, (2049, 12): 1, (2049, 13): 4, (65536, 12): 1, (65536, 13): 4}
    exp = []
    for (V, _), w in want.items():
        exp += 2 * [["grow_store_kernel", (V + 3) // 4, 256] if w == 1 else ["grow_store_block_kernel", V, 64 * w]]
    assert out == exp


def test_segments_by_average_and_count(record):
    out = hip_routes.run("""
p, out = R.pool(), []
for V, kb in ((1, 4), (1, 8), (512, 8), (512, 32), (512, 36), (1024, 8), (1024, 32), (2048, 16), (2048, 20), (2048, 36),
              (2049, 8), (2049, 12), (2049, 16), (2049, 20), (16385, 20), (16385, 36)):
    for elem in (4, 8):
        a = R.array(p, elem, V)
        R.segments(a, V * (kb * 1024 // elem))
        out.append(R.launches())
""", record)
    # waves per LFVector (0: a wave without a workgroup of its own), or the store launch's workgroups per LFVector
    want = [(1, 0), (1, 16), (512, 16), (512, 16), (512, "5"), (1024, 8), (1024, 8), (2048, 4), (2048, 8), (2048, "5"),
            (2049, 0), (2049, 4), (2049, 4), (2049, 8), (16385, 4), (16385, "2")]
    exp = []
    for V, w in want:
        if w == 0:
            form = [["segments_kernel", (V + 3) // 4, 256]]
        elif isinstance(w, str):
            form = [["segments_grow_kernel", (V + 3) // 4, 256], ["segments_store_kernel", V * int(w), 256]]
        else:
            form = [["segments_block_kernel", V, 64 * w]]
        exp += [form, form]
    assert out == exp


SETUP = """
p, out = R.pool(), []
a, offsets = R.array(p, 4, 512), R.memory(8 * 513)
def prefix():
    R.check(R.lib.ggarray_prefix(a, offsets, None))
def rw():
    R.check(R.lib.ggarray_rw(a, 0, None))
def insert():  # the same size again, so that a table once built is large enough
    R.check(R.lib.ggarray_shrink(a, 1, 1, None))
    R.insert(a, 1 << 24)
    R.launches()
def seen():
    out.append([k for k, _, _ in R.launches()])
"""
APART = ["scan_kernel", "tile_table_kernel", "stream_table_kernel"]


def test_the_offsets_alone_build_no_tile_table(record):
    """ggarray_prefix writes the tile table in its launch only where the last sizes it was asked for were streamed."""
    out = hip_routes.run(SETUP + """
insert(); prefix(); seen(); insert(); prefix(); seen()          # offsets alone
insert(); prefix(); rw(); seen(); insert(); prefix(); rw(); seen()  # offsets, then an r/w
insert(); prefix(); seen(); insert(); prefix(); seen()          # alone again: one table too many, then none
insert(); rw(); prefix(); seen()
""", record)
    assert out == [["scan_kernel"], ["scan_kernel"], APART, ["scan_table_kernel", "stream_table_kernel"],
                   ["scan_table_kernel"], ["scan_kernel"], ["scan_table_kernel", "stream_table_kernel"]]


def test_sizes_changed_by_graphs_scan_and_build_apart(record):
    """Once a graph changes the sizes, no eager call may rely on a table built before it: one build a call, not two."""
    out = hip_routes.run(SETUP + """
insert(); rw(); seen()
R.rec.rec_capture(7); R.insert(a, 512); rw(); seen(); R.rec.rec_capture(0)
rw(); seen(); rw(); seen(); prefix(); seen()
""", record)
    assert out == [["scan_table_kernel", "stream_table_kernel"],
                   ["grow_store_kernel", "scan_table_kernel", "stream_table_kernel"], APART, APART, ["scan_kernel"]]


def test_packed_rounds_of_one_tile_by_count_and_length(record):
    """A workgroup per LFVector for few of them or long tiles; a wave each, four to a workgroup that copies a tile of
    up to 255 values a thread together; waves of their own where the other LFVectors outlast such a tile."""
    out = hip_routes.run("""
p, out = R.pool(), []
for V, elem, chunk, kb in ((2047, 4, 100, 1), (2048, 4, 100, 1), (2048, 4, 1024, 8), (2048, 4, 1024, 9), (2048, 4, 64, 1),
                           (2048, 4, 65, 1), (2048, 8, 33, 1), (65536, 8, 1024, 8), (16384, 8, 257, 2)):
    a = R.array(p, elem, V)
    R.packed(a, V * chunk, V * kb * 1024 // elem)
    out.append(R.launches()[-1])
""", record)
    one, four, own = "packed_grow_copy_kernel", "packed_grow_copy_waves_kernel", "packed_grow_copy_kernel"
    assert out == [[one, 2047, 256], [four, 512, 256], [four, 512, 256], [one, 2048, 256], [own, 2048, 64],
                   [four, 512, 256], [four, 512, 256], [own, 65536, 64], [four, 4096, 256]]


def test_counts_rounds_of_one_tile_by_what_a_share_may_hold(record):
    """A wave per LFVector where no share can hold the launch, else a workgroup."""
    out = hip_routes.run("""
p, out = R.pool(), []
for V, chunk, most in ((2047, 64, 4), (2048, 256, 4), (2048, 257, 4), (2048, 64, 16), (2048, 65, 16), (8192, 256, 16),
                       (8192, 512, 8), (8192, 512, 9), (16384, 512, 16), (32768, 512, 16), (65536, 513, 2)):
    a = R.array(p, 4, V)
    R.counts(a, V * chunk, most)
    out.append(R.launches()[-1][2])
for V, chunk, each in ((2048, 256, 16), (2048, 512, 5), (2048, 512, 6), (8192, 512, 8), (8192, 512, 9), (65536, 512, 16)):
    a = R.array(p, 8, V)
    R.poisson(a, V * chunk, each)
    out.append(R.launches()[-1][2])
""", record)
    assert out == [256, 64, 256, 64, 256, 64, 64, 256, 256, 64, 256] + [64, 64, 256, 64, 256, 64]


def test_long_growth_passes_by_tiles(record):
    """Tile words of one LFVector: a wave to 256 tiles, then a workgroup in passes of 4096, past 4096 of 16384."""
    out = hip_routes.run("""
p, out = R.pool(), []
for tiles in (256, 257, 4096, 4097, 65536):
    a = R.array(p, 4, 1)
    R.insert(a, tiles * 4096, flags=True)
    out.append([R.rec.rec_name(i).decode() for i in range(R.rec.rec_count())][1])
""", record)
    assert ["flag_grow_kernel" in n for n in out] == [True, False, False, False, False]
    assert ["flag_grow_long_kernelILj%dE" % k in n for n, k in zip(out[1:], (4, 4, 16, 16))] == [True] * 4


def test_a_shrink_after_a_dense_round_is_queued_or_in_its_launch(record):
    """Only the one-wave-per-LFVector round of generated payloads shrinks by itself: from a buffer, of every form,
    the shrink is a launch of its own."""
    out = hip_routes.run("""
p, out = R.pool(), []
for mode in (0, 3):  # from a buffer, round tags
    for V, chunk in ((512, 100), (512, 5000), (2048, 5000), (16384, 2000), (16, 1 << 20)):
        a = R.array(p, 4, V)
        R.insert_shrink(a, V * chunk, mode, 1, 2)
        out.append([k for k, _, _ in R.launches()])
""", record)
    for names in out[:5]:
        assert [n.startswith("shrink") for n in names] == [False] * (len(names) - 1) + [True]
    assert out[5:9] == [["grow_store_kernel"]] * 4 and out[9][-1].startswith("shrink")


def test_rounds_in_two_passes_fall_back_when_memory_is_short(record):
    """Without room for the tiles' words a counts round takes the one-launch form, as it does in a capture; the words
    of an earlier round stay, and the next round with room takes two passes again."""
    out = hip_routes.run("""
p, out = R.pool(), []
def seen():
    out.append([k for k, _, _ in R.launches()])
n = 1024 * 2049  # tiles of one LFVector
a = R.array(p, 4, 1)
R.rec.rec_fail(2); R.counts(a, n); seen()  # the look-back words fit, the two passes' do not
R.counts(a, n); seen()
R.rec.rec_fail(2); R.counts(a, 4 * n); seen()
R.rec.rec_fail(0)
R.rec.rec_capture(5); R.counts(a, n); seen(); R.rec.rec_capture(0)
R.counts(a, 4 * n); seen()
b = R.array(p, 4, 1)
R.rec.rec_fail(1); R.counts(b, n, want=-4); R.rec.rec_fail(0)
""", record)
    one, two = ["insert_count_kernel"], ["counts_sum_kernel", "flag_grow_long_kernel", "counts_copy_kernel"]
    assert out == [one, two, one, two, two]


def test_server_creation_stages_its_items_without_throwing(record):
    """Of what grows with the arrays, only the list of handles comes from an operator new that throws."""
    out = hip_routes.run("""
import ctypes
from paper_2209_00103_amd.ggarray import ServerConfig
p, n = R.pool(), 512
arrays = (ctypes.c_void_p * n)(*[R.array(p, 4, 1).value for _ in range(n)])
cfg = ServerConfig(mode=1, seed=1, append_shift=20, rw_op=0, append_round=1, lanes=1, max_step=4, depth=4)
sv = ctypes.c_void_p()
R.rec.rec_new_largest.restype = ctypes.c_size_t
R.rec.rec_new_largest()
R.check(R.lib.gga_server_create(ctypes.byref(sv), arrays, n, None, R.u64(0), ctypes.byref(cfg)))
out = R.rec.rec_new_largest()
""", record)
    assert 0 < out <= 8 * 512


def test_long_segments_workgroups_are_odd(record):
    """An odd number of workgroups a segment, so that no XCD gets the idle ones of each; the most there may be where
    equal segments give each several rounds."""
    out = hip_routes.run("""
p, out = R.pool(), []
for V, kb in ((1024, 64), (512, 128), (512, 234), (2048, 128), (2048, 248), (2048, 256), (4096, 100), (1, 1 << 18)):
    a = R.array(p, 4, V)
    R.segments(a, V * kb * 256)
    out.append(R.launches()[-1][1] // V)
""", record)
    assert out == [9, 17, 31, 17, 17, 16, 9, 32769]


def test_segments_larger_than_the_cache_are_loaded_past_it(record):
    out = hip_routes.run("""
p, out = R.pool(), []
for elem in (4, 8):
    for n in ((256 << 20) // elem, (256 << 20) // elem + 1):
        a = R.array(p, elem, 512)
        R.segments(a, n)
        out.append(R.rec.rec_name(R.rec.rec_count() - 1).decode())
""", record)
    assert ["segments_store_kernelI" in n and "Lb1E" in n for n in out] == [False, True, False, True]


def test_batch_shrinks_by_whether_the_arrays_lists_line_up(record):
    """Chains from 32768 LFVectors on where the LFVectors of a residue share their free lists, else 16 lanes each."""
    out = hip_routes.run("""
import ctypes
p, q, out = R.pool(), R.pool(), []
def batch(shapes, gap=0, pools=(p, p)):
    arrays = []
    for k, (V, F) in enumerate(shapes):
        arrays.append(R.array(pools[k % 2], 4, V, F))
        if gap: R.array(p, 4, gap, 64)
    h, b = (ctypes.c_void_p * len(arrays))(*[a.value for a in arrays]), ctypes.c_void_p()
    R.check(R.lib.gga_batch_create(ctypes.byref(b), h, len(arrays), None))
    R.launches()
    R.check(R.lib.gga_batch_shrink(b, 1, 1, None))
    out.append(R.launches()[-1][0])
batch([(20000, 64)] * 4)
batch([(131, 64)] * 512)
batch([(30000, 64), (2767, 64)])
batch([(5001, 64)] * 16, gap=77)
batch([(20000, 64), (20000, 128)])
batch([(20000, 64)] * 2, pools=(p, q))
batch([(70000, 64), (20000, 64)], gap=77)   # most of it is one array
batch([(33000, 64), (70000, 128)], gap=4096)
""", record)
    chain, apart = "batch_shrink_chain_kernel", "batch_shrink_kernel"
    assert out == [chain, chain, apart, apart, apart, apart, chain, apart]
