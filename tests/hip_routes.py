"""The library on the CPU with its launches recorded (tests/host/hip_record.c in place
of the HIP runtime).  ``run(body)`` executes `body` in a child process, where `R` is
this module after ``load``; it returns what the body assigned to `out`.  Nothing is
computed: sizes stay zero on the "device", the host's own bookkeeping is real.
"""
import ctypes
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2209_00103_amd", "libggarray.so")
lib = rec = None


class Gen(ctypes.Structure):
    _fields_ = [("kind", ctypes.c_uint32), ("round", ctypes.c_uint32), ("seed", ctypes.c_uint64),
                ("tag_shift", ctypes.c_uint32), ("max_count", ctypes.c_uint32),
                ("thresholds", ctypes.c_uint64 * 16), ("tag", ctypes.c_uint64)]


def load(record):
    global lib, rec
    rec = ctypes.CDLL(record, mode=ctypes.RTLD_GLOBAL)
    rec.rec_name.restype = ctypes.c_char_p
    rec.rec_grid.restype = rec.rec_block.restype = ctypes.c_uint32
    rec.rec_capture.argtypes = [ctypes.c_uint64]
    lib = ctypes.CDLL(LIB)


def u64(x):
    return ctypes.c_uint64(x)


def ptr(x):
    return ctypes.c_void_p(x)


def check(rc, want=0):
    assert rc == want, f"status {rc}, not {want}"


def memory(n):
    p = ctypes.c_void_p()
    check(rec.hipMalloc(ctypes.byref(p), ctypes.c_size_t(n)))
    return p


def pool():
    p = ctypes.c_void_p()
    check(lib.gga_pool_create(ctypes.byref(p), memory(4 << 20), u64(4 << 20), None))
    return p


def array(p, elem, V, F=64):
    a = ctypes.c_void_p()
    check(lib.ggarray_create(ctypes.byref(a), p, elem, V, u64(F), None))
    rec.rec_clear()
    return a


def launches():
    """(kernel, grid, block) of the launches since the last look; names without their template's mangling."""
    out = []
    for i in range(rec.rec_count()):
        name = rec.rec_name(i).decode()
        out.append((name, rec.rec_grid(i), rec.rec_block(i)))
    rec.rec_clear()
    names = subprocess.run(["c++filt"], input="\n".join(n for n, _, _ in out), capture_output=True, text=True).stdout
    short = [n.replace("gga::(anonymous namespace)::", "").replace("gga::", "").split("(")[0].split(" ", 1)[-1]
             if n.startswith("void ") else n.replace("gga::(anonymous namespace)::", "").replace("gga::", "").split("(")[0]
             for n in names.split("\n")]
    return [(s.split("<")[0], g, b) for s, (_, g, b) in zip(short, out)]


SOMEWHERE = 0x10000  # an address for inputs that nothing reads here


def insert(a, n, flags=False):
    check(lib.ggarray_insert(a, ptr(SOMEWHERE), ptr(SOMEWHERE) if flags else None, u64(n), None))


def segments(a, n):
    check(lib.ggarray_insert_segments(a, ptr(SOMEWHERE), ptr(SOMEWHERE), u64(n), None))


def counts(a, n, most=4, want=0):
    check(lib.ggarray_insert_counts(a, ptr(SOMEWHERE), ptr(SOMEWHERE), most, u64(n), None), want)


def packed(a, n, n_values):
    check(lib.ggarray_insert_packed(a, ptr(SOMEWHERE), u64(n_values), ptr(SOMEWHERE), u64(n), None))


def poisson(a, n, each):
    """A round whose draws all pass `each` of sixteen thresholds, so that each thread inserts that many."""
    g = Gen(kind=3, round=1, seed=3, max_count=16)
    for k in range(16):
        g.thresholds[k] = 0 if k < each else (1 << 64) - 1
    check(lib.ggarray_insert_gen(a, ctypes.byref(g), u64(n), None))


class Desc(ctypes.Structure):  # gga::InsertDesc
    _fields_ = [("mode", ctypes.c_uint32), ("values", ctypes.c_void_p), ("flags", ctypes.c_void_p),
                ("max_count", ctypes.c_uint32), ("n_threads", ctypes.c_uint64), ("seed", ctypes.c_uint64),
                ("round", ctypes.c_uint32), ("tag_shift", ctypes.c_uint32), ("thresholds", ctypes.c_uint64 * 16),
                ("tag", ctypes.c_uint64)]


def insert_shrink(a, n, mode, num, den):
    """launch_insert with a shrink after the round, which the C entry points ask for with generated payloads only."""
    f = lib._ZN3gga13launch_insertEP7ggarrayRKNS_10InsertDescEP12ihipStream_tjj
    check(f(a, ctypes.byref(Desc(mode=mode, values=SOMEWHERE, n_threads=n, round=1)), None, num, den))


def run(body, record):
    prog = (f"import sys, json; sys.path.insert(0, {ROOT!r})\n"
            f"from tests import hip_routes as R\nR.load({record!r})\n{body}\nprint(json.dumps(out))")
    r = subprocess.run([sys.executable, "-c", prog], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    return json.loads(r.stdout.strip().split("\n")[-1])


def build_record(where):
    so = os.path.join(str(where), "libhiprecord.so")
    r = subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "host", "hip_record.c"),
                        "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return so
