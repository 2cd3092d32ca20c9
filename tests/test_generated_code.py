"""What the compiler makes of the insertion kernels, where their speed hangs on it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2209_00103_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC) and not shutil.which("hipcc"),
                                reason="hipcc not available")


@pytest.fixture(scope="module")
def insert_asm(tmp_path_factory):
    asm = str(tmp_path_factory.mktemp("asm") / "insert.s")
    r = subprocess.run([B.HIPCC, *B.CFLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, "insert.hip"), "-o", asm],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(asm) as f:
        return f.read()


def _kernels(asm, name):
    """(symbol, code) of the kernels whose mangled name holds `name` (a pattern)."""
    found = re.findall(r"^(_ZN\S*\d+%s\S*):\s*;.*?\n(.*?)\n\.Lfunc_end" % name, asm, re.S | re.M)
    assert found, name
    return found


@pytest.mark.parametrize("kernel", [
    "segments_kernel", "segments_block_kernel", "segments_store_kernel", "grow_store_block_kernel",
    r"grow_store_kernelI\wNS_10ProdBuffer", r"dense_insert_kernelI\wNS_10ProdBuffer",
    r"static_dense_kernelI\wNS_10ProdBuffer",
])
def test_buffer_copies_load_vectors(insert_asm, kernel):
    """A run of a buffer's elements is copied through four 16-byte loads a lane, not a load per element."""
    for name, code in _kernels(insert_asm, kernel):
        n = len(re.findall(r"\bglobal_load_dwordx4\b", code))
        assert n >= 4, f"{name}: {n} 16-byte loads"


@pytest.mark.parametrize("kernel", ["grow_store_kernel", "segments_kernel"])
def test_eight_waves_of_a_kernel_fit_a_simd(insert_asm, kernel):
    """Short rounds of many LFVectors wait for memory with every wave a CU can hold: 80 scalar and 64 vector
    registers are the most that eight waves of a SIMD may have."""
    for name, _ in _kernels(insert_asm, kernel):
        info = insert_asm[insert_asm.index(f".amdhsa_kernel {name}\n"):]
        if int(re.search(r"; NumVgprs: (\d+)", info).group(1)) <= 64:
            assert int(re.search(r"; TotalNumSgprs: (\d+)", info).group(1)) <= 80, name
        assert int(re.search(r"; NumVgprs: (\d+)", info).group(1)) <= 64, name


def test_small_generated_counts_rounds_fetch_one_form_of_the_hash(insert_asm):
    """A small round fetches each instruction anew: the workgroup kernel of drawn counts holds one form of its hashes
    (86 quarter-rate products for 4-byte elements, 74 for 8-byte ones; both forms make 114 and 98)."""
    seen = 0
    for name, code in _kernels(insert_asm, r"insert_count_kernelI\wNS_11ProdPoissonI\wEELb0ELb0"):
        assert len(re.findall(r"\bv_(?:mul_hi_u32|mul_lo_u32|mad_u64_u32)\b", code)) <= 90, name
        seen += 1
    assert seen == 2


@pytest.mark.parametrize("kernel", ["insert_block_kernel", "insert_count_wave_kernelI[jm]NS_1[01]Prod(?:CountsIm|Poisson)"])
def test_scalar_registers_of_the_allocating_rounds_leave_eight_waves(insert_asm, kernel):
    """More than 80 scalar registers cost a wave of every SIMD (1000 LFVectors of 4000 flagged threads: 15 -> 20 us)."""
    for name, _ in _kernels(insert_asm, kernel):
        info = insert_asm[insert_asm.index(f".amdhsa_kernel {name}\n"):]
        if int(re.search(r"; NumVgprs: (\d+)", info).group(1)) <= 64:
            assert int(re.search(r"; TotalNumSgprs: (\d+)", info).group(1)) <= 80, name
