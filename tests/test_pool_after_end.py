"""The device pool's allocation compiled for the CPU (tests/host/cpu_hip stands in for
the HIP runtime header) and stepped far past the end of its region."""
import os
import shutil
import subprocess

import pytest

from tests.conftest import ROOT


@pytest.mark.skipif(not shutil.which("g++"), reason="g++ not available")
def test_allocations_after_the_region_has_run_out(tmp_path):
    exe = str(tmp_path / "pool_after_end")
    host = os.path.join(ROOT, "tests", "host")
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-Wno-attributes", "-I", os.path.join(host, "cpu_hip"),
                        "-I", os.path.join(ROOT, "include"), os.path.join(host, "pool_after_end.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
