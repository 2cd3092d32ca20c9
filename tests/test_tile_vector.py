"""Where the flagged rounds load a tile's vectors from, checked on the host."""
import os
import shutil
import subprocess

import pytest

from paper_2209_00103_amd import build as B
from tests.conftest import ROOT


@pytest.mark.skipif(not os.path.exists(B.HIPCC) and not shutil.which("hipcc"), reason="hipcc not available")
def test_vectors_of_a_tile_stay_in_it(tmp_path):
    exe = str(tmp_path / "tile_vector_check")
    r = subprocess.run([B.HIPCC, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I", B.INCLUDE, "-I", B.CSRC,
                        os.path.join(ROOT, "tests", "host", "tile_vector_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
