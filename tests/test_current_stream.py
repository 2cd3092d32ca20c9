"""The binding asks torch for the current stream's handle by a private name; a torch without
it is asked the public way (no GPU needed: torch's answers are stand-ins)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BODY = """
import types, torch
if {private}:
    torch._C._cuda_getCurrentRawStream = lambda device: 100 + device
elif hasattr(torch._C, "_cuda_getCurrentRawStream"):
    del torch._C._cuda_getCurrentRawStream
torch.cuda.current_device = lambda: 3
torch.cuda.current_stream = lambda device=None: types.SimpleNamespace(cuda_stream=200 + device)
from paper_2209_00103_amd import ggarray
print(ggarray._stream(None), ggarray._stream(types.SimpleNamespace(cuda_stream=7)))
"""


@pytest.mark.parametrize("private,want", [(True, "103 7"), (False, "203 7")])
def test_current_stream_without_the_private_name(private, want):
    r = subprocess.run([sys.executable, "-c", BODY.format(private=private)], capture_output=True, text=True,
                       timeout=120, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split("\n")[-2] == want
