"""The package does not need torch's private call for a stream's handle: without
it it imports, and takes the handle from the Stream object."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import torch
if hasattr(torch._C, "_cuda_getCurrentRawStream"):
    del torch._C._cuda_getCurrentRawStream
import paper_2112_15079_amd as nb
from paper_2112_15079_amd import _capi as C
"""
GPU = """
side = torch.cuda.Stream()
with torch.cuda.stream(side):
    for device in ("cuda:0", "cuda", torch.device("cuda"), None):
        assert C.stream_handle(device) == side.cuda_stream != 0
    pos = torch.rand(3, 200, dtype=torch.float64, device="cuda:0")
    a = nb.accel(pos, pos[0].contiguous(), 1.0)
side.synchronize()
assert bool(torch.isfinite(a).all())
"""


def run(code):
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_imports():
    run(CODE)


@pytest.mark.gpu
def test_calls():
    run(CODE + GPU)
