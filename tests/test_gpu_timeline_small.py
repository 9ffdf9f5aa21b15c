"""The diagnostic library on a mesh that the product library runs as one launch."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_RUN = r"""
import ctypes
import torch
from paper_2104_04347_amd import binding, inputs, timeline
lib = timeline.load()
timeline.clear(lib, "1d")
with binding.Solver("euler", 3, 300, "transmissive") as s:
    s.write(inputs.euler_riemann(0, 3, 300)[0])
    s.run(20, 0.2)
    torch.cuda.synchronize()
    rec = timeline.read(lib, "1d")
full = rec[(rec["t0"] > 0) & (rec["t1"] > rec["t0"])]
print("waves", len(full))
"""


@pytest.mark.gpu
def test_small_meshes_leave_records():
    """300 intervals are five wave tiles: two blocks of four waves stamp both ends of the last half-step."""
    r = subprocess.run([sys.executable, "-c", _RUN], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-3000:]
    assert r.stdout.split()[-2:] == ["waves", "8"], r.stdout
