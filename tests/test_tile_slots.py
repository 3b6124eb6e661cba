"""Host-side bounds check of the balanced-tile and wave-tile kernels' LDS and cell indices (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tile_and_line_kernel_indices_in_bounds(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "slots_check")
    subprocess.run(["hipcc", "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2511_21031_amd", "csrc"),
                    os.path.join(ROOT, "tests", "tile_slots_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
