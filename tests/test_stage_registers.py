"""Wavefronts a SIMD that the 3D stage kernels of the mixed form get room for (compiled here, no GPU).

They sit at the edge of a step in the register file: a few registers more cost the general power's kernel a third of
its wavefronts (a step of 112^3 cells took 3068 us in place of 2466) and the kernels of 512 threads a CU's second workgroup.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

KERNELS = [   # template arguments of k_stage, wavefronts a SIMD
    ("3, 8, 8, 4, 256, float, false, CT_POLY", 3),      # the general power's only 3D shape
    ("3, 8, 4, 4, 128, float, true, CT_FIFTHS", 3),
    ("3, 8, 8, 7, 512, float, true, CT_FIFTHS", 4),
    ("3, 8, 8, 7, 512, float, false, CT_FIFTHS", 4),
]


def test_mixed_3d_stage_kernels_keep_their_wavefronts(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2511_21031_amd import build
    src = tmp_path / "kernels.hip"
    src.write_text('#include <hip/hip_runtime.h>\n#include "stage_kernel.hpp"\nusing namespace bub;\n' + "".join(
        f"template __global__ void bub::k_stage<{k}>(StageArgs, Grid, Phys, Bins);\n" for k, _ in KERNELS))
    cmd = ["hipcc"] + build.FLAGS + ["-Rpass-analysis=kernel-resource-usage", "--offload-device-only",
                                     "-I", os.path.join(ROOT, "include"), "-I", os.path.join(build.HERE, "csrc"),
                                     "-c", str(src), "-o", str(tmp_path / "kernels.o")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    got, name = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = subprocess.run(["c++filt", m.group(1)], capture_output=True, text=True).stdout
        m = re.search(r"(Occupancy \[waves/SIMD\]|VGPRs Spill): (\d+)", line)
        if m and "k_stage<" in name:
            args = re.search(r"k_stage<([^>]*)>", name).group(1)
            got.setdefault(args, {})[m.group(1).split(" ")[0]] = int(m.group(2))
    for k, waves in KERNELS:
        args = k.replace("CT_POLY", "0").replace("CT_FIFTHS", "1")
        assert got[args]["Occupancy"] >= waves, (k, got[args])
        assert got[args]["VGPRs"] == 0, (k, got[args])
