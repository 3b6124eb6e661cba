"""Build libbubbly.so for gfx950 with hipcc (in-tree, next to this file).

    python -m paper_2511_21031_amd.build        # or build() from Python
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SO = os.path.join(HERE, "libbubbly.so")
ARCH = "gfx950"

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed FP32 instructions are kept out of every kernel on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building libbubbly.so")


def build(verbose: bool = False, extra=None) -> str:
    """Compile every source (at the same time, each to its own object) and link them."""
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc")]
    srcs = sources()
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in srcs]
        cmds = [["hipcc"] + FLAGS + (extra or []) + inc + ["-c", s, "-o", o] for s, o in zip(srcs, objs)]
        with concurrent.futures.ThreadPoolExecutor(len(srcs)) as ex:
            list(ex.map(lambda c: _run(c, verbose), cmds))
        _run(["hipcc", "-shared", f"--offload-arch={ARCH}"] + objs + ["-o", SO + ".tmp"], verbose)
    os.replace(SO + ".tmp", SO)
    return SO


if __name__ == "__main__":
    print(build(verbose=True))
