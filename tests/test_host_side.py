"""Host side of the library over a stand-in HIP runtime (no GPU): memory that contexts and batches account for, the
routes that calls take, what is reported of them."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not available")
    from paper_2511_21031_amd import library_path
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc)))
    lib = library_path()
    exe = str(tmp_path_factory.mktemp("host") / "host_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host_check.cpp"), lib, "-o", exe,
                    "-Wl,--allow-shlib-undefined", "-Wl,-rpath," + os.path.dirname(lib)], check=True)
    return exe


@pytest.mark.parametrize("name", ["budget", "scratch", "unused", "cache", "classes", "shapes", "contents", "threads"])
def test_host_side(host_check, name, tmp_path):
    res = subprocess.run([host_check, name], capture_output=True, text=True, cwd=tmp_path)
    assert res.returncode == 0, res.stdout + res.stderr
