"""The rules that choose a stage's form, held against the measurements they were fitted to (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rules_take_the_faster_form(tmp_path):
    exe = str(tmp_path / "rules_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2511_21031_amd", "csrc"),
                    os.path.join(ROOT, "tests", "stage_rules_check.cpp"), "-o", exe], check=True, capture_output=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
