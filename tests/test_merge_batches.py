"""The launches that a merge's inputs are cut into, on the CPU (no GPU): tests/merge_batches.cpp
drives the host-side template with input sizes up to billions of entries."""
import os
import subprocess

from paper_2206_05269_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_merge_batches(tmp_path):
    exe = tmp_path / "merge_batches"
    subprocess.run([build.HIPCC, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1",
                    "-I", build.CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "merge_batches.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and "all ok" in r.stdout, r.stdout + r.stderr
