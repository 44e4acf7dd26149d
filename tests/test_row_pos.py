"""Column positions at the end of the accepted range (2^31 - 1 arcs): the walks
of the kernels' waves read every column of a row once and none outside it. No
graph of that size is built; the walks run on the host (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_walks_at_the_last_column(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "row_pos_check")
    r = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Wextra", "-fsanitize=undefined,address",
                        "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2606_05081_amd", "csrc"),
                        os.path.join(ROOT, "tests", "sanitize", "row_pos_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stdout[-4000:] + r.stderr[-4000:]
