"""Setup forms the dense map of the small P1 levels in the idle Krylov basis: the layout stays
within it for any hierarchy and basis size, and the passes are few (tests/host/check_collapse.cpp
against the library's host sources, under the host sanitizers)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_09389_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_collapse_layout_and_passes(tmp_path):
    exe = str(tmp_path / "check_collapse")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-D_GLIBCXX_ASSERTIONS", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "host", "check_collapse.cpp"), os.path.join(CSRC, "hdg_host.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.rstrip().endswith("ALL OK"), run.stdout + run.stderr[-2000:]
