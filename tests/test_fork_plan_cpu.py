"""Which streams the launches of a mixed batch go to (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_streams_of_a_mixed_batch(tmp_path):
    exe = tmp_path / "fork_plan_check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1609_08114_amd", "csrc"),
                           os.path.join(ROOT, "tests", "fork_plan_check.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stdout[-2000:]
