"""The chunk lists of a plan, one per XCD, hold about equal numbers of chunks
whatever part of the id space a KB uses (CPU): a subset of a large KB loaded
with its original ids keeps every XCD busy."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_06115_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_lists_are_balanced(tmp_path):
    exe = str(tmp_path / "plan_balance")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-pthread", "-I", CSRC, "-I",
                           os.path.join(ROOT, "tests", "c"),
                           os.path.join(ROOT, "tests", "c", "plan_balance.cpp"),
                           os.path.join(CSRC, "plan.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "lists balanced" in out.stdout
