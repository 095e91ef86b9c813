"""Chunk lengths of the entity layouts (CPU): shorter than the default only where a
chunk holds several rows and packing splits few of them; a forward pass then never
needs more scratch than default chunks without packing, which bounds what
kb_follow_noalloc's fixed scratch has to hold."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_06115_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_chunk_lengths(tmp_path):
    exe = str(tmp_path / "plan_chunk")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-pthread", "-I", CSRC, "-I",
                           os.path.join(ROOT, "tests", "c"),
                           os.path.join(ROOT, "tests", "c", "plan_chunk.cpp"),
                           os.path.join(CSRC, "plan.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "chunk lengths hold" in out.stdout
