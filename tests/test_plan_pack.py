"""Packed rows and wide combine tasks: the planner's properties (CPU), and the
passes against the oracle on both sides of a wide task's sizes (GPU)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from gpu_util import assert_close, from_em, to_em

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_06115_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_packed_plans(tmp_path):
    exe = str(tmp_path / "plan_pack")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC, "-I",
                           os.path.join(ROOT, "tests", "c"),
                           os.path.join(ROOT, "tests", "c", "plan_pack.cpp"),
                           os.path.join(CSRC, "plan.cpp"), "-o", exe])
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:verify_asan_link_order=0")
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "packed plans hold" in out.stdout


# Hub rows of 16-entry chunks (15 triples a partial): 33 partials (the smallest
# wide task), 256 and 257 (one and two rounds of a workgroup's 32 groups of 8
# lanes), 1024 and 1025 (two levels), and several of each, at one narrow, one
# ragged, one 8-lane and two sliced widths.
@pytest.mark.gpu
@pytest.mark.parametrize("b", [2, 10, 32, 93, 260])
@pytest.mark.parametrize("gamma", [None, 0.5])
def test_wide_combine(b, gamma, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2002_06115_amd as kbf
    monkeypatch.setenv("KBFOLLOW_CHUNK", "16")
    monkeypatch.setenv("KBFOLLOW_REL_CHUNK", "16")
    monkeypatch.setenv("KBFOLLOW_XCD", "1")  # a hub row is then one segment
    g = np.random.default_rng(b)
    n_e, n_r = 400, 3
    hubs = np.repeat(np.arange(8), [15 * 32 + 1, 15 * 33, 15 * 256, 15 * 257, 15 * 1024 - 3,
                                    15 * 1024 + 1, 15 * 1100, 700])
    o = np.concatenate([hubs, g.integers(20, n_e - 30, 900)]).astype(np.int32)
    s = g.integers(0, n_e, len(o)).astype(np.int32)
    r = g.integers(0, n_r, len(o)).astype(np.int32)
    X, dY = (g.standard_normal((b, n_e)).astype(np.float32) for _ in range(2))
    R = g.standard_normal((b, n_r)).astype(np.float32)
    kb = kbf.KB(s, r, o, n_e, n_r)
    assert kb.info()["n_levels"][0] == 2  # the row of 1025 partials or more
    Y = from_em(kb.follow(to_em(X), to_em(R), residual=gamma))
    dX, dR = kb.follow_backward(to_em(X), to_em(R), to_em(dY), residual=gamma)
    kb.close()
    if gamma is None:
        want = oracle.follow(s, r, o, n_e, n_r, X, R)
        want_dx, want_dr = oracle.follow_backward(s, r, o, n_e, n_r, X, R, dY)
    else:
        want = oracle.follow_residual(s, r, o, n_e, n_r, X, R, gamma)
        want_dx, want_dr = oracle.follow_backward_residual(s, r, o, n_e, n_r, X, R, dY, gamma)
    assert_close(Y, want, "Y")
    assert_close(from_em(dX), want_dx, "dX")
    assert_close(from_em(dR), want_dr, "dR")
