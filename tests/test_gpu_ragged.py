"""Widths that are not a multiple of 4: rows read 4 floats per lane, their last
lane taking the row's last 4 columns, against the oracle and, bit for bit,
against one float per lane (the sums and their order are the same), with the
rows no triple reaches written one by one or by a sweep over the output."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, from_em, to_em

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kbf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2002_06115_amd as kbf
    return kbf


def outputs(kbf, kb_args, n_e, n_r, X, R, dY, Z, weight):
    kb = kbf.KB(*kb_args, n_e, n_r, weight=weight)
    Y = kb.follow(X, R)
    Yr = kb.follow(X, R, residual=0.5)
    Za = Z.clone()
    kb.follow_accumulate(X, R, Za, 2.0, out=Za)  # in place: each row read, then written
    dX, dR = kb.follow_backward(X, R, dY)
    dXr, dRr = kb.follow_backward(X, R, dY, residual=0.5)
    out = [from_em(t) for t in (Y, Yr, Za, dX, dR, dXr, dRr)]
    kb.close()
    return out


# The narrowest and widest last lanes, one group of each size, slices of 128
# columns whose last lane reaches back into the slice before (129 .. 131), and
# the 32-column slices of dR from 128 columns on.
@pytest.mark.parametrize("b", [5, 6, 7, 9, 10, 15, 17, 31, 33, 63, 66, 127, 129, 130, 131, 257])
@pytest.mark.parametrize("weighted,path", [(False, "lds"), (False, "regs"), (False, "plain"),
                                           (False, "prefill"), (True, "lds"), (True, "plain")])
def test_ragged_widths(kbf, b, weighted, path, monkeypatch):
    monkeypatch.setenv("KBFOLLOW_REL_CHUNK", "16")
    monkeypatch.setenv("KBFOLLOW_FAN_IN", "3")
    if path == "plain":
        monkeypatch.setenv("KBFOLLOW_PLAIN_LOADS", "1")
    monkeypatch.setenv("KBFOLLOW_PREFILL", "1" if path == "prefill" else "0")
    if path == "regs":
        monkeypatch.setenv("KBFOLLOW_B_IN_LDS", "0")
    g = np.random.default_rng(b)
    n_e, n_r, n_t = 300, 7, 5000
    s = np.where(g.random(n_t) < 0.3, g.integers(0, 3, n_t), g.integers(0, n_e, n_t))
    o = np.where(g.random(n_t) < 0.3, g.integers(0, 3, n_t), g.integers(0, n_e - 40, n_t))
    r = g.integers(0, n_r, n_t)
    kb_args = [a.astype(np.int32) for a in (s, r, o)]
    w = g.uniform(0.1, 2.0, n_t).astype(np.float32) if weighted else None
    draw = lambda n: g.standard_normal((b, n)).astype(np.float32)  # noqa: E731
    X, R, dY, Z = draw(n_e), draw(n_r), draw(n_e), draw(n_e)
    dev = [to_em(a) for a in (X, R, dY, Z)]
    got = outputs(kbf, kb_args, n_e, n_r, *dev, w)
    Yo = oracle.follow(*kb_args, n_e, n_r, X, R, weight=w)
    dXo, dRo = oracle.follow_backward(*kb_args, n_e, n_r, X, R, dY, weight=w)
    assert_close(got[0], Yo, "Y")
    assert_close(got[3], dXo, "dX")
    assert_close(got[4], dRo, "dR")
    monkeypatch.setenv("KBFOLLOW_PREFILL", "0")
    monkeypatch.setenv("KBFOLLOW_SCALAR_LANES", "1")
    want = outputs(kbf, kb_args, n_e, n_r, *dev, w)
    for name, a, c in zip(("Y", "Y residual", "Z", "dX", "dR", "dX residual", "dR residual"),
                          got, want):
        assert np.array_equal(a, c), (name, b, weighted, path)
