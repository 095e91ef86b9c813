"""Widths that are not a multiple of 4: rows read 4 floats per lane, their last
lane taking the row's last 4 columns, against the oracle and, bit for bit,
against the same columns of a call padded to the next multiple of 4 (a column's
sums and their order are the same), with the rows no triple reaches written one
by one or by a sweep over the output."""
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
    monkeypatch.setenv("KBFOLLOW_B_IN_LDS", "2" if path in ("lds", "prefill") else "0")
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
    kb = kbf.KB(*kb_args, n_e, n_r, weight=w)
    for residual in (False, True):
        name = kb.phase_kernels(b, residual=residual)["fwd_stream"]
        assert name.startswith("stream_kernel<-4, "), name
        assert name.endswith("true>" if path in ("lds", "prefill") else "false>"), name
    kb.close()
    got = outputs(kbf, kb_args, n_e, n_r, *dev, w)
    Yo = oracle.follow(*kb_args, n_e, n_r, X, R, weight=w)
    dXo, dRo = oracle.follow_backward(*kb_args, n_e, n_r, X, R, dY, weight=w)
    assert_close(got[0], Yo, "Y")
    assert_close(got[3], dXo, "dX")
    assert_close(got[4], dRo, "dR")
    for name in ("PREFILL", "PLAIN_LOADS", "B_IN_LDS"):
        monkeypatch.setenv("KBFOLLOW_" + name, "0")
    pad = lambda a: np.concatenate([a, np.ones((-b % 4, a.shape[1]), np.float32)])  # noqa: E731
    want = outputs(kbf, kb_args, n_e, n_r, *(to_em(pad(a)) for a in (X, R, dY, Z)), w)
    for name, a, c in zip(("Y", "Y residual", "Z", "dX", "dR", "dX residual", "dR residual"),
                          got, want):
        assert np.array_equal(a, c[:b]), (name, b, weighted, path)


# Every cap on the lanes of a group, one lane included, at the narrowest row, a
# last lane of each kind, several slices, on both load paths.
@pytest.mark.parametrize("b", [5, 6, 7, 10, 33])
@pytest.mark.parametrize("max_lpt", ["1", "2", "4"])
@pytest.mark.parametrize("weighted,plain", [(False, "0"), (False, "1"), (True, "0"), (True, "1")])
def test_narrower_lane_groups(kbf, b, max_lpt, weighted, plain, monkeypatch):
    monkeypatch.setenv("KBFOLLOW_CHUNK", "16")
    monkeypatch.setenv("KBFOLLOW_REL_CHUNK", "16")
    monkeypatch.setenv("KBFOLLOW_B_IN_LDS", "0")
    monkeypatch.setenv("KBFOLLOW_PLAIN_LOADS", plain)
    g = np.random.default_rng(b)
    n_e, n_r, n_t = 300, 7, 5000
    s, r, o = (g.integers(0, n, n_t).astype(np.int32) for n in (n_e, n_r, n_e - 40))
    w = g.uniform(0.1, 2.0, n_t).astype(np.float32) if weighted else None
    X, R, dY, Z = (g.standard_normal((b, n)).astype(np.float32) for n in (n_e, n_r, n_e, n_e))
    dev = [to_em(a) for a in (X, R, dY, Z)]
    want = outputs(kbf, [s, r, o], n_e, n_r, *dev, w)
    assert_close(want[0], oracle.follow(s, r, o, n_e, n_r, X, R, weight=w), "Y")
    monkeypatch.setenv("KBFOLLOW_MAX_LPT", max_lpt)
    kb = kbf.KB(s, r, o, n_e, n_r, weight=w)
    kernel = kb.phase_kernels(b)["fwd_stream"]
    kb.close()
    assert kernel.startswith(f"stream_kernel<-4, {max_lpt}," if b > 4 * int(max_lpt) else
                             "stream_kernel<-4, "), kernel
    got = outputs(kbf, [s, r, o], n_e, n_r, *dev, w)
    for i, (a, c) in enumerate(zip(got, want)):
        assert np.array_equal(a, c), (i, b, max_lpt)


# The narrow kernel (a lane per entry): every width, chunks of one, several and
# many steps, B in LDS (few relations) and not (1500 relations at b = 4; X in dR).
@pytest.mark.parametrize("b", [1, 2, 3, 4])
@pytest.mark.parametrize("chunk,n_r,weighted", [("8", 7, False), ("16", 7, True), ("24", 5, False),
                                                ("40", 1500, False), ("256", 7, False),
                                                ("256", 6000, True)])
def test_narrow_widths(kbf, b, chunk, n_r, weighted, monkeypatch):
    monkeypatch.setenv("KBFOLLOW_CHUNK", chunk)
    monkeypatch.setenv("KBFOLLOW_REL_CHUNK", chunk)
    g = np.random.default_rng(b + n_r)
    n_e, n_t = 300, 9000
    s = np.where(g.random(n_t) < 0.3, g.integers(0, 3, n_t), g.integers(0, n_e, n_t))
    o = np.where(g.random(n_t) < 0.3, g.integers(0, 3, n_t), g.integers(0, n_e - 40, n_t))
    r = g.integers(0, n_r, n_t)
    kb_args = [a.astype(np.int32) for a in (s, r, o)]
    w = g.uniform(0.1, 2.0, n_t).astype(np.float32) if weighted else None
    draw = lambda n: g.standard_normal((b, n)).astype(np.float32)  # noqa: E731
    X, R, dY, Z = draw(n_e), draw(n_r), draw(n_e), draw(n_e)
    dev = [to_em(a) for a in (X, R, dY, Z)]
    got = outputs(kbf, kb_args, n_e, n_r, *dev, w)
    again = outputs(kbf, kb_args, n_e, n_r, *dev, w)
    dXo, dRo = oracle.follow_backward(*kb_args, n_e, n_r, X, R, dY, weight=w)
    dXr, _ = oracle.follow_backward_residual(*kb_args, n_e, n_r, X, R, dY, 0.5, weight=w)
    Yo = oracle.follow(*kb_args, n_e, n_r, X, R, weight=w)
    Yr = oracle.follow_residual(*kb_args, n_e, n_r, X, R, 0.5, weight=w)
    Zo = (Yo.astype(np.float64) + 2.0 * Z).astype(np.float32)
    for name, a, c in zip(("Y", "Y residual", "Z", "dX", "dR", "dX residual", "dR residual"), got,
                          (Yo, Yr, Zo, dXo, dRo, dXr, dRo)):
        # Z adds two rounded floats in the expectation: its own tolerance.
        if name == "Z":
            np.testing.assert_allclose(a, c, rtol=1e-5, atol=2e-6)
        else:
            assert_close(a, c, name)
    for a, c in zip(got, again):
        assert np.array_equal(a, c)


def test_narrow_keeps_infinities_in_their_rows(kbf):
    """A row that gathers an infinity or a NaN does not touch its neighbours in
    the scan, and a marker's place adds nothing."""
    n_e, n_t, b = 64, 600, 2
    g = np.random.default_rng(5)
    s = g.integers(0, n_e, n_t).astype(np.int32)
    o = np.sort(g.integers(0, n_e, n_t)).astype(np.int32)
    r = g.integers(0, 3, n_t).astype(np.int32)
    X = g.random((b, n_e)).astype(np.float32) + 0.5
    X[0, 7], X[1, 9] = np.inf, np.nan
    R = g.random((b, 3)).astype(np.float32) + 0.5
    kb = kbf.KB(s, r, o, n_e, 3)
    Y = from_em(kb.follow(to_em(X), to_em(R)))
    kb.close()
    want = np.zeros((b, n_e))
    for l in range(n_t):
        want[:, o[l]] += X[:, s[l]].astype(np.float64) * R[:, r[l]]
    assert np.array_equal(np.isfinite(Y), np.isfinite(want))
    assert np.array_equal(np.isnan(Y), np.isnan(want))
    ok = np.isfinite(want)
    np.testing.assert_allclose(Y[ok], want[ok], rtol=1e-6)
