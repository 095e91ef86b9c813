"""The residual and accumulating passes read X and Z through one buffer over both
arrays: Z before X and after it in memory, in place, and so far apart that
plain loads are taken, bit for bit the same."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, from_em, to_em

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [8, 32, 33, 128])
@pytest.mark.parametrize("weighted", [False, True])
def test_z_anywhere(b, weighted, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2002_06115_amd as kbf
    g = np.random.default_rng(b)
    n_e, n_r, n_t = 500, 9, 6000
    s, o = g.integers(0, n_e, n_t).astype(np.int32), g.integers(0, n_e - 60, n_t).astype(np.int32)
    r = g.integers(0, n_r, n_t).astype(np.int32)
    w = g.uniform(0.1, 2.0, n_t).astype(np.float32) if weighted else None
    X, R = (g.standard_normal((b, n)).astype(np.float32) for n in (n_e, n_r))
    Z = g.standard_normal((b, n_e)).astype(np.float32)
    want = oracle.follow(s, r, o, n_e, n_r, X, R, weight=w).astype(np.float64) + 0.5 * Z
    x, rr, z = to_em(X), to_em(R), to_em(Z)
    # One allocation of a little over 4 GB: places before and after X, near and far.
    pool = torch.empty(((1 << 32) + (64 << 20)) // 4, device="cuda")
    n = n_e * b

    def at(offset, src):
        t = pool[offset:offset + n].view(n_e, b)
        t.copy_(src)
        return t

    near, far = 16 << 18, (1 << 30) + (1 << 20)  # floats: 16 MB, 4 GB + 4 MB
    results = []
    for xo, zo in ((0, near), (near, 0), (0, far), (far, 0)):
        for plain in ("0", "1"):
            monkeypatch.setenv("KBFOLLOW_PLAIN_LOADS", plain)
            kb = kbf.KB(s, r, o, n_e, n_r, weight=w)
            xv, zv = at(xo, x), at(zo, z)
            results.append(from_em(kb.follow_accumulate(xv, rr, zv, 0.5)))
            kb.follow_accumulate(xv, rr, zv, 0.5, out=zv)
            results.append(from_em(zv))
            kb.close()
    assert_close(results[0], want.astype(np.float32), "accumulate")
    for i, a in enumerate(results[1:]):
        assert np.array_equal(a, results[0]), i
