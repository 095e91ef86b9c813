"""Column operations of the chain glue over long columns (the rows cut into
ranges, two launches with scratch) and at the edges of both paths' tiles,
against float64 formulas, with infinities and NaN as the one-launch form
treats them."""
import ctypes

import numpy as np
import pytest

from gpu_util import assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def chain():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_06115_amd import chain
    return chain


def cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.cpu().numpy().astype(np.float64)


# The last rows of the one-launch path and the first of the other; a last range
# of one row; every tile width; columns beyond one tile.
SHAPES = [(128, 5), (129, 4), (2048, 6), (2049, 5), (4097, 1), (4097, 33), (5000, 2), (20_011, 3), (9001, 7),
          (12_345, 16), (43_000, 93), (8193, 128), (70_001, 17), (4099, 300)]


# Wide columns: the first and last widths of each tile of the one-launch path, on
# both sides of 128 rows, with tiles that no XCD's share of the grid is full of.
WIDE = [(3, 1023), (128, 1024), (129, 1024), (1000, 1025), (128, 4095), (200, 4095), (128, 4096),
        (129, 4096), (60, 4100), (300, 5001)]


@pytest.mark.parametrize("n,b", SHAPES + WIDE)
def test_every_operation(chain, n, b):
    g = np.random.default_rng(n + b)
    z = (3 * g.standard_normal((n, b))).astype(np.float32)
    y = g.standard_normal((n, b)).astype(np.float32)
    t = (g.random((n, b)) < 3.0 / n).astype(np.float32) * np.float32(0.5)
    p = chain.softmax(cuda(z))
    z64, y64, t64 = (a.astype(np.float64) for a in (z, y, t))
    e = np.exp(z64 - z64.max(axis=0))
    want = e / e.sum(axis=0)
    assert_close(host(p), want, "softmax")
    pg = host(p)
    assert_close(host(chain.softmax_backward(p, cuda(y))), pg * (y64 - (y64 * pg).sum(axis=0)),
                 "softmax backward")
    u = np.abs(z)
    x, sums = chain.l1_normalize(cuda(u))
    np.testing.assert_allclose(host(sums), u.astype(np.float64).sum(axis=0), rtol=1e-13)
    assert_close(host(x), u / u.astype(np.float64).sum(axis=0), "l1")
    xg, sg = host(x), host(sums)
    assert_close(host(chain.l1_normalize_backward(x, sums, cuda(y))),
                 (y64 - (y64 * xg).sum(axis=0)) / sg, "l1 backward")
    loss, col, dz = chain.softmax_xent(cuda(z), cuda(t))
    logp = z64 - z64.max(axis=0) - np.log(e.sum(axis=0))
    np.testing.assert_allclose(host(col), -(t64 * logp).sum(axis=0), rtol=1e-12, atol=1e-14)
    assert_close(host(dz), (want * t64.sum(axis=0) - t64) / b, "xent dz")
    again = chain.softmax_xent(cuda(z), cuda(t))
    assert all((a == c).all() for a, c in zip((loss, col, dz), again))


@pytest.mark.parametrize("n", [300, 6000])
def test_infinities_and_nan(chain, n):
    """A column with -inf entries is a softmax over the others; +inf, NaN or
    nothing but -inf gives NaN in that column alone."""
    g = np.random.default_rng(n)
    z = g.standard_normal((n, 6)).astype(np.float32)
    t = np.full((n, 6), 1.0 / n, np.float32)
    z[: n // 2, 1] = -np.inf
    t[: n // 2, 1] = 0.0
    z[n - 1, 2] = np.inf
    z[n // 3, 3] = np.nan
    z[:, 4] = -np.inf
    z[:, 5] = -np.inf
    z[n - 2, 5] = 1.0
    p = host(chain.softmax(cuda(z)))
    dz = host(chain.softmax_xent(cuda(z), cuda(t))[2])
    with np.errstate(all="ignore"):
        z64 = z.astype(np.float64)
        e = np.exp(z64 - z64.max(axis=0))
        want = e / e.sum(axis=0)
        want_dz = (want * t.astype(np.float64).sum(axis=0) - t) / 6
    for c in (0, 1, 5):
        assert_close(p[:, c], want[:, c], f"softmax column {c}")
        assert_close(dz[:, c], want_dz[:, c], f"dz column {c}")
    for c in (2, 3, 4):
        assert np.isnan(want[:, c]).any()
        assert np.array_equal(np.isnan(p[:, c]), np.isnan(want[:, c])), c
    # Targets on finite logits only: a finite loss beside -inf logits has 0 * -inf.
    u = np.zeros((n, 2), np.float32)
    u[0, 0] = 2.0
    x, sums = chain.l1_normalize(cuda(u))
    assert host(sums)[0] == 2.0 and host(x)[0, 0] == 1.0
    assert np.isnan(host(x)[:, 1]).all()  # an empty column: 0 / 0


def test_scratch_and_plain_forms_agree(chain):
    """The plain C entries (no scratch) still take long columns; the *_scratch
    ones refuse scratch that is too small before launching."""
    import torch
    lib = chain._lib
    n, b = 30_000, 10
    u = torch.rand((n, b), device="cuda")
    x, sums = chain.l1_normalize(u)
    x2, s2 = torch.empty_like(x), torch.empty_like(sums)
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    P = ctypes.c_void_p
    lib.kbc_l1_normalize.argtypes = [ctypes.c_int64, ctypes.c_int32, P, P, P, P]
    assert lib.kbc_l1_normalize(n, b, p(u), p(x2), p(s2), stream) == 0
    torch.testing.assert_close(s2, sums, rtol=1e-13, atol=0)
    torch.testing.assert_close(x2, x, rtol=2e-7, atol=0)
    need = lib.kbc_scratch_size(n, b)
    assert need > 0
    small = torch.empty(need // 8, dtype=torch.float64, device="cuda")
    assert lib.kbc_l1_normalize_scratch(n, b, p(u), p(x2), p(s2), p(small), need - 8, stream) == 1
