"""The 64 x 64 tile factor at the edges of its 16-column panels: L, its inverse
and log-determinant against LAPACK on badly scaled tiles, and the row of the
first pivot that is not positive."""
import numpy as np
import pytest
import scipy.linalg as sla

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_06938_amd import dalia
    dalia.lib()
    return dalia


def _spd(n, seed, spread):
    rng = np.random.default_rng(seed)
    B = rng.standard_normal((n, n))
    s = 10.0 ** rng.uniform(-spread, spread, n)
    return s[:, None] * (B @ B.T / n + np.eye(n)) * s[None, :]


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x.T)).cuda().T


@pytest.mark.parametrize("n", [64, 192])
@pytest.mark.parametrize("spread", [0, 6])
@pytest.mark.parametrize("inverse", [False, True])
def test_factor_and_inverse(D, n, spread, inverse):
    A = _spd(n, n + spread, spread)
    Ad = _dev(A)
    ld, info = D.dpotrf(Ad, inverse=inverse)
    L = sla.cholesky(A, lower=True)
    want = sla.solve_triangular(L, np.eye(n), lower=True) if inverse else L
    got = Ad.cpu().numpy()
    assert int(info.item()) == 0 and np.array_equal(got, np.tril(got))
    assert abs(ld.item() - 2 * np.sum(np.log(np.diag(L)))) < 1e-12 * n * (1 + spread)
    # n eps cond of the scaled matrix (cond < 10), relative to the entry's
    # scale: row scaling for L, inverse column scaling for L^-1
    scale = np.abs(want).max(axis=0 if inverse else 1)
    err = np.abs(got - want) / (scale[None, :] if inverse else scale[:, None])
    assert err.max() < 100 * n * 2.2e-16


@pytest.mark.parametrize("bad", [1, 15, 16, 17, 32, 48, 63, 64, 65, 100, 128])
@pytest.mark.parametrize("value", [0.0, -1.0, float("nan")])
def test_first_bad_pivot(D, bad, value):
    n = 128
    A = np.diag(np.arange(2.0, n + 2.0))
    A[bad - 1, bad - 1] = value
    A[-1, -1] = A[-1, -1] if bad == n else -5.0  # a later one is not reported
    _, info = D.dpotrf(_dev(A))
    assert int(info.item()) == bad
