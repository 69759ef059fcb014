"""The condition number from the Cholesky factor's singular values (and from
the matrix's own where it has none), for every size P: against the
eigenvalues of the normalised matrix, with indefinite and non-finite matrices
among the positive definite ones of a wavefront.

The factor of a unit-diagonal matrix of condition kappa carries a relative
backward error of order P u in the matrix, which moves its smallest eigenvalue
by a relative P kappa u; the sweeps and numpy's eigenvalues add the same order
each: 16 P kappa u + 1e-12 bounds the sum."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


@pytest.mark.parametrize("P", list(range(1, 15)))
@pytest.mark.parametrize("method", ["cho", "cho_svd", "svd"])
def test_condition_number(lib, P, method):
    n = 41                                      # not a multiple of the four matrices of a wavefront
    rng = np.random.default_rng(P)
    A = np.empty((n, P, P))
    for e in range(n):
        q, _ = np.linalg.qr(rng.normal(size=(P, P)))
        lam = np.geomspace(1.0, 10.0 ** -rng.uniform(0.0, 6.0), P)
        if e % 7 == 3 and P > 1:
            lam[-1] = -lam[-1]                  # indefinite
        A[e] = (q * lam) @ q.T
        A[e] = 0.5 * (A[e] + A[e].T)
        s = 10.0 ** rng.uniform(-8.0, 8.0, P)   # rows of very different size
        A[e] *= s[:, None] * s[None, :]
    A[5, 0, 0] = np.nan
    F = torch.as_tensor(np.ascontiguousarray(np.moveaxis(A, 0, 2)), device="cuda")
    r = lib.covariance(F, method=method)
    cond, status = r["cond"].cpu().numpy(), r["status"].cpu().numpy()
    for e in range(n):
        if e == 5:
            assert status[e] != 0
            continue
        d = np.sqrt(np.diag(A[e])) if np.all(np.diag(A[e]) > 0) else np.ones(P)
        lam = np.abs(np.linalg.eigvalsh(A[e] / d[:, None] / d[None, :]))
        k = lam.max() / lam.min()
        if k * 1.1e-16 * 16 * P > 0.1:          # rows left unnormalised: no digit to compare
            continue
        assert abs(cond[e] / k - 1.0) <= 16 * P * k * 1.1e-16 + 1e-12, (e, cond[e], k)
    # a matrix's result does not depend on those that share its wavefront
    alone = lib.covariance(F[:, :, 8:9].contiguous(), method=method)
    assert float(alone["cond"][0]) == cond[8]
    assert torch.equal(alone["cov"][:, :, 0], r["cov"][:, :, 8])
