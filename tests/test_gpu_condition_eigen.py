"""The condition number and the statuses at cond_max are the same bits with the
eigen-decomposition as without it, and the eigenvalues and eigenvectors are those
of the normalised matrix, indefinite matrices beside positive definite ones.

The Jacobi ends with columns orthogonal to P u; the factor and the matrix carry
P u of the matrix's norm (1 to P): 64 P^2 u bounds residuals and orthogonality."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


@pytest.mark.parametrize("P", [1, 2, 5, 9, 11, 13, 14])
@pytest.mark.parametrize("method", ["cho", "cho_svd", "cho_dd", "svd"])
@pytest.mark.parametrize("mixed", [False, True])
def test_eigen_changes_no_condition_number(lib, P, method, mixed):
    n = 45
    rng = np.random.default_rng(P + 100)
    G = np.empty((n, P, P))
    for e in range(n):
        q, _ = np.linalg.qr(rng.normal(size=(P, P)))
        lam = np.geomspace(1.0, 10.0 ** -rng.uniform(0.0, 9.0), P)
        if mixed and e % 5 == 2 and P > 1:
            lam[-1] = -lam[-1]
        A = (q * lam) @ q.T
        A = 0.5 * (A + A.T)
        d = np.sqrt(np.diag(A)) if np.all(np.diag(A) > 0) else np.ones(P)
        G[e] = A / d[:, None] / d[None, :]
        np.fill_diagonal(G[e], 1.0 if np.all(np.diag(A) > 0) else np.diag(G[e]))
    F = torch.as_tensor(np.ascontiguousarray(np.moveaxis(G, 0, 2)), device="cuda")
    a = lib.covariance(F, method=method)
    b = lib.covariance(F, method=method, eigen=True)
    for k in ("cond", "status", "logdet", "cov", "sigma"):
        assert torch.equal(torch.nan_to_num(a[k].double(), nan=-7.0), torch.nan_to_num(b[k].double(), nan=-7.0)), k
    cut = float(a["cond"][n // 3])                # one matrix sits on the limit itself
    c, d = (lib.covariance(F, method=method, cond_max=cut, eigen=x) for x in (False, True))
    assert torch.equal(c["status"], d["status"]) and int(c["status"][n // 3]) == int(a["status"][n // 3])
    lam, V = b["eigval"].cpu().numpy(), b["eigvec"].cpu().numpy()
    tol = 64 * P * P * U
    for e in range(n):
        g, v, w = G[e], V[:, :, e], lam[:, e]
        assert np.all(np.diff(w) >= 0)
        assert np.abs(g @ v - v * w).max() <= tol and np.abs(v.T @ v - np.eye(P)).max() <= tol
        assert np.abs(w - np.linalg.eigvalsh(g)).max() <= tol
