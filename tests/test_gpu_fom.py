"""gwf_fom: the figure of merit's value and the covariances embedded in the
full matrix, against torch on the host, at the sizes where the workgroups'
split changes (one lane, one workgroup, several, more events than lanes).

The sums are of n terms of mixed sign in another order: n u times the sum of
the magnitudes bounds the difference; gbar is copied and must be equal."""
import math

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


@pytest.mark.parametrize("n", [1, 63, 256, 257, 65535, 65536, 70001])
@pytest.mark.parametrize("P,rows", [(13, (3, 4)), (11, tuple(range(11))), (14, (0, 13)), (3, (1,))])
def test_fom_terms(lib, n, P, rows):
    rng = np.random.default_rng(n + P)
    snr = torch.as_tensor(rng.uniform(0.5, 200.0, n), device="cuda")
    status = torch.as_tensor(rng.integers(0, 3, n) * (rng.random(n) < 0.3), dtype=torch.int32, device="cuda")
    logdet = torch.as_tensor(rng.normal(0.0, 30.0, n), device="cuda")
    logdet[status != 0] = math.nan
    cov = torch.as_tensor(rng.normal(size=(len(rows), len(rows), n)), device="cuda")
    inv = {"out": list(rows), "logdet": logdet, "status": status, "cov": cov}
    J, gbar = lib.fom_terms(snr, inv, P, 0.7, -1.3)
    J2, none = lib.fom_terms(snr, inv, P, 0.7, -1.3, want_gbar=False)
    ok = (status == 0).cpu().numpy()
    a, b = np.log(snr.cpu().numpy()[ok]), logdet.cpu().numpy()[ok]
    want = 0.7 * math.fsum(a) - 1.3 * math.fsum(b)
    size = 0.7 * np.abs(a).sum() + 1.3 * np.abs(b).sum()
    assert J.shape == () and J.dtype == torch.float64 and none is None
    assert abs(float(J) - want) <= max(n, 8) * 2.0 ** -53 * size
    assert float(J) == float(J2)
    full = torch.zeros((P, P, n), dtype=torch.float64, device="cuda")
    idx = torch.as_tensor(rows, device="cuda")
    full[idx.view(-1, 1), idx.view(1, -1)] = cov
    assert torch.equal(gbar, full)


def test_fom_refuses_rows_beyond_the_matrix(lib):
    z = torch.zeros(4, dtype=torch.float64, device="cuda")
    inv = {"out": [3], "logdet": z, "status": torch.zeros(4, dtype=torch.int32, device="cuda"), "cov": z.view(1, 1, 4)}
    with pytest.raises(lib.GwfError):
        lib.fom_terms(z, inv, 3, 1.0, 1.0)
