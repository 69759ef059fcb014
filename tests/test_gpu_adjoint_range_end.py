"""The per-event adjoint where the grid ends inside a stride of 128 lanes: the
lanes past the end take part in the exchanges with a point of zeros (no weight,
a frequency outside every sampled curve), never with unset values, which a
sampled curve would search its table by.

Against the work-item form, which differs in the order of the sums only: 1e-12
of each event's largest term (the bar of the work items' own test).  An event
alone gives the bits it gives among others."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2207_06910_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.load()
    return binding


def _workload(ecc, uneven):
    wl = synth.bns1e4(n=9, seed=31)
    wl.npts = np.array([2, 3, 127, 128, 129, 255, 257, 1000, 130], dtype=np.int32)
    rng = np.random.default_rng(1)
    g = np.geomspace(4.0, 900.0, 700)           # grids reach beyond both ends
    if uneven:
        g[1:-1] = np.sort(rng.uniform(4.0, 900.0, 698))
    S = (g / 15.0) ** -4 + 1.0 + (g / 250.0) ** 2
    wl.sites = [s.with_curve(g, S if i else np.sqrt(S), asd=i == 0, scale=1e-49) for i, s in enumerate(wl.sites)]
    return wl.with_eccentricity(np.full(wl.n, 0.05)) if ecc else wl


@pytest.mark.parametrize("ecc", [False, True])
@pytest.mark.parametrize("uneven", [False, True])
def test_lanes_past_the_end(lib, ecc, uneven):
    wl = _workload(ecc, uneven)
    dw = lib.DeviceWorkload(wl)
    F = lib.fisher(dw)["fisher"]
    P = F.shape[0]
    d = torch.sqrt(torch.diagonal(F, dim1=0, dim2=1).T).clamp_min(1e-300)
    g = torch.as_tensor(np.random.default_rng(2).normal(size=(P, P, wl.n)), device="cuda") / (d[:, None] * d[None])
    g = torch.where(torch.isfinite(g), g, torch.zeros_like(g))
    got = lib.fisher_adjoint(dw, g, w_snr=0.7, w_fisher=1.3)["grad_event"]
    plan = lib.Plan(dw, chunk=512)
    ref = plan.adjoint(g, w_snr=0.7, w_fisher=1.3)["grad_event"]
    torch.cuda.synchronize()
    plan.close()
    scale = ref.abs().amax(dim=(1, 2), keepdim=True)
    seen = scale[:, 0, 0] > 0                    # the two-point grids lie outside the curves
    assert bool(seen[2:].all()) and bool(torch.isfinite(got[seen]).all())
    assert float(((got - ref).abs() / scale)[seen].max()) < 1e-12
    for e in (2, 4, 7):
        one = lib.fisher_adjoint(lib.DeviceWorkload(wl.subset([e])), g[:, :, e:e + 1].contiguous(), w_snr=0.7,
                                 w_fisher=1.3)["grad_event"]
        assert torch.equal(one[0], got[e])
