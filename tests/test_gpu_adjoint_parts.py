"""gwf_plan_adjoint over its own work items (1024 points and more, shorter than
the plan's chunk), the plan's items where those are shorter still, and the
set-up's groups of four events: against the one-workgroup-per-event adjoint.

Both forms evaluate the same grid values and quadratic forms; they differ in
the order of the sums and in taking a direction's derivative per point or from
the summed coefficient gradients, a few hundred roundings of terms no larger
than the event's size for a Gbar scaled to the Fisher diagonal: 1e-12 of each
event's largest term."""
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


@pytest.mark.parametrize("chunk", [0, 512, 16384])
@pytest.mark.parametrize("kind,npts", [
    ("bns", [5000]),
    ("bns", [2, 127, 128, 129, 255, 257]),
    ("bns", [1023, 1024, 1025, 2049, 3000]),
    ("mixed", [4097, 1500, 2, 8191]),
    ("still", [1025, 640, 2048, 33]),
    ("ecc", [1300, 2, 2047]),
])
def test_plan_adjoint_items_against_plain(lib, kind, npts, chunk):
    n = len(npts)
    wl = synth.mixed1e4(n=n, seed=7) if kind == "mixed" else synth.bns1e4(n=n)
    wl.npts = np.array(npts, dtype=np.int32)
    if kind == "still":
        wl.flags &= ~synth.FLAG_EARTH_ROT
    if kind == "ecc":
        wl = wl.with_eccentricity(np.full(n, 0.05))
    dw = lib.DeviceWorkload(wl)
    r = lib.fisher(dw)
    P = r["fisher"].shape[0]
    d = torch.sqrt(torch.diagonal(r["fisher"], dim1=0, dim2=1).T).clamp_min(1e-300)
    g = torch.as_tensor(np.random.default_rng(n).normal(size=(P, P, n)), device="cuda") / (d[:, None] * d[None])
    g = torch.where(torch.isfinite(g), g, torch.zeros_like(g))
    plan = lib.Plan(dw, chunk=chunk)
    got = [plan.adjoint(g, w_snr=0.7, w_fisher=1.3)["grad_event"].clone() for _ in range(2)]
    ref = lib.fisher_adjoint(dw, g, w_snr=0.7, w_fisher=1.3)["grad_event"]
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(got[0], got[1])
    scale = ref.abs().amax(dim=(1, 2), keepdim=True)
    assert bool((scale > 0).all())
    assert float(((got[0] - ref).abs() / scale).max()) < 1e-12
