"""A sampled noise curve whose last value is infinite: the detector is blind in
the last interval, as it is beyond the last sample, so every call gives the
bits of the curve that ends one sample earlier (no grid point lies on a sample;
the values of the other intervals do not depend on the samples' number)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2207_06910_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


@pytest.mark.parametrize("asd", [False, True])
@pytest.mark.parametrize("ecc", [False, True])
def test_blind_last_interval(lib, asd, ecc):
    f = np.geomspace(3.0, 701.0, 400)
    f = np.append(f, 1300.0)                    # a wide last interval, inside the grids
    S = (f / 15.0) ** -4 + 1.0 + (f / 250.0) ** 2
    S[-1] = np.inf

    def calls(cut):
        wl = synth.bns1e4(n=5, seed=12)
        wl.npts = np.array([300, 900, 2500, 5000, 777], dtype=np.int32)
        if ecc:
            wl = wl.with_eccentricity(np.full(wl.n, 0.03))
        wl.sites = [s.with_curve(f[:cut], np.sqrt(S[:cut]) if asd else S[:cut], asd=asd, scale=1e-49)
                    for s in wl.sites]
        dw = lib.DeviceWorkload(wl)
        r, s = lib.fisher(dw), lib.snr(dw, per_ifo=True)
        th, fi = lib.fisher(dw, snr_th=1.0, per_ifo_snr=True), lib.fisher_ifo(dw)
        P = r["fisher"].shape[0]
        g = torch.as_tensor(np.random.default_rng(0).normal(size=(P, P, wl.n)), device="cuda")
        plan = lib.Plan(dw, chunk=1024)
        mixed = lib.Plan(dw, chunk=1024, mixed=True)
        out = {"fisher": r, "snr": s, "th": th, "ifo": fi, "plan": plan.run(), "mixed": mixed.run(),
               "adj": lib.fisher_adjoint(dw, g), "adj_plan": plan.adjoint(g)}
        torch.cuda.synchronize()
        plan.close()
        mixed.close()
        return {f"{a}.{k}": v.cpu().numpy() for a, d in out.items() for k, v in d.items()}

    got, ref = calls(len(f)), calls(len(f) - 1)
    assert np.all(ref["fisher.status"] == 0) and np.all(ref["snr.snr"] > 1.0)
    for k in ref:
        assert np.all(np.isfinite(ref[k])), k
        assert np.array_equal(got[k], ref[k]), k
