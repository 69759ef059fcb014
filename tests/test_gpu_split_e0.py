"""Eccentric catalogues with events whose e0 or reference frequency is refused:
the SNR does not know e0, so with a threshold or per-interferometer SNRs such an
event keeps its circular SNRs beside its status, in gwf_fisher_split as in
gwf_fisher.  Statuses and zeros equal, SNRs to 1e-12 (the same terms in another
order), against each other and against the circular catalogue."""
import ctypes

import numpy as np
import pytest

from paper_2207_06910_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


def _workload():
    wl = synth.bns1e4(n=10, seed=41)
    wl.npts = np.array([2, 700, 1025, 5000, 9000, 600, 513, 3000, 2100, 800], dtype=np.int32)
    e0, fref = np.full(10, 0.05), np.full(10, 10.0)
    e0[1], e0[3], e0[4], fref[5], fref[6] = 1.2, np.nan, -0.1, -3.0, np.inf
    wl = wl.with_eccentricity(e0.clip(0, 0.9), fref.clip(1.0, 20.0))
    wl.ecc, wl.f_ref_ecc = e0, fref
    wl.par[1, 7] = 0.3                            # eta beyond 1/4: refused in the SNR too
    return wl


@pytest.mark.parametrize("th", [0.0, 1e-3, "median", 1e9])
@pytest.mark.parametrize("per_ifo", [False, True])
def test_refused_e0(lib, monkeypatch, th, per_ifo):
    wl = _workload()
    dw = lib.DeviceWorkload(wl)
    real = lib._split

    def call(parts):
        def split(d, net, what, stream):
            if not parts:
                return None
            size = lib.load().gwf_split_bytes(d.n, ctypes.byref(net), d.flags, what, parts)
            return parts, torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        monkeypatch.setattr(lib, "_split", split if parts is not None else real)
        r = lib.fisher(dw, snr_th=cut, per_ifo_snr=per_ifo)
        s = lib.snr(dw, per_ifo=True)
        out = {**r, "s.snr": s["snr"], "s.ifo": s["snr_ifo"], "s.status": s["status"]}
        return {k: v.cpu().numpy() for k, v in out.items()}

    cut = 0.0
    snr = call(0)["s.snr"]
    cut = float(np.median(snr[snr > 0])) if th == "median" else th
    ref = call(0)
    bad = [1, 3, 4, 5, 6]
    assert np.all(ref["status"][bad] & 9 > 0) and np.all(ref["s.status"][bad] == 0) and ref["s.status"][7] == 1
    assert np.all(ref["s.snr"][bad] > 0.0)
    if cut > 0.0:
        assert np.array_equal(ref["snr"][bad], ref["s.snr"][bad])
    if per_ifo:
        assert np.array_equal(ref["snr_ifo"][:, bad], ref["s.ifo"][:, bad])
    for parts in (1, 5, 64, None):
        got = call(parts)
        for k in ref:
            if ref[k].dtype.kind != "f":
                assert np.array_equal(got[k], ref[k]), (parts, k)
            elif k == "fisher":
                d = np.sqrt(np.einsum("iie->ie", ref[k]))
                assert np.all(np.abs(got[k] - ref[k]) <= 1e-12 * d[:, None] * d[None]), (parts, k)
            else:
                np.testing.assert_allclose(got[k], ref[k], rtol=1e-12, err_msg=f"{parts} {k}")
