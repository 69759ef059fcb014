"""GPU: the split form of the plain calls (gwf_snr_split, gwf_fisher_split,
gwf_fisher_ifo_split) against the oracle and against the one-workgroup form:
grids that end before, at and after a part's and an iteration's last point,
one part and the most parts, invalid events between valid ones, the duty
factor, parameter sets, the SNR threshold, and sampled curves.

Bars as in the rest of the suite: SNR 1e-12, Fisher 1e-9 of
sqrt(G_ii G_jj); statuses, zeros and skipped events equal the one-workgroup
form's exactly, its sums to 1e-12 (the same terms in another order)."""
import ctypes

import numpy as np
import pytest

from paper_2207_06910_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = [2, 511, 512, 513, 1024, 1025, 1537, 2048, 2500, 700, 3000, 20000]


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


def _workload(flags=synth.FLAG_EARTH_ROT | synth.FLAG_TIDAL, ecc=False, invalid=True):
    wl = synth.catalog1e6(n=len(LENGTHS), seed=77)
    wl.npts = np.array(LENGTHS, dtype=np.int32)
    wl.flags, wl.npar = flags, 13 if flags & synth.FLAG_TIDAL else 11
    if not flags & synth.FLAG_TIDAL:
        wl.par_mask = None
    if ecc:
        wl = wl.with_eccentricity(np.linspace(0.0, 0.1, wl.n))
    wl = wl.with_duty_factor(0.8, seed=3)
    wl.active[:, 4] = 0                       # every interferometer off
    wl.active[:, [0, 1, 2, 11]] = 1
    if invalid:
        wl.par[1, 3] = 0.3                    # eta beyond 1/4
        wl.npts[9] = 1
        wl.par[0, 5] = np.nan
    return wl


def _forced(lib, monkeypatch, parts):
    """Every plain call in the split form with this many parts (0: none)."""
    def split(dw, net, what, stream):
        if not parts:
            return None
        size = lib.load().gwf_split_bytes(dw.n, ctypes.byref(net), dw.flags, what, parts)
        assert size > 0
        work = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")    # NaN wherever not written
        return parts, work
    monkeypatch.setattr(lib, "_split", split)


def _np(r):
    return {k: v.cpu().numpy() for k, v in r.items()}


def _calls(lib, dw):
    """Every plain call's outputs."""
    a = _np(lib.fisher(dw))
    b = _np(lib.fisher(dw, snr_th=float(np.median(a["snr"])), per_ifo_snr=True))
    c = _np(lib.fisher_ifo(dw))
    d = _np(lib.snr(dw, per_ifo=True))
    return {f"{n}.{k}": v for n, r in zip("abcd", (a, b, c, d)) for k, v in r.items()}


def _close(k, x, y):
    if x.dtype.kind != "f":
        assert np.array_equal(x, y), k
    elif "fisher" in k:
        assert np.array_equal(x == 0.0, y == 0.0), k
        d = np.sqrt(np.abs(np.einsum("...iie->...ie", y)))
        assert np.all(np.abs(x - y) <= 1e-12 * d[..., :, None, :] * d[..., None, :, :]), k
    else:
        np.testing.assert_allclose(x, y, rtol=1e-12, err_msg=k)


@pytest.mark.parametrize("flags,ecc", [(0, False), (synth.FLAG_EARTH_ROT, True), (synth.FLAG_TIDAL, False),
                                       (synth.FLAG_EARTH_ROT | synth.FLAG_TIDAL, False),
                                       (synth.FLAG_EARTH_ROT | synth.FLAG_TIDAL, True)])
def test_split_equals_one_workgroup(lib, monkeypatch, flags, ecc):
    dw = lib.DeviceWorkload(_workload(flags, ecc))
    _forced(lib, monkeypatch, 0)
    ref = _calls(lib, dw)
    assert {0, 1, 8, 16} <= set(ref["b.status"])
    for parts in (1, 3, 40, 64):
        _forced(lib, monkeypatch, parts)
        got = _calls(lib, dw)
        assert set(got) == set(ref)
        for k in ref:
            _close(k, got[k], ref[k])


def test_split_against_oracle(lib, orc, monkeypatch):
    wl = _workload(invalid=False)
    g = np.geomspace(1.0, 4000.0, 1500)
    wl.sites[1] = wl.sites[1].with_curve(g, 1e-1 * ((g / 15.0) ** -4 + 1 + (g / 250.0) ** 2), scale=1e-49)
    dw = lib.DeviceWorkload(wl)
    _forced(lib, monkeypatch, 7)
    ref = orc.fisher(wl, per_ifo=True)
    r, s = _np(lib.fisher(dw)), _np(lib.snr(dw, per_ifo=True))
    assert np.all(r["status"] == 0)
    np.testing.assert_allclose(r["snr"], ref["snr"], rtol=1e-12)
    np.testing.assert_allclose(s["snr_ifo"], ref["snr_ifo"], rtol=1e-12)
    d = np.sqrt(np.abs(np.einsum("iie->ie", ref["fisher"])))
    assert np.all(np.abs(r["fisher"] - ref["fisher"]) <= 1e-9 * d[:, None, :] * d[None, :, :])


def test_workspace_arguments(lib):
    """Too small, misaligned or missing workspace and part counts out of range
    are refused before any launch."""
    dw = lib.DeviceWorkload(_workload())
    ev, net, grid, keep = dw.descriptors()
    L = lib.load()
    size = L.gwf_split_bytes(dw.n, ctypes.byref(net), dw.flags, 0, 4)
    work = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
    snr = torch.full((dw.n,), -1.0, dtype=torch.float64, device="cuda")

    def call(parts, ptr, nbytes):
        return L.gwf_snr_split(ctypes.byref(ev), ctypes.byref(net), ctypes.byref(grid), dw.flags, parts,
                               snr.data_ptr(), None, None, ptr, nbytes, lib._stream(None))
    p = work.data_ptr()
    assert [call(4, p, size - 1), call(4, None, size), call(4, p + 8, size), call(0, p, size),
            call(65, p, size)] == [lib.GWF_E_INVALID_ARG] * 5
    torch.cuda.synchronize()
    assert np.all(snr.cpu().numpy() == -1.0)
    assert call(4, p, size) == lib.GWF_OK
    torch.cuda.synchronize()
    assert np.all(snr.cpu().numpy() >= 0.0)
