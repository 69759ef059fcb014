"""GPU: Fisher matrices and SNR where the per-workgroup accumulation changes
its way: grids of one point less and more than a wavefront's, a workgroup's
and an iteration's points (256 lanes, two points each in the work-item form),
work items of the smallest length, each set of parameters, sites with none,
one or two effective interferometers, against the oracle.

Bars: SNR 1e-12 relative, Fisher 1e-9 of sqrt(G_ii G_jj) (mixed form 5e-7 and
1e-6), as everywhere in the suite: the accumulation is FP64 and its error does
not depend on the grid's length."""
import numpy as np
import pytest

from paper_2207_06910_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = [2, 3, 63, 65, 255, 256, 257, 511, 512, 513, 767, 1024, 1025]


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


def _workload(flags, ecc):
    """One event per grid length; interferometers off in turn, so that sites
    with zero, one and two effective interferometers occur (never all off)."""
    wl = synth.bns1e4(n=len(LENGTHS), seed=4242)
    wl.npts = np.array(LENGTHS, dtype=np.int32)
    wl.flags = flags
    wl.npar = 13 if flags & synth.FLAG_TIDAL else 11
    act = np.ones((wl.n_ifo, wl.n), dtype=np.uint8)
    for e in range(wl.n):
        act[e % 5, e] = 0
        if e % 3 == 0:
            act[[0, 1, 2] if e % 2 else [3, 4], e] = 0
    wl.active = act
    return wl.with_eccentricity(np.linspace(0.0, 0.1, wl.n)) if ecc else wl


def _check(r, ref, snr_tol=1e-12, f_tol=1e-9):
    snr, F = r["snr"].cpu().numpy(), r["fisher"].cpu().numpy()
    assert np.all(r["status"].cpu().numpy() == 0)
    np.testing.assert_allclose(snr, ref["snr"], rtol=snr_tol)
    d = np.sqrt(np.abs(np.einsum("iie->ie", ref["fisher"])))
    scale = d[:, None, :] * d[None, :, :]
    assert np.all(np.abs(F - ref["fisher"]) <= f_tol * scale)


@pytest.mark.parametrize("ecc", [False, True])
@pytest.mark.parametrize("flags", [0, synth.FLAG_EARTH_ROT, synth.FLAG_TIDAL,
                                   synth.FLAG_EARTH_ROT | synth.FLAG_TIDAL])
def test_grid_lengths(lib, orc, flags, ecc):
    wl = _workload(flags, ecc)
    dw = lib.DeviceWorkload(wl)
    ref = orc.fisher(wl)
    _check(lib.fisher(dw), ref)
    for chunk in (256, 512, 16384):
        plan = lib.Plan(dw, chunk=chunk)
        _check(plan.run(), ref)
        plan.close()
    plan = lib.Plan(dw, chunk=512, mixed=True)
    _check(plan.run(), ref, 5e-7, 1e-6)
    plan.close()
