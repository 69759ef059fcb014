"""GPU: the strain and its derivatives where an event's grid is shared out over
workgroups: every alignment of an event's first column (runs start on lines
of eight columns), grids shorter and longer than one run, more workgroups than
runs, invalid events, gaps that must stay untouched, against the oracle.

Bar of the strain (as in the strain tests): |dh| <= 1e-13 max |h| +
|h| (1e-13 + 64 u (|Psi_PN| + 2 pi f (|tc| + tau + 0.03 s)));
here the grids start at 40 Hz, where the phase stays below 1e4 rad, so
4e-10 of the largest |h| of the row bounds it; each derivative row alike."""
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


@pytest.mark.parametrize("n", [1, 13, 2100])
def test_alignment_and_parts(lib, orc, n):
    lengths = [2, 7, 249, 256, 257, 263, 511, 1030, 16, 300, 5, 64, 700]
    wl = synth.bns1e4(n=n, seed=900 + n)
    wl.fmin[:] = 40.0
    wl.npts = np.array([lengths[e % len(lengths)] for e in range(n)], dtype=np.int32)
    gap = (np.arange(n) * 3 + 1) % 11          # every first column modulo 8 occurs
    off = np.concatenate([[0], np.cumsum(wl.npts[:-1] + gap[:-1], dtype=np.int64)]) + 5
    total = int(off[-1] + wl.npts[-1] + 9)     # odd row strides as well
    if n > 5:
        wl.par[1, 5] = 0.4                     # invalid: writes nothing
    dw = lib.DeviceWorkload(wl)
    offd = torch.as_tensor(off, device="cuda")
    mark = 123.25
    h = torch.full((dw.n_ifo, total), mark, dtype=torch.complex128, device="cuda")
    dh = torch.full((13, dw.n_ifo, total), mark, dtype=torch.complex128, device="cuda") if n < 100 else None
    st = lib.waveform(dw, offd, total, out={"h": h})["status"].cpu().numpy()
    assert np.array_equal(st != 0, np.arange(n) == (5 if n > 5 else -1))
    if dh is not None:
        lib.waveform_deriv(dw, offd, total, out={"dh": dh})
        dh = dh.cpu().numpy()
    h = h.cpu().numpy()
    written = np.zeros(total, dtype=bool)
    sites = wl.site_array()
    for e in range(n):
        if st[e]:
            continue
        c = slice(int(off[e]), int(off[e]) + int(wl.npts[e]))
        written[c] = True
        if n > 100 and e % 61:
            continue
        f, _ = orc.grid(40.0, orc.cut_frequency(*wl.par[:2, e]), int(wl.npts[e]))
        ref, dref = orc.strain(wl.par[:, e], sites, f, wl.flags)
        big = np.abs(ref).max(axis=1, keepdims=True)
        assert np.all(np.abs(h[:, c] - ref) <= 4e-10 * big), e
        if dh is not None:
            d = np.moveaxis(dref, 2, 0)
            big = np.abs(d).max(axis=2, keepdims=True)
            assert np.all(np.abs(dh[:, :, c] - d) <= 4e-10 * big), e
    assert np.all(h[:, ~written] == mark) and np.all(h[:, written] != mark)
    if dh is not None:
        assert np.all(dh[:, :, ~written] == mark)
