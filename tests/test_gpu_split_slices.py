"""GPU: the split form of a catalogue whose constants and partial sums need more
than the workspace's limit (GWF_SPLIT_SLICE_BYTES) takes the events in slices:
every plain call's outputs, bit for bit those of the one-workgroup form, for
sizes that two and three slices share unevenly, with an output row longer than a
slice, the duty factor, parameter sets, e0, invalid events and the threshold;
and the real rule takes such a catalogue in the split form."""
import ctypes

import numpy as np
import pytest

from paper_2207_06910_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LIMIT = 256 << 20
SNR, FISHER, BOTH, IFOS = 0, 1, 2, 3


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


def _workload(n, ecc=False):
    wl = synth.catalog1e6(n=n, seed=79)
    wl.npts = np.random.Generator(np.random.PCG64(5)).integers(2, 40, n).astype(np.int32)
    wl.npts[[0, n // 2, n - 1]] = 6000               # long ones at the ends of slices
    if ecc:
        wl = wl.with_eccentricity(np.linspace(0.0, 0.1, n))
    wl = wl.with_duty_factor(0.85, seed=6)
    wl.par[1, n // 3] = 0.3                          # eta beyond 1/4
    wl.npts[n - 2] = 1
    return wl


def _calls(lib, dw, what):
    if what == SNR:
        r = lib.snr(dw, per_ifo=True)
    elif what == IFOS:
        r = lib.fisher_ifo(dw)
    else:
        r = lib.fisher(dw, **({"snr_th": 8.0, "per_ifo_snr": True} if what == BOTH else {}))
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in r.items()}


@pytest.mark.parametrize("what,n,slices,ecc", [
    (FISHER, 6001, 2, False), (FISHER, 11003, 3, True), (BOTH, 6001, 2, True), (IFOS, 1500, 2, False),
    (IFOS, 2501, 3, False), (SNR, 70001, 2, False)])
def test_slices(lib, monkeypatch, what, n, slices, ecc):
    dw = lib.DeviceWorkload(_workload(n, ecc))
    net = dw.descriptors()[1]
    L = lib.load()
    size = L.gwf_split_bytes(n, ctypes.byref(net), dw.flags, what, 64)
    # the number of slices, from the linear growth of a workspace below the limit
    one = (L.gwf_split_bytes(512, ctypes.byref(net), dw.flags, what, 64)
           - L.gwf_split_bytes(256, ctypes.byref(net), dw.flags, what, 64)) / 256
    assert size <= LIMIT and int(np.ceil(n * one / LIMIT)) == slices
    monkeypatch.setattr(lib, "_split", lambda *a: None)
    ref = _calls(lib, dw, what)
    monkeypatch.setattr(lib, "_split",
                        lambda *a: (64, torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")))
    got = _calls(lib, dw, what)
    for k, v in ref.items():
        assert np.array_equal(got[k], v, equal_nan=True), k


def test_rule_takes_large_catalogues(lib):
    wl = synth.bns1e4(n=60000, seed=3).with_npts(10000)
    dw = lib.DeviceWorkload(wl)
    net = dw.descriptors()[1]
    for what, parts in ((SNR, 3), (FISHER, 4), (BOTH, 4), (IFOS, 4)):
        got = lib._split(dw, net, what, None)
        assert got is not None and got[0] == parts and got[1].numel() <= LIMIT
