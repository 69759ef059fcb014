"""Which form the plain calls take, on both sides of each line of the rule: the
number of events, the longest grid, the catalogue's points, explicit grids, the
workspace's limit; and the number of parts, one per stretch of the longest grid."""
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


SNR, FISHER, BOTH, IFOS = 0, 1, 2, 3


@pytest.mark.parametrize("n,npts,what,pop,parts", [
    (1, 2048, FISHER, "bns", None), (1, 2049, FISHER, "bns", 1), (1, 2560, BOTH, "bns", 1), (1, 2561, BOTH, "bns", 2),
    (1, 4096, SNR, "bns", None), (1, 4097, SNR, "bns", 2), (1, 8193, SNR, "bns", 3),
    (512, 600, FISHER, "bbh", None), (513, 600, FISHER, "bbh", 1), (513, 500, FISHER, "bbh", None),
    (512, 4096, SNR, "bbh", None), (513, 100, SNR, "bbh", 1),
    (1, 100, IFOS, "bns", 1), (1, 100, IFOS, "bbh", None), (1, 20000, IFOS, "bbh", 7),
    (2, 64 * 2560, FISHER, "bbh", 64), (2, 64 * 2560 + 1, FISHER, "bbh", 64), (2, 2, SNR, "bbh", None)])
def test_rule(lib, monkeypatch, n, npts, what, pop, parts):
    wl = synth.bns1e4(n=n, seed=3).with_npts(npts) if pop == "bns" else synth.bbh100(n=n, npts=npts, seed=3)
    dw = lib.DeviceWorkload(wl)
    ev, net, grid, keep = dw.descriptors()
    got = lib._split(dw, net, what, None)
    assert (None if got is None else got[0]) == parts
    if got is None:
        return
    size = got[1].numel()
    assert size == lib.load().gwf_split_bytes(n, ctypes.byref(net), dw.flags, what, parts)
    monkeypatch.setattr(lib, "SPLIT_WORK_MAX", size - 1)
    assert lib._split(dw, net, what, None) is None
    gx = lib.DeviceWorkload(wl.with_grid_f([np.geomspace(10.0, 200.0, npts)] * n))
    ev, net, grid, keep = gx.descriptors()
    monkeypatch.setattr(lib, "SPLIT_WORK_MAX", size)
    assert lib._split(gx, net, what, None) is None
