"""The plain calls (SNR, Fisher, per-interferometer Fisher) give an event the
same bits whatever form they take: one workgroup per event or the split form,
alone or among others, eagerly or replayed from a captured graph, with the
workspace or without.  Grids end before, at and after a stretch's and an
iteration's last point and beyond the most stretches; every set of parameters,
curves, eccentricity, the duty factor and a threshold."""
import numpy as np
import pytest

from paper_2207_06910_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = [2, 511, 513, 2560, 2561, 3072, 3073, 4096, 4097, 8193, 20000, 64 * 3072 + 5]


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


def _workload(flags, ecc, curves):
    wl = synth.catalog1e6(n=len(LENGTHS), seed=78)
    wl.npts = np.array(LENGTHS, dtype=np.int32)
    wl.flags, wl.npar = flags, 13 if flags & synth.FLAG_TIDAL else 11
    if not flags & synth.FLAG_TIDAL:
        wl.par_mask = None
    if curves:
        g = np.geomspace(1.0, 4000.0, 1500)
        wl.sites[1] = wl.sites[1].with_curve(g, (g / 15.0) ** -4 + 1 + (g / 250.0) ** 2, scale=1e-49)
    if ecc:
        wl = wl.with_eccentricity(np.linspace(0.0, 0.1, wl.n))
    return wl.with_duty_factor(0.9, seed=4)


def _calls(lib, dw, th=8.0):
    res = {"f": lib.fisher(dw), "t": lib.fisher(dw, snr_th=th, per_ifo_snr=True), "i": lib.fisher_ifo(dw),
           "s": lib.snr(dw, per_ifo=True)}
    torch.cuda.synchronize()
    return {f"{a}.{k}": v.cpu().numpy() for a, r in res.items() for k, v in r.items()}


@pytest.mark.parametrize("flags", [0, 1, 2, 3])
@pytest.mark.parametrize("ecc", [False, True])
@pytest.mark.parametrize("curves", [False, True])
def test_forms_agree_bit_for_bit(lib, monkeypatch, flags, ecc, curves):
    wl = _workload(flags, ecc, curves)
    dw = lib.DeviceWorkload(wl)
    taken = []
    real = lib._split
    monkeypatch.setattr(lib, "_split", lambda *a: taken.append(real(*a)) or taken[-1])
    split = _calls(lib, dw)
    assert all(t is not None for t in taken)
    monkeypatch.setattr(lib, "SPLIT_WORK_MAX", 0)         # no workspace: one workgroup per event
    del taken[:]
    plain = _calls(lib, dw)
    assert not any(taken)
    for k in split:
        assert np.array_equal(split[k], plain[k], equal_nan=True), k
    monkeypatch.undo()
    for e in (1, 5, 7, 10):                               # alone: other forms, other numbers of parts
        one = _calls(lib, lib.DeviceWorkload(wl.subset([e])))
        for k in one:
            assert np.array_equal(one[k][..., 0], split[k][..., e], equal_nan=True), (k, e)


def test_captured_calls_give_the_eager_bits(lib):
    dw = lib.DeviceWorkload(_workload(3, False, False))
    eager = _calls(lib, dw)
    outs = [{}, {}, {}, {}]
    calls = [lambda: lib.fisher(dw, out=outs[0]), lambda: lib.fisher(dw, snr_th=8.0, per_ifo_snr=True, out=outs[1]),
             lambda: lib.fisher_ifo(dw, out=outs[2]), lambda: lib.snr(dw, per_ifo=True, out=outs[3])]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for c in calls:
            c()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for c in calls:
            c()
    for rep in range(3):
        for o in outs:
            for v in o.values():
                v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for a, o in zip("ftis", outs):
            for k, v in o.items():
                assert np.array_equal(v.cpu().numpy(), eager[f"{a}.{k}"]), (rep, a, k)
