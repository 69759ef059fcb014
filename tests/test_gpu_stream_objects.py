"""Streams given to the plain calls: a torch stream, an external one, the null
stream, and any object that carries a stream's handle as ``cuda_stream``, for
calls that take a workspace and calls that do not; the results are those on the
current stream, bit for bit."""
import numpy as np
import pytest

from paper_2207_06910_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class Handle:
    def __init__(self, cuda_stream):
        self.cuda_stream = cuda_stream


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


@pytest.mark.parametrize("npts", [400, 7000])
def test_any_object_with_a_handle(lib, npts):
    dw = lib.DeviceWorkload(synth.bns1e4(n=5, seed=9).with_npts(npts))
    side = torch.cuda.Stream()

    def calls(stream):
        out = {"f": lib.fisher(dw, snr_th=2.0, stream=stream), "s": lib.snr(dw, per_ifo=True, stream=stream),
               "i": lib.fisher_ifo(dw, stream=stream)}
        torch.cuda.synchronize()
        return {f"{a}.{k}": v.cpu().numpy() for a, r in out.items() for k, v in r.items()}

    ref = calls(None)
    for stream in (side, torch.cuda.ExternalStream(side.cuda_stream), Handle(side.cuda_stream), Handle(0), Handle(None)):
        torch.cuda.synchronize()
        got = calls(stream)
        for k in ref:
            assert np.array_equal(got[k], ref[k]), k
