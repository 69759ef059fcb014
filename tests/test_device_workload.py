"""A DeviceWorkload takes its grid lengths from anything numpy makes an array of,
and counts its points (by which the plain calls choose their form) from them;
on host memory here, no call made."""
import numpy as np
import pytest

from paper_2207_06910_amd import binding, synth

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("form", [np.asarray, list, tuple, torch.as_tensor, lambda a: a.astype(np.int64),
                                  lambda a: torch.as_tensor(a, dtype=torch.int64)])
@pytest.mark.parametrize("n", [0, 1, 5])
def test_grid_lengths(form, n):
    wl = synth.bns1e4(n=5)
    npts = np.array(wl.npts[:n], dtype=np.int32)
    wl = wl.subset(np.arange(n))
    wl.npts = form(npts)
    dw = binding.DeviceWorkload(wl, device="cpu")
    assert dw.npts.dtype == torch.int32 and dw.npts.tolist() == npts.tolist()
    assert (dw.points_max, dw.points) == (max(npts.tolist(), default=0), int(npts.sum()))
