"""gwf_fom through the binding on a stream of the caller's: its workspace is
freed on return, so it has to come from that stream's memory, or the current
stream could be given it again while the call still uses it."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


def test_workspace_belongs_to_the_call_s_stream(lib, monkeypatch):
    n = 5000
    snr = torch.full((n,), math.e, dtype=torch.float64, device="cuda")
    z = torch.zeros(n, dtype=torch.float64, device="cuda")
    inv = {"out": [0], "logdet": z, "status": torch.zeros(n, dtype=torch.int32, device="cuda"), "cov": z.view(1, 1, n)}
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    made = []
    empty = torch.empty

    def spy(*size, **kw):
        made.append((size, torch.cuda.current_stream()))
        return empty(*size, **kw)
    monkeypatch.setattr(torch, "empty", spy)
    for stream in (side, None):
        made.clear()
        J, _ = lib.fom_terms(snr, inv, 3, 1.0, 1.0, stream=stream)
        torch.cuda.synchronize()
        assert abs(float(J) - n) <= 1e-12 * n
        work = [s for size, s in made if size == (lib.FOM_WORK,)]
        assert work == [stream or torch.cuda.current_stream()]
