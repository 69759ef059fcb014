"""network_fom_value with weights that are tensors: J keeps their shape and
carries their gradient, as a sum of tensors does, and equals the value with plain
numbers to the rounding of a sum of 2 n terms in another order (n u of their
size)."""
import pytest

torch = pytest.importorskip("torch")
from paper_2207_06910_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2207_06910_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    binding.load()
    return binding


def test_tensor_weights(lib):
    from paper_2207_06910_amd import autodiff
    dw = lib.DeviceWorkload(synth.mixed1e4(n=30, seed=3))
    xi = autodiff.site_parameters(dw)
    val = lambda a, b: autodiff.network_fom_value(xi, dw, a, b, rows=(3, 4))  # noqa: E731
    s, d = float(val(1.0, 0.0)[0]), float(val(0.0, 1.0)[0])
    tol = 60 * 2.0 ** -53 * (abs(s) + abs(d)) * 10
    w = torch.tensor([0.5, 2.0], dtype=torch.float64, device="cuda", requires_grad=True)
    J, ok = val(w, -1.5)
    assert J.shape == (2,) and bool(ok.any())
    assert (J.detach().cpu() - torch.tensor([0.5 * s - 1.5 * d, 2.0 * s - 1.5 * d], dtype=torch.float64)).abs().max() <= tol
    J.sum().backward()
    assert (w.grad.cpu() - s).abs().max() <= tol
    v = torch.tensor(0.25, dtype=torch.float64, device="cuda", requires_grad=True)
    J, _ = val(1.0, v)
    J.backward()
    assert J.shape == () and abs(float(v.grad) - d) <= tol and abs(J.item() - (s + 0.25 * d)) <= tol
