"""Which C entry points the autograd form of the energy calls, on the CPU with
a recorder in the library's place: the gradient's first half is computed in the
forward only where a backward with respect to c can follow."""
import pytest

torch = pytest.importorskip("torch")

HALF, E_ONLY = "fft3d_energy_vpsi_fwd", "fft3d_energy"


@pytest.fixture
def calls(monkeypatch):
    from paper_2006_08435_amd import autograd

    names = []

    class Recorder:
        def __getattr__(self, name):
            return lambda *args: names.append(name) or 0

    class Plan:
        handle = 0

    monkeypatch.setattr(autograd._lib, "lib", lambda: Recorder())
    monkeypatch.setattr(autograd, "get_plan", lambda *args: Plan())
    monkeypatch.setattr(autograd, "_stream_handle", lambda: 0)
    monkeypatch.setattr(autograd, "_check_energy_args", lambda c, V: (c.unsqueeze(0) if c.dim() == 3 else c, V))
    return names


def make(c_grad, V_grad):
    c = torch.zeros((2, 3, 4, 4), dtype=torch.complex64).requires_grad_(c_grad)
    return c, torch.zeros((3, 4, 4)).requires_grad_(V_grad)


@pytest.mark.parametrize("off", [torch.no_grad, torch.inference_mode])
@pytest.mark.parametrize("save_psi", [True, False])
def test_evaluation_without_grad_mode(calls, off, save_psi):
    from paper_2006_08435_amd.autograd import local_potential_energy
    c, V = make(True, False)
    with off():
        E = local_potential_energy(c, V, save_psi)
    assert not E.requires_grad
    assert calls == [E_ONLY]


@pytest.mark.parametrize("c_grad,V_grad", [(False, False), (False, True)])
def test_c_without_gradient(calls, c_grad, V_grad):
    from paper_2006_08435_amd.autograd import local_potential_energy
    c, V = make(c_grad, V_grad)
    E = local_potential_energy(c, V)
    assert calls == [E_ONLY]
    if V_grad:      # V's gradient is not provided; c may change before a backward
        c.zero_()
        E.backward()
        assert V.grad is None and calls == [E_ONLY]


@pytest.mark.parametrize("V_grad", [False, True])
@pytest.mark.parametrize("save_psi,want", [(True, [HALF, "fft3d_energy_vpsi_bwd"]), (False, [E_ONLY, "fft3d_energy_bwd"])])
def test_training_step(calls, save_psi, want, V_grad):
    from paper_2006_08435_amd.autograd import local_potential_energy
    c, V = make(True, V_grad)
    E = local_potential_energy(c, V, save_psi)
    E.backward()
    assert calls == want
    assert c.grad is not None and c.grad.shape == c.shape and V.grad is None


def test_intermediate_c_in_grad_mode(calls):
    """c is not a leaf but follows from one."""
    from paper_2006_08435_amd.autograd import local_potential_energy
    c, V = make(True, False)
    local_potential_energy(2 * c, V).backward()
    assert calls == [HALF, "fft3d_energy_vpsi_bwd"]
    assert c.grad is not None
