"""Lazily conjugated tensors (torch keeps x.conj() as a flag on x's memory) as
inputs and outputs: the same values as with the conjugate carried out first."""
import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 5e-6


@pytest.fixture(scope="module")
def F():
    import paper_2006_08435_amd as m
    from paper_2006_08435_amd import autograd  # noqa: F401
    return m


def grid(n, b, seed):
    return torch.from_numpy(workloads.uniform_grid(n, seed, batch=b)).cuda()


def done(x):
    return x.resolve_conj().clone()


def rel(a, b):
    return float((a.to(torch.complex128) - b).norm() / b.norm())


@pytest.mark.parametrize("side", [False, True])
def test_functions(F, side):
    x = grid(12, 3, 1)
    lazy = x.conj()
    assert lazy.is_conj() and lazy.is_contiguous()
    s = torch.cuda.Stream() if side else None
    for f in (F.fftn, F.ifftn):
        assert torch.equal(f(lazy), f(done(lazy)))
        assert torch.equal(f(lazy[0]), f(done(lazy[0])))
        assert torch.equal(f(lazy.transpose(1, 3)), f(done(lazy).transpose(1, 3)))
        out = torch.empty_like(x).conj()
        assert torch.equal(f(x, out), f(x)) and torch.equal(out, f(x))
    plan = F.Plan(12, 12, 12, 3)
    torch.cuda.synchronize()
    got, want = plan.exec(lazy, stream=s), plan.exec(done(lazy))
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert torch.equal(x, lazy.conj())                    # the input as it was
    own = done(lazy).conj().resolve_conj().conj()         # in place on a lazy tensor
    assert own.is_conj()
    want = plan.exec(done(own))
    torch.cuda.synchronize()
    r = plan.exec(own, own, stream=s)
    torch.cuda.synchronize()
    assert r is own and torch.equal(own, want)
    assert torch.equal(F.quantize(lazy), F.quantize(done(lazy)))


def test_operators(F):
    n, b, r2 = 20, 2, 30.0
    c = grid(n, b, 2)
    lazy = c.conj()
    V = torch.rand((n, n, n), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    neg = torch._neg_view(-V)
    assert neg.is_neg() and torch.equal(neg, V)
    occ = torch.tensor([0.5, 1.5], device="cuda")
    plan = F.Plan(n, n, n, b, "fp32", 1)
    E, E2 = (torch.zeros((), dtype=torch.float64, device="cuda") for _ in range(2))
    assert torch.equal(plan.apply_potential(lazy, neg, E=E), plan.apply_potential(done(lazy), V, E=E2))
    assert E.item() == E2.item() != 0.0
    out = torch.empty_like(c).conj()
    assert torch.equal(plan.apply_potential(c, V, out), plan.apply_potential(c, V)) and out.is_conj()
    assert torch.equal(plan.density(lazy, occ), plan.density(done(lazy), occ))
    plan.set_cutoff(r2)
    packed = plan.pack(lazy)
    assert torch.equal(packed, plan.pack(done(lazy)))
    assert torch.equal(plan.unpack(packed.conj()), plan.unpack(done(packed.conj())))
    dense = torch.empty_like(c).conj()
    assert torch.equal(plan.exec_packed(dense, packed.conj()), plan.exec_packed(torch.empty_like(c), done(packed.conj())))
    assert dense.is_conj()
    many = F.PlanMany([(24, 2), (30, 1)], 1)
    xs = [grid(24, 2, 3), grid(30, 1, 4)]
    want = [t.clone() for t in many.exec([done(xs[0].conj()), xs[1]])]
    outs = [torch.empty_like(xs[0]), torch.empty_like(xs[1]).conj()]
    for got in (many.exec([xs[0].conj(), xs[1]]), many.exec([xs[0].conj(), xs[1]], outs)):
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    rho = torch.rand((2, n, n, n), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    half = F.rfftn(rho)
    assert torch.equal(F.rfftn(torch._neg_view(-rho)), half)
    assert torch.equal(F.irfftn(half.conj(), n), F.irfftn(done(half.conj()), n))


def test_gradients_arrive_conjugated(F):
    """The gradient of a conjugate is a lazy conjugate: it reaches the backward
    of the transforms as a flag."""
    x = grid(10, 2, 5)
    w = grid(10, 2, 6)
    for f, g in ((F.FFT3D, torch.fft.fftn), (F.IFFT3D, lambda t, dim: torch.fft.ifftn(t, dim=dim, norm="forward"))):
        a = x.clone().requires_grad_(True)
        (f.apply(a).conj() * w).real.sum().backward()
        r = x.to(torch.complex128).requires_grad_(True)
        (g(r, dim=(1, 2, 3)).conj() * w.to(torch.complex128)).real.sum().backward()
        assert rel(a.grad, r.grad) <= TOL


@pytest.mark.parametrize("save_psi", [True, False])
def test_energy_of_a_conjugate(F, save_psi):
    c = grid(16, 2, 7)
    V = torch.rand((16, 16, 16), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")

    def step(x):
        a = x.detach().clone().requires_grad_(True)
        E = F.local_potential_energy(a.conj(), V, save_psi)
        E.backward()
        return E.item(), a.grad
    E, grad = step(c)
    psi = torch.fft.ifftn(c.to(torch.complex128).conj(), dim=(1, 2, 3), norm="forward")
    want = torch.fft.fftn(2 * V.double() * psi, dim=(1, 2, 3)).conj()
    assert abs(E - float((V.double() * psi.abs() ** 2).sum())) <= 1e-6 * E
    assert rel(grad.resolve_conj(), want) <= TOL
    assert F.energy(c.conj(), V).item() == F.energy(c.conj().resolve_conj(), V).item()
    # a lazily negated gradient of E
    a = c.clone().requires_grad_(True)
    F.local_potential_energy(a, V, save_psi).backward(torch._neg_view(torch.tensor(1.0, dtype=torch.float64, device="cuda")))
    b = c.clone().requires_grad_(True)
    F.local_potential_energy(b, V, save_psi).backward()
    assert torch.equal(a.grad, -b.grad)
