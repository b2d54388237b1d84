"""What is timed: the transforms and plane-wave operators that a program built on this package calls.

A case is a dict of plain values; its ``kind`` names one of the entry points
below and the other values give its sizes.  Grids are [batch][z][y][x], the
inputs are the plane-wave coefficients of the workloads in ``workloads`` (a
Gaussian-weighted sphere |G| < N/4), real densities, or, for a single small
box, uniform noise.  Everything is drawn on the GPU from the seed.

``exact`` computes the same values in 64 bits with torch's own FFT.
"""
from __future__ import annotations

import math

import torch

import paper_2006_08435_amd as fft3d
from paper_2006_08435_amd import FFT3D_FORWARD, FFT3D_INVERSE

# Every length 2^a 3^b 5^c: up to 128 points the two-pass forms, above it the three-pass one.
LENGTHS = [8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72, 75, 80, 81, 90, 96,
           100, 108, 120, 125, 128]
LARGE = [135, 144, 150, 160, 162, 180, 192, 200, 216, 225, 240, 243, 250, 256, 270, 288, 300, 320, 324, 360, 375, 384,
         400, 405, 432, 450, 480, 486, 500, 512]
MANY = [24, 30, 32, 36, 40, 48, 50, 60, 64, 72, 80, 90, 96, 100, 120, 128]
SCALED = [16, 32, 48, 64, 80, 96, 128]
EVEN = [n for n in LENGTHS if n % 2 == 0]

MAX_POINTS = 32 * 128 ** 3      # of one transform batch (67 million, 0.5 GiB of complex64)
MAX_ORBITAL_POINTS = 128 * 96 ** 3


def listed():
    return [
        # One small box through the plain functions: the paper's smallest grid.
        # A call at a time, so launches and host time are all there is.
        {"name": "box16", "kind": "functions", "nx": 16, "ny": 16, "nz": 16, "batch": 1},
        # The paper's 64^3 grid, one at a time: still launch- and latency-bound.
        {"name": "grid64", "kind": "functions", "nx": 64, "ny": 64, "nz": 64, "batch": 1},
        # The orbitals of a small molecule: a batch of small, not power-of-two grids.
        {"name": "molecule30", "kind": "plan", "nx": 30, "ny": 30, "nz": 30, "batch": 400},
        # The large batch of the benchmark: 32 grids of 128^3.
        {"name": "batch128", "kind": "plan", "nx": 128, "ny": 128, "nz": 128, "batch": 32},
        # An orthorhombic cell: three different lengths, none a power of two.
        {"name": "cell100x72x90", "kind": "plan", "nx": 100, "ny": 72, "nz": 90, "batch": 16},
        # A big cell at a density cutoff: grids whose planes exceed a compute unit.
        {"name": "large256", "kind": "plan", "nx": 256, "ny": 256, "nz": 256, "batch": 4},
        # 16-bit storage of the large batch, the result converted back.
        {"name": "fp16_128", "kind": "scaled", "n": 128, "batch": 32, "precision": "fp16"},
        # Orbitals and the grids of a multi-level basis in one call, as planned by default.
        {"name": "mixed", "kind": "many", "groups": "64x256,48x1,72x1,96x1,100x1,120x1"},
        # Training step of the plane-wave energy: E and its gradient over 128 orbitals.
        {"name": "energy96", "kind": "energy", "nx": 96, "ny": 96, "nz": 96, "batch": 128, "save_psi": True},
        # H psi of a plane-wave code: packed coefficients in, V applied on the grid, packed coefficients out.
        {"name": "hpsi90", "kind": "hpsi", "nx": 90, "ny": 90, "nz": 90, "batch": 64},
        # Electron density of the occupied orbitals, given inside the cutoff sphere.
        {"name": "density96", "kind": "density", "nx": 96, "ny": 96, "nz": 96, "batch": 128, "cutoff": True},
        # Real densities to reciprocal space and back.
        {"name": "real128", "kind": "real", "nx": 128, "ny": 128, "nz": 128, "batch": 32},
    ]


def _batch(rng, points, limit, most):
    """A batch of grids of `points` points, spread over the logarithm of its range."""
    top = max(1, min(most, limit // points))
    return max(1, min(top, round(math.exp(rng.uniform(0.0, math.log(top + 0.49))))))


def draw(rng):
    kind = rng.choice(["functions", "plan", "plan", "box", "large", "scaled", "many", "energy", "hpsi", "density",
                       "real"])
    if kind == "functions":     # single grids, cubic or not
        n = [rng.choice(LENGTHS) for _ in range(3)] if rng.random() < 0.3 else [rng.choice(LENGTHS)] * 3
        return {"kind": "functions", "nx": n[0], "ny": n[1], "nz": n[2], "batch": 1}
    if kind == "plan":          # batches of cubic grids, or of square planes with another height
        n = rng.choice(LENGTHS)
        nz = n if rng.random() < 0.75 else rng.choice(LENGTHS)
        return {"kind": "plan", "nx": n, "ny": n, "nz": nz, "batch": _batch(rng, n * n * nz, MAX_POINTS, 4096)}
    if kind == "box":           # batches of cells with three lengths
        nx, ny, nz = rng.choice(LENGTHS), rng.choice(LENGTHS), rng.choice(LENGTHS)
        return {"kind": "plan", "nx": nx, "ny": ny, "nz": nz, "batch": _batch(rng, nx * ny * nz, MAX_POINTS, 4096)}
    if kind == "large":         # grids above 128 points a side
        while True:
            nx, ny, nz = (rng.choice(LARGE) for _ in range(3))
            if rng.random() < 0.6:
                ny = nz = nx
            if nx * ny * nz <= MAX_POINTS:
                return {"kind": "plan", "nx": nx, "ny": ny, "nz": nz,
                        "batch": _batch(rng, nx * ny * nz, MAX_POINTS, 8)}
    if kind == "scaled":
        n = rng.choice(SCALED)
        return {"kind": "scaled", "n": n, "batch": _batch(rng, n ** 3, MAX_POINTS, 2048),
                "precision": rng.choice(["fp16", "bf16"])}
    if kind == "many":
        sizes = rng.sample(MANY, rng.randint(2, 6))
        share = MAX_POINTS // len(sizes)
        return {"kind": "many", "groups": ",".join("%dx%d" % (n, _batch(rng, n ** 3, share, 256)) for n in sizes)}
    if kind == "real":
        n = rng.choice(EVEN)
        nz = n if rng.random() < 0.75 else rng.choice(LENGTHS)
        return {"kind": "real", "nx": n, "ny": n, "nz": nz, "batch": _batch(rng, n * n * nz, MAX_POINTS, 1024)}
    # the operators over orbitals
    n = rng.choice(LENGTHS)
    nz = n if rng.random() < 0.75 else rng.choice(LENGTHS)
    case = {"kind": kind, "nx": n, "ny": n, "nz": nz, "batch": _batch(rng, n * n * nz, MAX_ORBITAL_POINTS, 256)}
    if kind == "energy":
        case["save_psi"] = rng.random() < 0.7
    if kind == "density":
        case["cutoff"] = rng.random() < 0.6
    return case


# ------------------------------------------------------------------ inputs --

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _signed(n):
    k = torch.arange(n, device="cuda")
    return torch.where(2 * k < n, k, k - n)


def _g2(nx, ny, nz):
    gz, gy, gx = _signed(nz), _signed(ny), _signed(nx)
    return gz[:, None, None] ** 2 + gy[None, :, None] ** 2 + gx[None, None, :] ** 2


def _cutoff(nx, ny, nz):
    """Squared radius of the sphere |G| < N/4, N the smallest side."""
    return (min(nx, ny, nz) / 4.0) ** 2


def _coefficients(nx, ny, nz, batch, seed):
    """Plane-wave coefficients: complex normal, Gaussian-weighted, zero outside the sphere."""
    g2 = _g2(nx, ny, nz)
    r2 = _cutoff(nx, ny, nz)
    weight = (torch.exp(-g2.double() / (r2 / 4.0)) * (g2 < r2)).float()
    c = torch.randn((batch, nz, ny, nx, 2), generator=_generator(seed), device="cuda")
    c *= weight[..., None]
    return torch.view_as_complex(c)


def _uniform(nx, ny, nz, batch, seed):
    u = torch.rand((batch, nz, ny, nx, 2), generator=_generator(seed), device="cuda")
    return torch.view_as_complex(u.mul_(2).sub_(1))


def _density(nx, ny, nz, batch, seed):
    """Real, positive grids."""
    return torch.rand((batch, nz, ny, nx), generator=_generator(seed), device="cuda").square_()


def _potential(nx, ny, nz, seed):
    """A smooth periodic potential: sixteen long waves."""
    gen = _generator(seed + 1)
    waves = torch.randint(-2, 3, (16, 3), generator=gen, device="cuda").double()
    amp = torch.rand(16, generator=gen, device="cuda").double() + 0.5
    phase = torch.rand(16, generator=gen, device="cuda").double() * (2 * math.pi)
    z = torch.arange(nz, device="cuda").double()[:, None, None] / nz
    y = torch.arange(ny, device="cuda").double()[None, :, None] / ny
    x = torch.arange(nx, device="cuda").double()[None, None, :] / nx
    v = torch.zeros((nz, ny, nx), dtype=torch.float64, device="cuda")
    for j in range(16):
        v += amp[j] * torch.cos(2 * math.pi * (waves[j, 0] * x + waves[j, 1] * y + waves[j, 2] * z) + phase[j])
    return v.float()


def _occupations(batch, seed):
    """Between 0 and 2 electrons an orbital."""
    return 2 * torch.rand(batch, generator=_generator(seed + 2), device="cuda")


def _groups(case):
    return [tuple(int(v) for v in g.split("x")) for g in case["groups"].split(",")]


def _grid_input(case, seed):
    nx, ny, nz, b = (case[k] for k in ("nx", "ny", "nz", "batch"))
    make = _uniform if max(nx, ny, nz) <= 16 else _coefficients
    return make(nx, ny, nz, b, seed)


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "scaled":
        n, b, p = case["n"], case["batch"], case["precision"]
        c = _coefficients(n, n, n, b, seed)
        s.update(shape=c.shape, precision=p, c=fft3d.quantize(c, p),
                 inverse=fft3d.Plan(n, n, n, b, p, FFT3D_INVERSE), forward=fft3d.Plan(n, n, n, b, p, FFT3D_FORWARD))
        s["psi"], s["back"] = torch.empty_like(s["c"]), torch.empty_like(s["c"])
        return s
    if kind == "many":
        groups = _groups(case)
        s["c"] = [_coefficients(n, n, n, b, seed + 10 * k) for k, (n, b) in enumerate(groups)]
        s["psi"] = [torch.empty_like(c) for c in s["c"]]
        s["plan"] = fft3d.PlanMany(groups, FFT3D_INVERSE)
        return s
    nx, ny, nz, b = (case[k] for k in ("nx", "ny", "nz", "batch"))
    if kind == "functions":
        s["c"] = _grid_input(case, seed)
    elif kind == "plan":
        s["c"] = _grid_input(case, seed)
        s["psi"], s["back"] = torch.empty_like(s["c"]), torch.empty_like(s["c"])
        s["inverse"] = fft3d.Plan(nx, ny, nz, b, "fp32", FFT3D_INVERSE)
        s["forward"] = fft3d.Plan(nx, ny, nz, b, "fp32", FFT3D_FORWARD)
    elif kind == "energy":
        s["c"] = _coefficients(nx, ny, nz, b, seed).requires_grad_(True)
        s["V"] = _potential(nx, ny, nz, seed)
        s["save_psi"] = case["save_psi"]
    elif kind == "hpsi":
        s["plan"] = fft3d.Plan(nx, ny, nz, b, "fp32", FFT3D_INVERSE)
        s["plan"].set_cutoff(_cutoff(nx, ny, nz))
        s["dense"] = _coefficients(nx, ny, nz, b, seed)
        s["packed"] = s["plan"].pack(s["dense"])
        s["result"] = torch.empty_like(s["packed"])
        s["V"] = _potential(nx, ny, nz, seed)
        s["E"] = torch.empty((), dtype=torch.float64, device="cuda")
    elif kind == "density":
        s["plan"] = fft3d.Plan(nx, ny, nz, b, "fp32", FFT3D_INVERSE)
        if case["cutoff"]:
            s["plan"].set_cutoff(_cutoff(nx, ny, nz))
        s["c"] = _coefficients(nx, ny, nz, b, seed)
        s["occ"] = _occupations(b, seed)
        s["rho"] = torch.empty((nz, ny, nx), device="cuda")
        s["work"] = torch.empty_like(s["c"])
    elif kind == "real":
        s["rho"] = _density(nx, ny, nz, b, seed)
        s["forward"] = fft3d.RealPlan(nx, ny, nz, b, FFT3D_FORWARD)
        s["inverse"] = fft3d.RealPlan(nx, ny, nz, b, FFT3D_INVERSE)
        s["half"] = torch.empty(s["forward"].half_shape, dtype=torch.complex64, device="cuda")
        s["back"] = torch.empty_like(s["rho"])
    else:
        raise ValueError("unknown kind %r" % kind)
    return s


# --------------------------------------------------------------------- run --

def run(s):
    kind = s["kind"]
    if kind == "functions":
        psi = fft3d.ifftn(s["c"])
        return {"psi": psi, "back": fft3d.fftn(psi)}
    if kind == "plan":
        s["inverse"].exec(s["c"], s["psi"])
        s["forward"].exec(s["psi"], s["back"])
        return {"psi": s["psi"], "back": s["back"]}
    if kind == "scaled":
        s["inverse"].exec(s["c"], s["psi"])
        s["forward"].exec(s["psi"], s["back"])
        return fft3d.dequantize(s["back"], s["shape"], s["precision"])
    if kind == "many":
        return s["plan"].exec(s["c"], s["psi"])
    if kind == "energy":
        s["c"].grad = None
        E = fft3d.local_potential_energy(s["c"], s["V"], s["save_psi"])
        E.backward()
        return {"E": E.detach(), "grad": s["c"].grad}
    if kind == "hpsi":
        plan, dense = s["plan"], s["dense"]
        plan.unpack(s["packed"], dense)
        plan.apply_potential(dense, s["V"], dense, s["E"])
        return {"hpsi": plan.pack(dense, s["result"]), "E": s["E"]}
    if kind == "density":
        return s["plan"].density(s["c"], s["occ"], s["rho"], s["work"])
    if kind == "real":
        s["forward"].exec(s["rho"], s["half"])
        return s["inverse"].exec(s["half"], s["back"])     # overwrites the half spectrum
    raise ValueError("unknown kind %r" % kind)


# -------------------------------------------------------------------- work --

def work(case):
    kind = case["kind"]
    if kind == "many":
        pts = [(n ** 3, b) for n, b in _groups(case)]
        return {"bytes": sum(16 * v * b for v, b in pts), "flops": sum(5 * v * math.log2(v) * b for v, b in pts)}
    if kind == "scaled":
        v, b = case["n"] ** 3, case["batch"]
        per = 4 * v + case["n"] ** 2
        # inverse and forward on 16-bit grids, then the conversion to complex64
        return {"bytes": b * (4 * per + per + 8 * v), "flops": 2 * 5 * v * math.log2(v) * b}
    nx, ny, nz, b = (case[k] for k in ("nx", "ny", "nz", "batch"))
    v = nx * ny * nz
    flops = 5 * v * math.log2(v) * b
    inside = math.pi * 4 / 3 * _cutoff(nx, ny, nz) ** 1.5
    if kind in ("functions", "plan"):
        return {"bytes": 32 * v * b, "flops": 2 * flops}
    if kind == "energy":        # c in, the gradient out
        return {"bytes": 16 * v * b + 4 * v, "flops": 2 * flops}
    if kind == "hpsi":          # the sphere in and out
        return {"bytes": 16 * inside * b + 4 * v, "flops": 2 * flops}
    if kind == "density":
        return {"bytes": 8 * (inside if case["cutoff"] else v) * b + 4 * v, "flops": flops}
    half = (nx // 2 + 1) * ny * nz
    return {"bytes": b * 2 * (4 * v + 8 * half), "flops": flops}


# ------------------------------------------------------------------- exact --

def _fft(x, inverse):
    """Unnormalised transform over the last three axes in 64 bits."""
    if inverse:
        return torch.fft.ifftn(x, dim=(-3, -2, -1), norm="forward")
    return torch.fft.fftn(x, dim=(-3, -2, -1))


def _batched_fft(x, inverse):
    out = torch.empty(x.shape, dtype=torch.complex128, device=x.device)
    for j in range(x.shape[0]):
        out[j] = _fft(x[j].to(torch.complex128), inverse)
    return out


def _as_stored(c, precision):
    """complex64 rows as the scaled 16-bit format holds them: one power of two a row, 16-bit parts."""
    parts = torch.view_as_real(c).double()
    m = parts.abs().amax(dim=(-2, -1), keepdim=True)
    e = torch.where(m > 0, torch.frexp(m).exponent - 1 - 14, torch.zeros_like(m, dtype=torch.int32))
    scale = torch.exp2(e.clamp(-128, 127).double())
    half = torch.float16 if precision == "fp16" else torch.bfloat16
    return torch.view_as_complex((parts / scale).float().to(half).double() * scale)


def exact(case, seed):
    kind = case["kind"]
    if kind == "many":
        return [_batched_fft(_coefficients(n, n, n, b, seed + 10 * k), True)
                for k, (n, b) in enumerate(_groups(case))]
    if kind == "scaled":
        n, b = case["n"], case["batch"]
        return _as_stored(_coefficients(n, n, n, b, seed), case["precision"]) * float(n) ** 3
    nx, ny, nz, b = (case[k] for k in ("nx", "ny", "nz", "batch"))
    v = float(nx * ny * nz)
    if kind in ("functions", "plan"):
        c = _grid_input(case, seed)
        return {"psi": _batched_fft(c, True), "back": c.to(torch.complex128) * v}
    if kind == "real":
        return _density(nx, ny, nz, b, seed).double() * v
    c = _coefficients(nx, ny, nz, b, seed)
    if kind == "density":
        rho = torch.zeros((nz, ny, nx), dtype=torch.float64, device="cuda")
        for f, orbital in zip(_occupations(b, seed).double(), c):
            psi = _fft(orbital.to(torch.complex128), True)
            rho += f * (psi.real ** 2 + psi.imag ** 2)
        return rho
    V = _potential(nx, ny, nz, seed).double()
    keep = (_g2(nx, ny, nz) < _cutoff(nx, ny, nz)) if kind == "hpsi" else None
    E = torch.zeros((), dtype=torch.float64, device="cuda")
    rows = []
    for orbital in c.detach():
        psi = _fft(orbital.to(torch.complex128), True)
        E = E + (V * (psi.real ** 2 + psi.imag ** 2)).sum()
        h = _fft(V * psi, False)
        rows.append(h[keep] if kind == "hpsi" else 2 * h)
    out = torch.stack(rows)
    return {"hpsi": out, "E": E} if kind == "hpsi" else {"E": E, "grad": out}
