"""Edge sizes of the kernels that a dispatch rule chooses between: remainders
of tiles and loops, the smallest and the largest sizes of each rule, against
the FP64 oracle.

Bars: relative L2 <= 5e-6 for FP32 transforms and operators; a sum of
non-negative FP32 products in FP64 to 1e-6 relative.
"""
import numpy as np
import pytest

import oracle
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 5e-6
INVERSE, FORWARD = 1, -1


@pytest.fixture(scope="module")
def F():
    import paper_2006_08435_amd as m
    assert torch.cuda.is_available()
    return m


def rel(a, b):
    a = np.asarray(a, np.complex128).ravel()
    b = np.asarray(b, np.complex128).ravel()
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("b", [1, 1023, 1025, 3073, 4096, 4097, 9001])
def test_sum_of_partials(F, b):
    """One partial per 8 x 8 x 1 grid: every remainder of the sum's loops."""
    c = workloads.uniform_grid((8, 8, 1), 100 + b, batch=b)
    V = (workloads.uniform_grid((8, 8, 1), 99).real + 2.0).astype(np.float32)
    E = F.energy(torch.from_numpy(c).cuda(), torch.from_numpy(V).cuda()).item()
    psi = np.fft.ifftn(c.astype(np.complex128), axes=(1, 2, 3), norm="forward")
    want = float((V.astype(np.float64) * np.abs(psi) ** 2).sum())
    assert abs(E - want) <= 1e-6 * want


@pytest.mark.parametrize("nz", [1, 2, 3, 15, 16, 18, 20, 75, 81, 100, 108, 120, 125])
@pytest.mark.parametrize("cut", [False, True])
def test_operator_lengths(F, nz, cut):
    """The fused z kernel of the operator at one-, two- and three-stage
    lengths, 10 x 10 lines a grid: the last tile of 64 lines is ragged."""
    n, b = 10, 3
    r2 = 2.5 ** 2
    gz = workloads.signed_freq(nz)[:, None, None]
    g = workloads.signed_freq(n)
    inside = (g[None, None, :] ** 2 + g[None, :, None] ** 2 + gz ** 2) < r2
    c = workloads.uniform_grid((n, n, nz), 300 + nz, batch=b)
    if cut:
        c = (c * inside).astype(np.complex64)
    V = (workloads.uniform_grid((n, n, nz), 400 + nz).real + 1.5).astype(np.float32)
    plan = F.Plan(n, n, nz, b, "fp32", INVERSE)
    if cut:
        plan.set_cutoff(r2)
    E = torch.zeros((), dtype=torch.float64, device="cuda")
    scale = torch.tensor(-0.5, dtype=torch.float64, device="cuda")
    out = plan.apply_potential(torch.from_numpy(c).cuda(), torch.from_numpy(V).cuda(), E=E, scale=scale).cpu().numpy()
    want = -0.5 * oracle.apply_potential(c.astype(np.complex128), V.astype(np.float64))
    if cut:
        out, want = out[:, inside], want[:, inside]
    assert rel(out, want) <= TOL
    E_ref, _, _ = oracle.energy(c.astype(np.complex128), V.astype(np.float64), want_grad=False)
    assert abs(E.item() - E_ref) <= 1e-6 * abs(E_ref)


@pytest.mark.parametrize("cut", [False, True])
@pytest.mark.parametrize("n,nz,b", [(15, 3, 9), (16, 3, 9), (18, 3, 1), (18, 3, 2), (18, 3, 11), (30, 4, 9), (50, 2, 1),
                                    (90, 2, 1), (90, 2, 2)])
def test_operator_tile_order(F, n, nz, b, cut):
    """Tiles taken in runs of an XCD: grids of fewer lines than eight runs
    have, one group short of full, exactly one, and several with a rest."""
    r2 = (0.3 * n) ** 2
    g = workloads.signed_freq(n)
    inside = (g[None, None, :] ** 2 + g[None, :, None] ** 2 + workloads.signed_freq(nz)[:, None, None] ** 2) < r2
    c = workloads.uniform_grid((n, n, nz), 500 + n, batch=b)
    if cut:
        c = (c * inside).astype(np.complex64)
    V = (workloads.uniform_grid((n, n, nz), 600 + n).real + 1.5).astype(np.float32)
    plan = F.Plan(n, n, nz, b, "fp32", INVERSE)
    if cut:
        plan.set_cutoff(r2)
    E = torch.zeros((), dtype=torch.float64, device="cuda")
    out = plan.apply_potential(torch.from_numpy(c).cuda(), torch.from_numpy(V).cuda(), E=E).cpu().numpy()
    psi = np.fft.ifftn(c.astype(np.complex128), axes=(1, 2, 3), norm="forward")
    want = np.fft.fftn(V.astype(np.float64) * psi, axes=(1, 2, 3))
    if cut:
        out, want = out[:, inside], want[:, inside]
    for k in range(b):
        assert rel(out[k], want[k]) <= TOL, k
    E_ref = float((V.astype(np.float64) * np.abs(psi) ** 2).sum())
    assert abs(E.item() - E_ref) <= 1e-6 * abs(E_ref)


@pytest.mark.parametrize("n,nz,b", [(15, 2, 146), (18, 2, 100), (18, 2, 101), (18, 2, 103), (25, 3, 60), (50, 2, 14), (90, 2, 5)])
def test_tile_order(F, n, nz, b):
    """The z passes' tiles in runs of an XCD, launches of just under and over
    the 512 tiles from which they are taken, whole groups and rests: the plain
    and the energy form."""
    c = workloads.uniform_grid((n, n, nz), 700 + n, batch=b)
    V = (workloads.uniform_grid((n, n, nz), 800 + n).real + 1.5).astype(np.float32)
    psi = np.fft.ifftn(c.astype(np.complex128), axes=(1, 2, 3), norm="forward")
    x, v = torch.from_numpy(c).cuda(), torch.from_numpy(V).cuda()
    want = float((V.astype(np.float64) * np.abs(psi) ** 2).sum())
    out = F.ifftn(x).cpu().numpy()
    E, psi_e = F.energy_and_psi(x, v)
    psi_e = psi_e.cpu().numpy()
    for k in range(b):
        assert rel(out[k], psi[k]) <= TOL, k
        assert rel(psi_e[k], psi[k]) <= TOL, k
    assert abs(E.item() - want) <= 1e-6 * want
    assert abs(F.energy(x, v).item() - want) <= 1e-6 * want
    plan = F.Plan(n, n, nz, b, "fp32", INVERSE)
    op = plan.apply_potential(x, v, E=torch.zeros((), dtype=torch.float64, device="cuda")).cpu().numpy()
    want = np.fft.fftn(V.astype(np.float64) * psi, axes=(1, 2, 3))
    for k in range(b):
        assert rel(op[k], want[k]) <= TOL, k


@pytest.mark.parametrize("n,nz,b,r2", [(1, 1, 3, 1.0), (2, 3, 2, 0.5), (3, 2, 5, 1e9), (8, 8, 300, 4.0), (15, 4, 2, 14.0),
                                       (16, 5, 3, 1e9), (90, 3, 2, 0.1), (90, 2, 2, 506.25), (125, 2, 1, 3844.0)])
def test_sphere_copies(F, n, nz, b, r2):
    """Spheres from the origin alone to every point, odd and even rows, planes
    of less than a wave: data movement, so bit for bit."""
    gz = workloads.signed_freq(nz)[:, None, None]
    g = workloads.signed_freq(n)
    inside = (g[None, None, :] ** 2 + g[None, :, None] ** 2 + gz ** 2) < r2
    x = workloads.uniform_grid((n, n, nz), 500 + n, batch=b)
    plan = F.Plan(n, n, nz, b, "fp32", INVERSE)
    plan.set_cutoff(r2)
    packed = plan.pack(torch.from_numpy(x).cuda())
    assert np.array_equal(packed.cpu().numpy().view(np.uint64), x[:, inside].view(np.uint64))
    dense = torch.full((b, nz, n, n), complex("nan"), dtype=torch.complex64, device="cuda")
    got = plan.unpack(packed, dense).cpu().numpy()
    want = np.where(inside[None], x, np.complex64(0))
    assert np.array_equal(got.view(np.uint64), want.view(np.uint64))


@pytest.mark.parametrize("n,nz,b", [(2, 1, 1), (9, 16, 3), (25, 20, 3), (30, 75, 2), (45, 64, 2), (96, 12, 3), (128, 9, 3)])
@pytest.mark.parametrize("direction", [INVERSE, FORWARD])
def test_energy_with_half_gradient(F, n, nz, b, direction):
    """E bit for bit as the form that stores psi, the gradient against the
    oracle, out of place and with every buffer the same."""
    lib = F._lib.lib()
    c = workloads.uniform_grid((n, n, nz), 600 + n, batch=b)
    V = (workloads.uniform_grid((n, n, nz), 700 + nz).real + 1.5).astype(np.float32)
    plan = F.Plan(n, n, nz, b, "fp32", direction)
    ct, Vt = torch.from_numpy(c).cuda(), torch.from_numpy(V).cuda()
    E = torch.zeros(2, dtype=torch.float64, device="cuda")
    gE = torch.tensor(-0.75, dtype=torch.float64, device="cuda")
    half, grad = torch.empty_like(ct), torch.empty_like(ct)
    s = torch.cuda.current_stream().cuda_stream
    assert lib.fft3d_energy_fwd(plan.handle, ct.data_ptr(), Vt.data_ptr(), half.data_ptr(), E[0:].data_ptr(), s) == 0
    assert lib.fft3d_energy_vpsi_fwd(plan.handle, ct.data_ptr(), Vt.data_ptr(), half.data_ptr(), E[1:].data_ptr(),
                                     s) == 0
    assert lib.fft3d_energy_vpsi_bwd(plan.handle, half.data_ptr(), gE.data_ptr(), grad.data_ptr(), s) == 0
    assert torch.equal(ct.cpu(), torch.from_numpy(c))
    same = ct.clone()
    assert lib.fft3d_energy_vpsi_fwd(plan.handle, same.data_ptr(), Vt.data_ptr(), same.data_ptr(), E[1:].data_ptr(),
                                     s) == 0
    assert lib.fft3d_energy_vpsi_bwd(plan.handle, same.data_ptr(), gE.data_ptr(), same.data_ptr(), s) == 0
    assert E[0].item() == E[1].item()
    _, _, want = oracle.energy(c.astype(np.complex128), V.astype(np.float64))
    assert rel(grad.cpu().numpy(), -0.75 * want) <= TOL
    assert torch.equal(same, grad)
    assert lib.fft3d_energy_vpsi_fwd(plan.handle, ct.data_ptr() + 8, Vt.data_ptr(), half.data_ptr(), E.data_ptr(),
                                     s) == -6
    assert lib.fft3d_energy_vpsi_bwd(plan.handle, half.data_ptr(), None, grad.data_ptr(), s) == -1


@pytest.mark.parametrize("groups,mode", [
    ([(24, 1), (50, 1)], "mode=grouped"),                                              # too little for one launch
    ([(24, 2), (30, 1), (32, 1), (40, 1), (48, 1), (60, 1)], "mode=persistent"),       # six small groups
    ([(64, 200), (24, 1), (30, 1), (36, 1), (48, 1), (50, 1)], "mode=hybrid grouped=64^3x200 "),
])
def test_default_schedule_of_a_mixed_batch(F, groups, mode):
    plan = F.PlanMany(groups, FORWARD)
    assert mode in plan.describe() and "default" in plan.describe()
    xs = [workloads.uniform_grid(n, 800 + n, batch=b) for n, b in groups]
    outs = plan.exec([torch.from_numpy(x).cuda() for x in xs])
    for (n, b), x, y in zip(groups, xs, outs):
        for j in {0, b - 1}:
            assert rel(y[j].cpu().numpy(), oracle.fft3d(x[j].astype(np.complex128), FORWARD)) <= TOL
    assert F._lib.lib().fft3d_plan_check(plan.handle) == 0


@pytest.mark.parametrize("rows,C", [(1, 1), (7, 2), (5, 3), (4097, 4), (3, 6), (69, 30), (17, 128), (1025, 16), (2, 4096),
                                    (3, 5002), (1, 4099)])
@pytest.mark.parametrize("precision", ["fp16", "bf16"])
def test_dequantize_rows(F, rows, C, precision):
    """Every value is payload * 2^exponent, bit for bit: pairs and single
    points, ragged last workgroups, rows longer than a workgroup's share."""
    rng = np.random.default_rng(900 + rows + C)
    x = workloads.uniform_grid((C, rows, 1), 900 + rows + C)[0] * np.exp2(rng.integers(-40, 40, (rows, 1)))
    buf = F.quantize(torch.from_numpy(x.astype(np.complex64)).cuda(), precision)
    got = F.dequantize(buf, (rows, C), precision).cpu().numpy()
    raw = buf.cpu()
    pay = raw[:4 * rows * C].view(torch.float16 if precision == "fp16" else torch.bfloat16).double().numpy()
    exp = raw[4 * rows * C:].numpy().view(np.int8).astype(np.float64)
    want = pay.reshape(rows, C, 2) * np.exp2(exp)[:, None, None]
    assert np.array_equal(got.view(np.float32).reshape(rows, C, 2).astype(np.float64), want)


@pytest.mark.parametrize("n,nz,b", [(5, 6, 3), (5, 6, 4), (5, 6, 9), (30, 12, 41), (75, 8, 33), (80, 4, 31), (80, 4, 32),
                                    (90, 3, 50), (128, 2, 40)])
@pytest.mark.parametrize("cut", [False, True])
def test_density_ranges(F, n, nz, b, cut):
    """One orbital range and several, uneven ranges, a ragged last tile of
    lines, work on top of c."""
    r2 = (min(n, nz) / 2.5) ** 2
    gz = workloads.signed_freq(nz)[:, None, None]
    g = workloads.signed_freq(n)
    inside = (g[None, None, :] ** 2 + g[None, :, None] ** 2 + gz ** 2) < r2
    c = workloads.uniform_grid((n, n, nz), 1000 + n, batch=b)
    if cut:
        c = (c * inside).astype(np.complex64)
    occ = np.random.default_rng(b).uniform(0, 2, b).astype(np.float32)
    plan = F.Plan(n, n, nz, b, "fp32", INVERSE)
    if cut:
        plan.set_cutoff(r2)
    ct, ot = torch.from_numpy(c).cuda(), torch.from_numpy(occ).cuda()
    rho = plan.density(ct, ot)
    again = plan.density(ct, ot, work=ct)
    psi = np.fft.ifftn(c.astype(np.complex128), axes=(1, 2, 3), norm="forward")
    want = np.tensordot(occ.astype(np.float64), np.abs(psi) ** 2, axes=1)
    assert rel(rho.cpu().numpy(), want) <= TOL
    assert torch.equal(rho, again)


@pytest.mark.parametrize("n,b", [(8, 511), (8, 512), (9, 513), (15, 512), (16, 600), (18, 2), (20, 1), (24, 7), (24, 8), (25, 63), (25, 64),
                                 (27, 64), (30, 95), (30, 96), (32, 95), (32, 97)])
@pytest.mark.parametrize("sign", [INVERSE, FORWARD])
def test_whole_grid_lines(F, n, b, sign):
    """The whole-grid kernel at every kind of length (one line a thread, waves
    with idle lanes) and on both sides of its batch limits; in place too."""
    x = workloads.uniform_grid(n, 1100 + n, batch=b)
    plan = F.Plan(n, n, n, b, "fp32", sign)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    least = 2 * cus if n <= 16 else 1 if n <= 20 else cus // 32 if n <= 24 else cus // 4 if n <= 27 else cus * 3 // 8
    assert plan.describe().startswith("cube lines" if b >= least else "cube" if n <= 16 else "plane")
    xt = torch.from_numpy(x).cuda()
    y = plan.exec(xt)
    z = xt.clone()
    plan.exec(z, z)
    assert torch.equal(y, z)
    for j in {0, b // 2, b - 1}:
        assert rel(y[j].cpu().numpy(), oracle.fft3d(x[j].astype(np.complex128), sign)) <= TOL


@pytest.mark.parametrize("nx,ny,nz,b", [(15, 16, 2, 3), (8, 25, 3, 2), (100, 2, 1, 5), (2, 100, 3, 2), (32, 32, 135, 1),
                                        (9, 128, 2, 2), (128, 8, 2, 2), (64, 60, 2, 3), (81, 50, 3, 2), (64, 81, 2, 1),
                                        (100, 72, 2, 2), (75, 125, 2, 1), (128, 80, 2, 2), (128, 81, 1, 2),
                                        (120, 125, 2, 1), (128, 125, 3, 1), (128, 128, 144, 1), (12, 16, 5, 2), (12, 20, 8, 256), (12, 20, 8, 257)])
@pytest.mark.parametrize("sign", [INVERSE, FORWARD])
def test_rectangular_planes(F, nx, ny, nz, b, sign):
    """Unequal x and y: both sides of every class of plane sizes, odd and even
    rows, one- to three-stage lengths, planes too small for it; in place too."""
    x = workloads.uniform_grid((nx, ny, nz), 1200 + nx + ny, batch=b)
    plan = F.Plan(nx, ny, nz, b, "fp32", sign)
    if nx != ny:
        assert ("k_plane_rect" in plan.describe()) == (nx * ny >= 300 or b * nz <= 2048)
    xt = torch.from_numpy(x).cuda()
    y = plan.exec(xt)
    assert torch.equal(xt.cpu(), torch.from_numpy(x))
    z = xt.clone()
    plan.exec(z, z)
    assert torch.equal(y, z)
    for j in {0, b // 2, b - 1}:
        assert rel(y[j].cpu().numpy(), oracle.fft3d(x[j].astype(np.complex128), sign)) <= TOL


@pytest.mark.parametrize("n,b", [(135, 1), (144, 2), (150, 1), (160, 1), (162, 1), (180, 1), (192, 1), (200, 1), (216, 1),
                                 (225, 1), (240, 2), (240, 3), (243, 1), (250, 1), (256, 1)])
def test_two_passes_above_128(F, n, b):
    """Every length of the two-pass form (whole and ragged x tiles, one and two
    points a load) and its neighbours without one: out of place, in place, and
    pass by pass."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.view_as_complex(torch.rand((b, n, n, n, 2), generator=gen, device="cuda") - 0.5)
    lib = F._lib.lib()
    s = torch.cuda.current_stream().cuda_stream
    two = n not in (225, 243, 250) and (n != 240 or b > 2)
    for sign in (INVERSE, FORWARD):
        plan = F.Plan(n, n, n, b, "fp32", sign)
        assert ("k_split_plane,k_split_z" in plan.describe()) == two
        y = plan.exec(x)
        z = x.clone()
        plan.exec(z, z)
        p = torch.empty_like(x)
        for k in range(lib.fft3d_plan_passes(plan.handle)):
            src = x if k == 0 else p
            assert lib.fft3d_exec_pass(plan.handle, k, src.data_ptr(), p.data_ptr(), s) == 0
        assert torch.equal(p, y)
        # the last pass from one buffer into another, its input left alone
        assert lib.fft3d_exec_pass(plan.handle, 0, x.data_ptr(), p.data_ptr(), s) == 0
        for k in range(1, lib.fft3d_plan_passes(plan.handle) - 1):
            assert lib.fft3d_exec_pass(plan.handle, k, p.data_ptr(), p.data_ptr(), s) == 0
        mid, last = p.clone(), torch.empty_like(p)
        k = lib.fft3d_plan_passes(plan.handle) - 1
        assert lib.fft3d_exec_pass(plan.handle, k, p.data_ptr(), last.data_ptr(), s) == 0
        assert torch.equal(last, y) and torch.equal(p, mid)
        q = x.clone()
        for k in range(lib.fft3d_plan_passes(plan.handle)):
            assert lib.fft3d_exec_pass(plan.handle, k, q.data_ptr(), q.data_ptr(), s) == 0
        assert torch.equal(q, z)
        for j in range(b):
            want = oracle.fft3d(x[j].cpu().numpy().astype(np.complex128), sign)
            assert rel(y[j].cpu().numpy(), want) <= TOL
            assert rel(z[j].cpu().numpy(), want) <= TOL


@pytest.mark.parametrize("form", ["lines", "rows", "split", "density", "energy", "spheres"])
def test_captured_and_replayed(F, form):
    """The forms above from a HIP graph, replayed with new inputs and eager work
    in between, against the eager call bit for bit."""
    shape, b = {"lines": ((20, 20, 20), 3), "rows": ((100, 72, 5), 2), "split": ((135, 135, 135), 1),
                "density": ((24, 24, 6), 20), "energy": ((30, 30, 6), 3), "spheres": ((18, 18, 6), 2)}[form]
    n = shape[0]
    plan = F.Plan(*shape, b, "fp32", INVERSE)
    if form == "spheres":
        plan.set_cutoff((n / 4) ** 2)
    xs = [torch.from_numpy(workloads.uniform_grid(shape, 1300 + k, batch=b)).cuda() for k in range(3)]
    V = torch.from_numpy(workloads.uniform_grid(shape, 1299).real.copy()).cuda()
    occ = torch.linspace(0.5, 2.0, b, device="cuda")
    x = torch.empty_like(xs[0])
    out, work, E = torch.empty_like(x), torch.empty_like(x), torch.zeros((), dtype=torch.float64, device="cuda")
    rho = torch.empty(V.shape, dtype=torch.float32, device="cuda")
    lib = F._lib.lib()

    def call():
        if form == "density":
            return plan.density(x, occ, rho, work)
        if form == "energy":
            s = torch.cuda.current_stream().cuda_stream
            assert lib.fft3d_energy_vpsi_fwd(plan.handle, x.data_ptr(), V.data_ptr(), work.data_ptr(), E.data_ptr(),
                                             s) == 0
            assert lib.fft3d_energy_vpsi_bwd(plan.handle, work.data_ptr(), E.data_ptr(), out.data_ptr(), s) == 0
            return out
        if form == "spheres":
            return plan.unpack(plan.pack(x, packed), out)
        return plan.exec(x, out)

    packed = torch.empty((b, plan.sphere_points), dtype=torch.complex64, device="cuda") if form == "spheres" else None
    want = []
    for v in xs:
        x.copy_(v)
        want.append(call().clone())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        got = call()
    for k in (0, 1, 2, 1):
        x.copy_(xs[k])
        got.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want[k]), k


@pytest.mark.parametrize("rows,C", [(1, 4096), (2, 4098), (3, 8192), (2, 8194), (600, 500), (700, 770), (1, 400002), (1, 1 << 20)])
@pytest.mark.parametrize("precision", ["fp16", "bf16"])
def test_dequantize_long_rows(F, rows, C, precision):
    """Whole and part workgroups of 256, 512, 1024 and 2048 pairs, rows shorter and
    longer than those: payload * 2^exponent, bit for bit."""
    rng = np.random.default_rng(1400 + rows + C)
    x = workloads.uniform_grid((C, rows, 1), 1400 + rows)[0] * np.exp2(rng.integers(-40, 40, (rows, 1)))
    buf = F.quantize(torch.from_numpy(x.astype(np.complex64)).cuda(), precision)
    got = F.dequantize(buf, (rows, C), precision).cpu().numpy()
    raw = buf.cpu()
    pay = raw[:4 * rows * C].view(torch.float16 if precision == "fp16" else torch.bfloat16).double().numpy()
    exp = raw[4 * rows * C:].numpy().view(np.int8).astype(np.float64)
    want = pay.reshape(rows, C, 2) * np.exp2(exp)[:, None, None]
    assert np.array_equal(got.view(np.float32).reshape(rows, C, 2).astype(np.float64), want)


def test_dequantize_time_does_not_depend_on_the_row_length(F):
    """2^22 points as one row and as rows of 128: the same bytes, so a few
    times as long at most (one workgroup alone would take a hundred times)."""
    def best(rows, C):
        buf = torch.zeros(F.scaled16_bytes((rows, C)), dtype=torch.uint8, device="cuda")
        times = []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                F.dequantize(buf, (rows, C))
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)
    assert best(1, 1 << 22) < 5 * best(1 << 15, 128)


@pytest.mark.parametrize("n,b", [(135, 2), (144, 1), (150, 1), (160, 1), (162, 1), (180, 1), (192, 1), (200, 1), (216, 1),
                                 (240, 3), (256, 1)])
@pytest.mark.parametrize("sign", [INVERSE, FORWARD])
def test_in_place_above_128(F, n, b, sign):
    """In place a plan of the two-pass form takes three passes of other
    kernels with the same butterflies: the same bits."""
    gen = torch.Generator(device="cuda").manual_seed(n + 1)
    x = torch.view_as_complex(torch.rand((b, n, n, n, 2), generator=gen, device="cuda") - 0.5)
    plan = F.Plan(n, n, n, b, "fp32", sign)
    assert "k_split_plane,k_split_z" in plan.describe()
    y = plan.exec(x)
    plan.exec(x, x)
    assert torch.equal(x, y)


def run_of(lines, es, tiles, with_V):
    """Tiles of an XCD's run by the rule of the strided passes of 64 lines; 0: launch order."""
    gains = es % 16 != 0 or (with_V and lines % 512 != 0)
    return (lines + 256) // 512 if gains and tiles >= 512 and lines >= 256 else 0


# whole groups of eight runs and a rest, rests of a few tiles and of most of a group
RUNS = [(30, 3, 40), (50, 2, 14), (90, 2, 5), (90, 3, 13)]


def run_case(n, nz, b, cut, with_V):
    tiles = (n * n * b + 63) // 64
    run = run_of(n * n, n * n, tiles, with_V)
    assert run >= 2 and tiles > 8 * run and tiles % (8 * run)     # permuted, and a part that is not
    r2 = (0.3 * n) ** 2
    g = workloads.signed_freq(n)
    inside = (g[None, None, :] ** 2 + g[None, :, None] ** 2 + workloads.signed_freq(nz)[:, None, None] ** 2) < r2
    c = workloads.uniform_grid((n, n, nz), 1500 + n, batch=b)
    V = (workloads.uniform_grid((n, n, nz), 1600 + n).real + 1.5).astype(np.float32)
    return r2, inside, (c * inside).astype(np.complex64) if cut else c, V


@pytest.mark.parametrize("n,nz,b,cut", [c + (cut,) for c in RUNS for cut in (False, True)] + [(72, 2, 7, False)])
def test_operator_in_runs_of_tiles(F, n, nz, b, cut):
    """The operator's z pass and the energies with tiles dealt in runs of two
    or more (72 points: rows of whole cache lines, only V gains by it)."""
    r2, inside, c, V = run_case(n, nz, b, cut, not cut)
    plan = F.Plan(n, n, nz, b, "fp32", INVERSE)
    if cut:
        plan.set_cutoff(r2)
    x, v = torch.from_numpy(c).cuda(), torch.from_numpy(V).cuda()
    E = torch.zeros((), dtype=torch.float64, device="cuda")
    out = plan.apply_potential(x, v, E=E).cpu().numpy()
    psi = np.fft.ifftn(c.astype(np.complex128), axes=(1, 2, 3), norm="forward")
    want = np.fft.fftn(V.astype(np.float64) * psi, axes=(1, 2, 3))
    if cut:
        out, want = out[:, inside], want[:, inside]
    for k in range(b):
        assert rel(out[k], want[k]) <= TOL, k
    E_ref = float((V.astype(np.float64) * np.abs(psi) ** 2).sum())
    assert abs(E.item() - E_ref) <= 1e-6 * E_ref
    if not cut:
        E2, psi2 = F.energy_and_psi(x, v)
        assert abs(E2.item() - E_ref) <= 1e-6 * E_ref and abs(F.energy(x, v).item() - E_ref) <= 1e-6 * E_ref
        for k in range(b):
            assert rel(psi2[k].cpu().numpy(), psi[k]) <= TOL, k


@pytest.mark.parametrize("n,nz,b", RUNS)
def test_transforms_in_runs_of_tiles(F, n, nz, b):
    """The dense and pruned z passes, likewise; the pruned forward ones, which
    keep launch order, with them."""
    r2, inside, c, _ = run_case(n, nz, b, True, False)
    full = workloads.uniform_grid((n, n, nz), 1700 + n, batch=b)
    psi = np.fft.ifftn(c.astype(np.complex128), axes=(1, 2, 3), norm="forward")
    spec = np.fft.fftn(full.astype(np.complex128), axes=(1, 2, 3))
    inv, fwd = F.Plan(n, n, nz, b, "fp32", INVERSE), F.Plan(n, n, nz, b, "fp32", FORWARD)
    x, f = torch.from_numpy(c).cuda(), torch.from_numpy(full).cuda()
    dense = [(inv.exec(x), psi), (fwd.exec(f), spec)]
    inv.set_cutoff(r2)
    fwd.set_cutoff(r2)
    dense.append((inv.exec(x), psi))
    packed = torch.from_numpy(np.ascontiguousarray(c[:, inside])).cuda()
    dense.append((inv.exec_packed(torch.full_like(x, complex("nan")), packed), psi))
    pruned = fwd.exec(f).cpu().numpy()[:, inside]
    got = torch.full((b, fwd.sphere_points), complex("nan"), dtype=torch.complex64, device="cuda")
    fwd.exec_packed(f.clone(), got)
    for y, want in dense + [(torch.from_numpy(pruned), spec[:, inside]), (got, spec[:, inside])]:
        y = y.cpu().numpy()
        for k in range(b):
            assert rel(y[k], want[k]) <= TOL, k


@pytest.mark.parametrize("n,nz,b", [(90, 3, 9), (50, 2, 27)])
def test_real_grids_in_runs_of_tiles(F, n, nz, b):
    """The z pass over half spectra, rows of n / 2 + 1 points."""
    half = n // 2 + 1
    assert run_of(half * n, half * n, (half * n * b + 63) // 64, False) >= 2
    rho = workloads.uniform_grid((n, n, nz), 1800 + n, batch=b).real.astype(np.float32)
    want = np.fft.rfftn(rho.astype(np.float64), axes=(1, 2, 3))
    h = F.rfftn(torch.from_numpy(rho).cuda())
    back = F.irfftn(h, n).cpu().numpy() / (n * n * nz)
    for k in range(b):
        assert rel(h[k].cpu().numpy(), want[k]) <= TOL, k
        assert rel(back[k], rho[k]) <= TOL, k


@pytest.mark.parametrize("n,b", [(10, 512), (10, 515), (12, 513), (12, 600)])
@pytest.mark.parametrize("sign", [INVERSE, FORWARD])
def test_whole_grid_lines_of_10_and_12(F, n, b, sign):
    """The two lengths of the whole-grid kernel whose last wave has idle lanes
    and whose exchanges move whole points; in place too."""
    x = workloads.uniform_grid(n, 1900 + n, batch=b)
    plan = F.Plan(n, n, n, b, "fp32", sign)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert plan.describe().startswith("cube lines") == (b >= 2 * cus)
    xt = torch.from_numpy(x).cuda()
    y = plan.exec(xt)
    plan.exec(xt, xt)
    assert torch.equal(y, xt)
    for j in {0, b // 2, b - 1}:
        assert rel(y[j].cpu().numpy(), oracle.fft3d(x[j].astype(np.complex128), sign)) <= TOL


@pytest.mark.parametrize("shape,text", [
    ((100, 72, 90), "axes plane x=100(10x10) y=72(12x6) threads=1024 lds="),
    ((100, 72, 270), "axes plane x=100(10x10) y=72(12x6) threads=512 lds="),
    ((128, 125, 1), "axes plane x=128(8x16) y=125(5x5x5) threads=1024 lds="),
    ((10, 4, 160), "axes plane x=10(10) y=4(4) threads=128 lds="),
    ((256, 256, 256), "axes split n=256 parts=4 plane(x 16x16, y 8x8, t1024, lds 131584) z(y 4, z 16x16, t1024, lds 133120)"),
    ((135, 135, 135), "axes split n=135 parts=3 plane(x "),
    ((250, 250, 250), "axes x=250("),
])
def test_describe_names_the_kernels_that_run(F, shape, text):
    """Threads, radices and LDS of the plane kernels, not of the 1D passes."""
    d = F.Plan(*shape, 1, "fp32", INVERSE).describe()
    assert d.startswith(text), d
    kernels = d.split("kernels=")[1].split(",")
    assert kernels[0] == ("k_plane_rect" if "plane x=" in d else "k_split_plane" if "split" in d else "k_axis_row")
    if "plane x=" in d:
        assert ("; z=%d(" % shape[2] in d) == (shape[2] > 1) and ("k_axis_str" in kernels) == (shape[2] > 1)


@pytest.mark.parametrize("n,nz,b,r2", [(24, 2, 1, 36.0), (32, 1, 1, 1e9), (125, 3, 1, 900.0), (128, 8, 2, 900.0),
                                       (16, 3, 683, 16.0), (30, 5, 409, 30.0), (30, 5, 410, 30.0), (15, 3, 682, 30.0),
                                       (15, 3, 700, 1e9), (18, 4, 512, 40.0), (25, 3, 700, 60.0)])
def test_unpack_planes_shared_by_workgroups(F, n, nz, b, r2):
    """Few planes (many workgroups each, the last ones with fewer units) to
    more than 2048 (one each): bit for bit."""
    gz = workloads.signed_freq(nz)[:, None, None]
    g = workloads.signed_freq(n)
    inside = (g[None, None, :] ** 2 + g[None, :, None] ** 2 + gz ** 2) < r2
    x = workloads.uniform_grid((n, n, nz), 2200 + n, batch=b)
    plan = F.Plan(n, n, nz, b, "fp32", INVERSE)
    plan.set_cutoff(r2)
    dense = torch.full((b, nz, n, n), complex("nan"), dtype=torch.complex64, device="cuda")
    packed = torch.from_numpy(np.ascontiguousarray(x[:, inside])).cuda()
    got = plan.unpack(packed, dense).cpu().numpy()
    assert np.array_equal(got.view(np.uint64), np.where(inside[None], x, np.complex64(0)).view(np.uint64))
    assert torch.equal(plan.pack(torch.from_numpy(x).cuda()), packed)


def best_replay(call, calls=10):
    """Milliseconds of `calls` calls, the best of several replays of a graph."""
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(calls):
            call()
    times = []
    for _ in range(6):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        graph.replay()
        end.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(end))
    return min(times)


def test_unpack_time_of_few_grids(F):
    """One grid of 125^3 in a fifth of the time of sixteen at most (a workgroup
    a plane takes a third of it)."""
    def best(b):
        plan = F.Plan(125, 125, 125, b, "fp32", INVERSE)
        plan.set_cutoff((125 / 4) ** 2)
        dense = torch.zeros(plan.shape, dtype=torch.complex64, device="cuda")
        packed = plan.pack(dense)
        return best_replay(lambda: plan.unpack(packed, dense))
    assert 5 * best(1) < best(16)


@pytest.mark.parametrize("nx,ny", [(45, 25), (64, 60), (64, 81), (125, 80), (20, 16)])
@pytest.mark.parametrize("planes", [255, 256, 257])
def test_rectangular_planes_of_one_turn(F, nx, ny, planes):
    """Twice the threads up to 256 planes; the same bits on both sides."""
    x = workloads.uniform_grid((nx, ny, 1), 2300 + nx, batch=planes)
    xt = torch.from_numpy(x).cuda()
    plan = F.Plan(nx, ny, 1, planes, "fp32", FORWARD)
    assert "plane x=" in plan.describe()
    y = plan.exec(xt)
    assert torch.equal(y, F.Plan(nx, ny, 1, 600, "fp32", FORWARD).exec(xt.repeat(3, 1, 1, 1)[:600].contiguous())[:planes])
    for j in {0, planes - 1}:
        assert rel(y[j].cpu().numpy(), oracle.fft3d(x[j].astype(np.complex128), FORWARD)) <= TOL
