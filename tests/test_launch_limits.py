"""Batches whose workgroups exceed what one launch may hold (fewer than 2^32
work items in a dimension): every pass still runs, and the grids at both ends
and around the seams hold what a small batch of them gives, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GIB = 1 << 30


@pytest.fixture
def F():
    import paper_2006_08435_amd as m
    yield m
    torch.cuda.empty_cache()


def grids(shape, gib):
    """Zeros of `shape` with a few noisy grids, and those grids' numbers."""
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (gib + 8) * GIB:
        pytest.skip("needs %d GiB of device memory" % gib)
    x = torch.empty(shape, dtype=torch.complex64, device="cuda")
    x.zero_()
    b = shape[0]
    seams = {0, 1, b - 1}
    for k in range(1, 9):
        seams |= {b * k // 8 - 1, b * k // 8}
    for seam in (1 << 21, 1 << 22, 1 << 23):
        seams |= {v for v in (seam - 1, seam, seam + 1, b - seam - 1, b - seam) if 0 <= v < b}
    at = sorted(v for v in seams if v < b)
    gen = torch.Generator(device="cuda").manual_seed(b)
    for k in at:
        x[k] = torch.view_as_complex(torch.rand(shape[1:] + (2,), generator=gen, device="cuda") - 0.5)
    return x, at


def test_rectangular_planes(F):
    """2^24 planes of 32 x 36 points, 256 threads each: 2^32 work items."""
    b = 1 << 24
    x, at = grids((b, 1, 36, 32), 144)
    few = torch.stack([x[k] for k in at])
    plan = F.Plan(32, 36, 1, b, "fp32", 1)
    assert "k_plane_rect" in plan.describe()
    plan.exec(x, x)
    want = F.Plan(32, 36, 1, len(at), "fp32", 1).exec(few)
    for j, k in enumerate(at):
        assert torch.equal(x[k], want[j]), k


def test_columns_of_the_two_pass_form(F):
    """The first pass above 128 points alone and in place: nine workgroups of
    1024 threads a plane."""
    n, b = 135, 3460
    x, at = grids((b, n, n, n), 64)
    few = torch.stack([x[k] for k in at])
    lib, s = F._lib.lib(), torch.cuda.current_stream().cuda_stream
    plan, small = F.Plan(n, n, n, b, "fp32", 1), F.Plan(n, n, n, len(at), "fp32", 1)
    assert "k_split_plane" in plan.describe()
    assert lib.fft3d_exec_pass(plan.handle, 0, x.data_ptr(), x.data_ptr(), s) == 0
    assert lib.fft3d_exec_pass(small.handle, 0, few.data_ptr(), few.data_ptr(), s) == 0
    for j, k in enumerate(at):
        assert torch.equal(x[k], few[j]), k


@pytest.mark.parametrize("n,b", [(128, 8200), (50, 53700)])
def test_strided_tiles(F, n, b):
    """More than 2^21 tiles of z lines: the plain pass, the energy and the
    operator, with tiles in launch order (128) and in runs (50)."""
    x, at = grids((b, 2, n, n), 3)
    few = torch.stack([x[k] for k in at])
    V = torch.rand((2, n, n), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    plan, small = F.Plan(n, n, 2, b, "fp32", 1), F.Plan(n, n, 2, len(at), "fp32", 1)
    zero = torch.zeros((), dtype=torch.float64, device="cuda")
    E, E_few = zero.clone(), zero.clone()
    for call in (lambda p, v, e: p.exec(v), lambda p, v, e: p.apply_potential(v, V, E=e)):
        y, want = call(plan, x, E), call(small, few, E_few)
        for j, k in enumerate(at):
            assert torch.equal(y[k], want[j]), k
        assert y.count_nonzero() == want.count_nonzero()
        del y
    assert E.item() == pytest.approx(E_few.item(), rel=1e-12)
    assert F.energy(x, V).item() == pytest.approx(E_few.item(), rel=1e-12)


@pytest.mark.parametrize("n", [1, 2])
def test_whole_grids(F, n):
    """2^26 grids and a few of one workgroup each."""
    b = (1 << 26) + 5
    x, at = grids((b, n, n, n), 5)
    few = torch.stack([x[k] for k in at])
    F.Plan(n, n, n, b, "fp32", -1).exec(x, x)
    want = F.Plan(n, n, n, len(at), "fp32", -1).exec(few)
    for j, k in enumerate(at):
        assert torch.equal(x[k], want[j]), k


def test_rows(F):
    """2^26 tiles of 16 short rows and a few."""
    b = 360000000
    x, at = grids((b, 1, 3, 2), 17)
    few = torch.stack([x[k] for k in at])
    plan = F.Plan(2, 3, 1, b, "fp32", -1)
    assert "k_axis_row" in plan.describe()
    plan.exec(x, x)
    want = F.Plan(2, 3, 1, len(at), "fp32", -1).exec(few)
    for j, k in enumerate(at):
        assert torch.equal(x[k], want[j]), k


@pytest.mark.parametrize("rows,C", [((1 << 32) + 777, 1), ((1 << 26) + 9, 4)])
@pytest.mark.parametrize("precision", ["fp16", "bf16"])
def test_scaled_rows(F, rows, C, precision):
    """Conversion to 16 bits and back of more rows than a launch has waves."""
    x, at = grids((rows, C), 100 if C == 1 else 8)
    few = torch.stack([x[k] for k in at])
    buf = F.quantize(x, precision)
    del x
    back = F.dequantize(buf, (rows, C), precision)
    want = F.dequantize(F.quantize(few, precision), few.shape, precision)
    for j, k in enumerate(at):
        assert torch.equal(back[k], want[j]), k
