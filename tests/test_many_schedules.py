"""Mixed batches in each launch mode by name: calls in place, repeated calls and
plain transforms of the same grids, whatever mode an untuned plan takes."""
import os

import numpy as np
import pytest

import oracle
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 5e-6
MODES = [(1024, 1), (1024, 4), (512, 1), (512, 4), (-1024, 1), (-512, 2), (0, 1)]


@pytest.fixture(scope="module")
def F(tmp_path_factory):
    import paper_2006_08435_amd as m
    os.environ["FFT3D_TUNE_CACHE"] = str(tmp_path_factory.mktemp("tc") / "tune.json")
    return m


def rel(a, b):
    a = np.asarray(a, np.complex128).ravel()
    b = np.asarray(b, np.complex128).ravel()
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def mode_of(threads):
    return "mode=grouped" if threads == 0 else "mode=hybrid" if threads < 0 else "mode=persistent"


@pytest.mark.parametrize("threads,chunk", MODES)
@pytest.mark.parametrize("direction", [-1, 1])
def test_in_place_and_repeated(F, threads, chunk, direction):
    """64^3 x 40 is plain in the hybrid mode, the others share the persistent
    launch; ten calls in place, each on fresh input, leave the same bits."""
    groups = [(64, 40), (48, 3), (100, 1), (30, 5)]
    xs = [workloads.uniform_grid(n, 2000 + n, batch=b) for n, b in groups]
    plan = F.PlanMany(groups, direction)
    plan.set_schedule(threads, chunk)
    assert mode_of(threads) in plan.describe()
    ins = [torch.from_numpy(x).cuda() for x in xs]
    first = [t.clone() for t in plan.exec(ins)]
    for t, x in zip(ins, xs):
        assert torch.equal(t.cpu(), torch.from_numpy(x))
    for r in range(10):
        bufs = [t.clone() for t in ins]
        plan.exec(bufs, bufs)
        for a, b in zip(first, bufs):
            assert torch.equal(a, b), r
    for (n, b), x, y in zip(groups, xs, first):
        for j in {0, b - 1}:
            assert rel(y[j].cpu().numpy(), oracle.fft3d(x[j].astype(np.complex128), direction)) <= TOL, (n, j)
    assert F._lib.lib().fft3d_plan_check(plan.handle) == 0


@pytest.mark.parametrize("threads,chunk", MODES)
def test_plain_transforms_of_the_same_grids(F, threads, chunk):
    groups = [(96, 2), (60, 3), (64, 70)]
    xs = [workloads.uniform_grid(n, 2100 + n, batch=b) for n, b in groups]
    plan = F.PlanMany(groups, 1)
    plan.set_schedule(threads, chunk)
    assert mode_of(threads) in plan.describe()
    got = plan.exec([torch.from_numpy(x).cuda() for x in xs])
    for (n, b), x, y in zip(groups, xs, got):
        for j in {0, b // 2, b - 1}:
            plain = F.ifftn(torch.from_numpy(x[j]).cuda())
            assert rel(y[j].cpu().numpy(), plain.cpu().numpy()) <= 1e-6, (n, j)
    assert F._lib.lib().fft3d_plan_check(plan.handle) == 0
