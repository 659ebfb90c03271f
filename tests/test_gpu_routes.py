"""The kernels that the edge tests are named for are the ones their shapes take.

The plan chooses kernels by estimated time, so a change of an estimate could leave a
test green on another kernel.  The profiler's names of what a call launches are
compared with what each test claims of its shapes.
"""
import re

import numpy as np
import pytest

import test_gpu_backprojection as back
import test_gpu_band_projection as band
import test_gpu_split as split

pytestmark = pytest.mark.gpu


def _kernels(call):
    """Names of the library's kernels that call() launches, template arguments included."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "mpi3d" in e.name]
    if not names:
        pytest.skip("the profiler recorded no kernels")
    return [re.sub(r"\(anonymous namespace\)::|mpi3d::|^void ", "", n).split("(")[0] for n in names]


@pytest.mark.parametrize("name", list(band.SHAPES))
def test_band_projection_shapes(name):
    import torch
    from paper_2511_06627_amd.plan import Plan
    nx, ny, nz, M = band.SHAPES[name]
    theta, q = np.random.default_rng(3).uniform(-np.pi, 2 * np.pi, M), np.pi / 4     # that test's angles
    theta[:16] = [0.0, q, 2 * q, 3 * q, 4 * q, -q, 6 * q, 7 * q, 1e-9, 2 * q + 1e-7, 3e-4, 2 * q - 2e-4, 4 * q + 1e-5,
                  q + 1e-7, q - 1e-7, 6 * q + 9e-4]
    plan = Plan(nx, ny, nz, M, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 4, 1, 1.0, theta=theta)
    x = torch.zeros(plan.shape, device="cuda")
    assert any("proj_fwd_band_kernel" in k for k in _kernels(lambda: plan.project(x)))


@pytest.mark.parametrize("shape", [(211, 230, 13, 60), (256, 209, 34, 33)])
def test_band_projection_bf16_shapes(shape):
    import torch
    from paper_2511_06627_amd.plan import Plan
    plan = Plan(*shape, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 4, 1, 1.0, precisions=("fp32", "mixed"))
    x = torch.zeros(plan.shape, device="cuda")
    assert any("proj_fwd_band_kernel" in k for k in _kernels(lambda: plan.forward(x, precision="mixed")))


def test_backprojection_shapes_take_every_group():
    import torch
    groups = set()
    for nx, ny, nz, M in back.SHAPES + [(nx, ny, 4, M) for nx, ny, _, M in back.SHAPES]:
        plan = back._plan(nx, ny, nz, M)
        rho = torch.zeros(plan.proj_shape, device="cuda")
        for k in _kernels(lambda: plan.backproject(rho)):
            groups |= {int(g) for g in re.findall(r"proj_adj_kernel<(\d+)>", k)}
    print("slices a block:", sorted(groups), flush=True)
    assert groups == {4, 8, 16, 24, 32, 64}


def test_dense_split_shapes():
    import torch
    from paper_2511_06627_amd.plan import Plan
    mark = [m for m in split.test_dense_split_stages.pytestmark if m.name == "parametrize" and "nx" in m.args[0]][0]
    seen = set()
    for nx, nz, M, T, hi, hb in mark.args[1]:
        for sweep in (0.0, nx / 2.0):
            plan = Plan(nx, 12, nz, M, T, T / 128 + 1 / 3, 2.0, 1, hi, hb, 1.0, raster_sweep=sweep)
            rho = torch.zeros(plan.lines_shape, device="cuda")
            y = torch.zeros(plan.data_shape, dtype=torch.complex64, device="cuda")
            names = _kernels(lambda: (plan.signal_fwd(rho), plan.signal_adj(y)))
            assert sum("split_fwd_kernel" in k for k in names) == 1 and sum("split_adj_kernel" in k for k in names) == 1
            seen |= {k for k in names if "split_" in k}
    print("%d kernels of the dense stage on pairs: %s" % (len(seen), sorted(seen)), flush=True)
