"""Oblong volumes keep the one- and two-slice projection kernels where those are faster.

At 216 x 327 x 82, 10 angles, the four-slice kernel takes 78 us and the kernel of
one slice a texel 69.
"""
import pytest

from test_gpu_routes import _kernels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,mixed,taken", [((216, 327, 82, 10), False, False), ((205, 321, 32, 31), False, False),
                                              ((192, 192, 96, 36), False, True), ((192, 282, 11, 93), True, False),
                                              ((256, 256, 64, 24), True, True)])
def test_four_slice_kernel_where_it_is_faster(dims, mixed, taken):
    import torch
    from paper_2511_06627_amd.plan import Plan
    plan = Plan(*dims, 1024, 8.0, 3.0, 1, 4, 0, 1e-3, precisions=("fp32", "mixed"))
    x = torch.zeros(plan.shape, device="cuda")
    names = _kernels(lambda: plan.forward(x, precision="mixed") if mixed else plan.project(x))
    assert any("proj_fwd_band_kernel" in k for k in names) == taken
