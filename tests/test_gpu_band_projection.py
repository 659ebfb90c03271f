"""The four-slice band projection against the FP64 oracle at its edges.

Odd sizes (bands and slice groups with remainders, unaligned rows), both
angle classes and their border at 45 degrees, rays along the grid axes (exact
and off by less than a sample over the grid) and angles beyond 180 degrees;
enough rays that the plan takes this kernel
(by the estimates of its rule, 1.3 to 2 times faster here).  FP32 tolerance of the other
projection tests.
"""
import numpy as np
import pytest

from oracle import projector
from helpers import oracle_geometry, rel_l2, random_volume

pytestmark = pytest.mark.gpu

TOL32 = 1e-5

# (nx, ny, nz, M)
SHAPES = {"wide": (131, 67, 41, 120), "tall": (70, 190, 13, 640), "square": (192, 192, 93, 40)}


@pytest.mark.parametrize("name", list(SHAPES))
def test_band_projection(name):
    import torch
    from paper_2511_06627_amd.plan import Plan
    nx, ny, nz, M = SHAPES[name]
    rng = np.random.default_rng(3)
    theta = rng.uniform(-np.pi, 2 * np.pi, M)
    q = np.pi / 4
    theta[:16] = [0.0, q, 2 * q, 3 * q, 4 * q, -q, 6 * q, 7 * q, 1e-9, 2 * q + 1e-7, 3e-4, 2 * q - 2e-4, 4 * q + 1e-5,
                  q + 1e-7, q - 1e-7, 6 * q + 9e-4]
    g = oracle_geometry(nx, ny, nz, M, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 4, 1)
    g.theta = theta
    plan = Plan(nx, ny, nz, M, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 4, 1, 1.0, theta=theta)
    x = random_volume(g, 4)
    want = projector.project(g, np.asarray(x, dtype=np.float64))
    got = plan.project(torch.from_numpy(np.ascontiguousarray(x)).float().cuda()).cpu().numpy()
    per = [rel_l2(got[m], want[m]) for m in range(M)]
    print("%s: worst angle %.2e (%.6f rad)" % (name, max(per), theta[int(np.argmax(per))]), flush=True)
    assert max(per) <= TOL32
    # lines are padded with zeros in the operator's workspace: A sees the same projections
    b = plan.forward(torch.from_numpy(np.ascontiguousarray(x)).float().cuda())
    assert torch.equal(b, plan.signal_fwd(torch.from_numpy(got).cuda()))


def test_angles_beyond_half_turn():
    """Rays with sin < 0 through the one- and two-slice kernels (a scan too small for the band kernel)."""
    import torch
    from paper_2511_06627_amd.plan import Plan
    nx, ny, nz, M = 40, 28, 5, 7
    theta = np.array([3.3, 4.0, 4.7124, 5.0, 6.0, -0.4, -2.0])
    g = oracle_geometry(nx, ny, nz, M, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 4, 1)
    g.theta = theta
    plan = Plan(nx, ny, nz, M, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 4, 1, 1.0, theta=theta)
    x = random_volume(g, 5)
    want = projector.project(g, np.asarray(x, dtype=np.float64))
    got = plan.project(torch.from_numpy(np.ascontiguousarray(x)).float().cuda()).cpu().numpy()
    assert rel_l2(got, want) <= TOL32
