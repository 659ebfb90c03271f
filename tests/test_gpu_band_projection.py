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


@pytest.mark.parametrize("shape", [(211, 230, 13, 60), (256, 209, 34, 33)])
def test_band_projection_bf16(shape):
    """The mixed operator's gathers in large volumes: the volume rounded to bf16 on the way, the fp32 kernel's sums."""
    import torch
    from paper_2511_06627_amd.plan import Plan
    nx, ny, nz, M = shape
    plan = Plan(nx, ny, nz, M, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 4, 1, 1.0, precisions=("fp32", "mixed"))
    x = torch.rand(plan.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(6))
    x16 = x.to(torch.bfloat16).float()
    got = plan.forward(x, precision="mixed")
    assert torch.equal(got, plan.forward(x16, precision="mixed"))
    # the fp32 projections of the same values (their sums perhaps in another
    # order, 1e-6 apart): of the signal stage's fp16 operands (a unit is 2^-11
    # to 2^-10 of a value) some 0.4% round the other way, 2^-10 sqrt(0.004) = 6e-5
    want = plan.signal_fwd(plan.project(x16), precision="mixed")
    assert float((got - want).norm() / want.norm()) <= 1e-4
    # a solver's iterations gather from a bf16 copy of their own: one CGLS step
    # along p = A^H b is alpha p, alpha = |p|^2 / (|A p|^2 + lam |p|^2)
    b = plan.forward(x)
    got, _ = plan.solve(b, 1e-3, precision="mixed", refine_sweeps=1, inner_iters=1)
    p = plan.adjoint(b, precision="mixed")
    if not torch.isfinite(p).all() or float((got.double() * p.double()).sum()) == 0.0:
        raise AssertionError("empty step")
    q = plan.forward(p, precision="mixed")
    pp = float((p.double() ** 2).sum())
    alpha = pp / (float((q.to(torch.complex128).abs() ** 2).sum()) + 1e-3 * pp)
    # fp32 against mixed first residuals and directions: the mixed operator's own error
    rel = float((got.double() - alpha * p.double()).norm() / (alpha * p.double()).norm())
    print("one mixed step: %.2e" % rel, flush=True)
    assert rel <= 5e-3
