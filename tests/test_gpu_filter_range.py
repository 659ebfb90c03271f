"""FP32 signal stages behind a receive filter of wide range (eq. DCmodel's D_Gamma).

Gains that are powers of two scale a bin's results exactly: A with gains D is D
times A without, and A^T b with gains D is the unfiltered A^T of D b, bit for bit,
for gains from 1 down to 2^-100 and 0.  Every form of the FP32 stage: factored at
C = 32 and 64, tensor lines, two line groups, dense on fp16 pairs, dense on fp32
MFMA (a plan that also holds the mixed operator).
"""
import numpy as np
import pytest

from oracle import signal
from helpers import oracle_geometry, random_data

pytestmark = pytest.mark.gpu

# name: (nx, ny, nz, M, T, drive cycles, k_hi, half band), options, C the plan takes
FORMS = {
    "factored32": ((70, 12, 5, 7, 2048, 2048 / 256 + 1 / 3, 15, 2), {}, 32),
    "factored64": ((100, 16, 4, 9, 8192, 64 + 1 / 3, 56, 3), {}, 64),
    "tensor": ((64, 12, 6, 5, 2048, 2048 / 256 + 1 / 3, 15, 2), {"psf_rows": 2}, 32),
    "raster": ((90, 12, 7, 5, 2048, 2048 / 256 + 1 / 3, 15, 2), {"raster_sweep": 45.0}, 32),
    "dual": ((48, 12, 20, 3, 2048, 2048 / 256 + 1 / 3, 15, 2), {"drive_axes": 2}, 32),
    "dense_pairs": ((131, 12, 9, 7, 3001, 3001 / 128 + 1 / 3, 31, 3), {}, 0),
    "dense_pairs_raster": ((64, 12, 9, 7, 2050, 2050 / 128 + 1 / 3, 11, 3), {"raster_sweep": 32.0}, 0),
    "dense_fp32": ((64, 12, 9, 7, 2050, 2050 / 128 + 1 / 3, 11, 3), {"precisions": ("fp32", "mixed")}, 0),
}


def _plan(name, gains):
    from paper_2511_06627_amd.plan import Plan
    (nx, ny, nz, M, T, P, hi, hb), opts, C = FORMS[name]
    plan = Plan(nx, ny, nz, M, T, P, 2.0, 1, hi, hb, 1.0, rx_filter=gains, **opts)
    assert plan.dft_cycles == C, plan.dft_cycles
    return plan


@pytest.mark.parametrize("name", list(FORMS))
def test_power_of_two_gains_are_exact(name):
    import torch
    (nx, ny, nz, M, T, P, hi, hb), _, _ = FORMS[name]
    nb = hi * (2 * hb + 1)
    gains = 2.0 ** -((37 * np.arange(nb)) % 101).astype(np.float64)
    gains[nb // 3] = 0.0
    one, plan = _plan(name, None), _plan(name, gains)
    d = torch.from_numpy(gains).float().cuda()
    rng = np.random.default_rng(3)
    lines = rng.uniform(0, 1, plan.lines_shape).astype(np.float32)
    if "drive_axes" in FORMS[name][1]:
        lines[M * nz:, nz:] = 0.0                    # z-drive lines hold nz values
    rho = torch.from_numpy(lines).cuda()
    got, want = torch.view_as_real(plan.signal_fwd(rho)), torch.view_as_real(one.signal_fwd(rho)) * d[:, None]
    print("%s forward: %d of %d values differ" % (name, int((got != want).sum()), got.numel()), flush=True)
    assert torch.equal(got, want)
    y = torch.from_numpy((rng.standard_normal(plan.data_shape) + 1j * rng.standard_normal(plan.data_shape))
                         .astype(np.complex64)).cuda()
    for k in (0, 50):                                # all bins; only those with gains below 2^-50
        yk = y * (d <= 2.0 ** -k)
        yd = torch.view_as_complex((torch.view_as_real(yk) * d[:, None]).contiguous())
        got, want = plan.signal_adj(yk), one.signal_adj(yd)
        print("%s adjoint: %d of %d values differ" % (name, int((got != want).sum()), got.numel()), flush=True)
        assert torch.isfinite(got).all() and bool(got.abs().max() > 0)
        assert torch.equal(got, want)


@pytest.mark.parametrize("name", ["factored32", "factored64", "dense_pairs"])
def test_bins_behind_weak_gains(name):
    """Complex gains of every size against the oracle, bin by bin.  Only the weights'
    roundings change with the gains, each of the same size beside its weight, so a
    bin's error relative to its own norm stays within four times the unfiltered
    plan's (another draw of the same roundings) and 1e-6."""
    import torch
    (nx, ny, nz, M, T, P, hi, hb), _, _ = FORMS[name]
    nb = hi * (2 * hb + 1)
    rng = np.random.default_rng(4)
    gains = (10.0 ** rng.uniform(-12, 0, nb) * np.exp(2j * np.pi * rng.uniform(0, 1, nb))).astype(np.complex64)
    rho = rng.uniform(0, 1, (M * nz, nx)).astype(np.float32)
    errs = []
    for filt in (None, gains):
        g = oracle_geometry(nx, ny, nz, M, T, P, 2.0, 1, hi, hb, rx_filter=filt)
        plan = _plan(name, filt)
        got = plan.signal_fwd(torch.from_numpy(rho.reshape(plan.lines_shape)).cuda()).cpu().numpy().reshape(M * nz, nb)
        want = signal.forward(g, rho).reshape(M * nz, nb)
        errs.append(np.linalg.norm(got - want, axis=0) / np.linalg.norm(want, axis=0))
    print("%s: worst bin %.2e without, %.2e with gains" % (name, errs[0].max(), errs[1].max()), flush=True)
    assert (errs[1] <= 4 * errs[0] + 1e-6).all()
