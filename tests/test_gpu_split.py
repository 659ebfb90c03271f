"""The factored FP32 signal stage's fp16-pair products (hi + lo) at their edges.

Stage entries against the FP64 oracle's dense definition: every residue of C =
32 present (the slot shared by residues 0 and C / 2, conjugate pairs), C = 64
with 20 and 24 slots, all padded widths, odd line strides, a ragged last line
tile, phase counts that no stage divides.  Tolerance: a pair holds a number to
2^-23, so a product of two pairs without lo lo is within 2^-22 + 2 2^-23 of
exact; three such contractions in a row and their fp32 sums stay below
8 x 2^-22 = 1.9e-6 of a line's norm.
"""
import numpy as np
import pytest

from oracle import signal
from helpers import oracle_geometry, random_data

pytestmark = pytest.mark.gpu

TOL = 1.9e-6

# name: (nx, ny, nz, M, T, drive cycles, w, k_lo, k_hi, half band, C the plan takes)
CASES = {
    "all_residues_u150": (150, 20, 5, 7, 6144, 6144 / 256 + 1 / 3, 3.0, 1, 20, 3, 32),
    "slots20_u256": (256, 16, 3, 11, 8192, 64 + 1 / 3, 3.0, 1, 47, 3, 64),
    "slots24_u100": (100, 16, 4, 9, 8192, 64 + 1 / 3, 3.0, 1, 56, 3, 64),
    "p63_u33": (33, 24, 8, 9, 2016, 2016 / 256 + 1 / 3, 2.0, 1, 15, 2, 32),
    "one_line": (64, 16, 1, 1, 4096, 4096 / 256 + 1 / 3, 2.0, 1, 31, 3, 32),
}


def _plan(name):
    from paper_2511_06627_amd.plan import Plan
    nx, ny, nz, M, T, P, w, klo, khi, D, C = CASES[name]
    g = oracle_geometry(nx, ny, nz, M, T, P, w, klo, khi, D)
    plan = Plan(nx, ny, nz, M, T, P, w, klo, khi, D, 1.0)
    assert plan.dft_cycles == C, "plan took C = %d" % plan.dft_cycles
    return g, plan


def _line_errors(a, b):
    a, b = np.asarray(a), np.asarray(b)
    a, b = a.reshape(-1, a.shape[-1]), b.reshape(-1, b.shape[-1])
    return np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)


@pytest.mark.parametrize("name", list(CASES))
def test_stages_per_line(name):
    """Each line on its own, lines scaled apart by powers of two."""
    import torch
    g, plan = _plan(name)
    rng = np.random.default_rng(5)
    L = g.n_lines
    sc = 2.0 ** rng.integers(-80, 81, L)
    rho = (rng.uniform(0, 1, (L, g.n_u)) ** 3).astype(np.float32)
    want = signal.forward(g, rho) * sc[:, None]
    x = torch.from_numpy((rho * sc[:, None]).astype(np.float32).reshape(plan.lines_shape)).cuda()
    ef = _line_errors(plan.signal_fwd(x).cpu().numpy(), want.reshape(plan.data_shape))
    y = np.asarray(random_data(g, 6)).reshape(L, -1).astype(np.complex64)
    want = signal.adjoint(g, y) * sc[:, None]
    b = torch.from_numpy((y * sc[:, None]).astype(np.complex64).reshape(plan.data_shape)).cuda()
    ea = _line_errors(plan.signal_adj(b).cpu().numpy(), want.reshape(plan.lines_shape))
    print("%s: forward %.2e adjoint %.2e" % (name, ef.max(), ea.max()), flush=True)
    assert ef.max() <= TOL and ea.max() <= TOL


def test_non_finite_line_stays_alone():
    """A line with an infinity or a NaN gives non-finite results and leaves every other line's bits."""
    import torch
    g, plan = _plan("p63_u33")
    rng = np.random.default_rng(7)
    rho = torch.from_numpy(rng.uniform(0, 1, plan.lines_shape).astype(np.float32)).cuda()
    ref = plan.signal_fwd(rho).cpu()
    y = torch.from_numpy(np.asarray(random_data(g, 8)).astype(np.complex64).reshape(plan.data_shape)).cuda()
    refa = plan.signal_adj(y).cpu()
    keep = torch.ones(ref.shape[:2], dtype=torch.bool)
    keep[2, 3] = keep[5, 0] = False
    rho[2, 3, 10], rho[5, 0, 4] = float("inf"), float("nan")
    y[2, 3, 10], y[5, 0, 4] = float("inf"), float("nan")
    got, gota = plan.signal_fwd(rho).cpu(), plan.signal_adj(y).cpu()
    assert torch.equal(torch.view_as_real(got[keep]), torch.view_as_real(ref[keep])) and torch.equal(gota[keep], refa[keep])
    assert not torch.isfinite(torch.view_as_real(got[~keep])).any() and not torch.isfinite(gota[~keep]).any()


@pytest.mark.parametrize("nu,rows", [(33, 1), (33, 2), (64, 3), (100, 1), (128, 2), (70, 3), (150, 1), (192, 2), (180, 3),
                                     (256, 1), (200, 2)])
def test_tensor_lines(nu, rows):
    """The forward's virtual lines of 2 to 4 symmetric sums, the adjoint's tables of their own."""
    import torch
    from paper_2511_06627_amd.plan import Plan
    nz, M, T = 6, 7, 2048
    args = (nu, 12, nz, M, T, T / 256 + 1 / 3, 2.0, 1, 15, 2)
    g = oracle_geometry(*args)
    g.psf_rows = rows
    plan = Plan(*args, 1.0, psf_rows=rows)
    assert plan.dft_cycles == 32
    rng = np.random.default_rng(9)
    rho = rng.uniform(0, 1, (g.n_lines, nu)).astype(np.float32)
    got = plan.signal_fwd(torch.from_numpy(rho.reshape(plan.lines_shape)).cuda()).cpu().numpy()
    ef = _line_errors(got, signal.forward(g, rho).reshape(plan.data_shape)).max()
    y = np.asarray(random_data(g, 10)).reshape(g.n_lines, -1).astype(np.complex64)
    got = plan.signal_adj(torch.from_numpy(y.reshape(plan.data_shape)).cuda()).cpu().numpy()
    ea = _line_errors(got, signal.adjoint(g, y).reshape(plan.lines_shape)).max()
    print("n_u %d R %d: forward %.2e adjoint %.2e" % (nu, rows, ef, ea), flush=True)
    assert ef <= TOL and ea <= TOL


def test_two_line_groups():
    """A raster's two classes, each with its own tables: classes of unequal size, ragged tiles."""
    import torch
    from paper_2511_06627_amd.plan import Plan
    args = (90, 12, 7, 9, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 15, 2)
    g = oracle_geometry(*args)
    g.raster_sweep = 45.0
    plan = Plan(*args, 1.0, raster_sweep=45.0)
    assert plan.dft_cycles == 32
    rng = np.random.default_rng(11)
    rho = rng.uniform(0, 1, (g.n_lines, g.n_u)).astype(np.float32)
    got = plan.signal_fwd(torch.from_numpy(rho.reshape(plan.lines_shape)).cuda()).cpu().numpy()
    assert _line_errors(got, signal.forward(g, rho).reshape(plan.data_shape)).max() <= TOL
    y = np.asarray(random_data(g, 12)).reshape(g.n_lines, -1).astype(np.complex64)
    got = plan.signal_adj(torch.from_numpy(y.reshape(plan.data_shape)).cuda()).cpu().numpy()
    assert _line_errors(got, signal.adjoint(g, y).reshape(plan.lines_shape)).max() <= TOL


@pytest.mark.parametrize("nx,nz,M,T,hi,hb", [(32, 3, 2, 1999, 15, 2), (64, 16, 9, 2050, 11, 3), (70, 37, 11, 3001, 31, 3),
                                             (128, 33, 24, 2500, 9, 2), (131, 12, 7, 6001, 31, 3),
                                             (192, 50, 30, 4999, 31, 3), (200, 5, 3, 2047, 7, 2), (256, 64, 40, 2999, 40, 3)])
@pytest.mark.parametrize("raster", [False, True])
def test_dense_split_stages(nx, nz, M, T, hi, hb, raster):
    """T no multiple of 32: the dense stage, at one and several column groups, few and many lines."""
    import torch
    from paper_2511_06627_amd.plan import Plan
    args = (nx, 12, nz, M, T, T / 128 + 1 / 3, 2.0, 1, hi, hb)
    sweep = nx / 2.0 if raster else 0.0
    g = oracle_geometry(*args)
    g.raster_sweep = sweep
    plan = Plan(*args, 1.0, raster_sweep=sweep)
    assert plan.dft_cycles == 0
    rng = np.random.default_rng(13)
    rho = rng.uniform(0, 1, (g.n_lines, g.n_u)).astype(np.float32)
    rho[1] *= 1e-20
    rho[2] = 0.0
    got = plan.signal_fwd(torch.from_numpy(rho.reshape(plan.lines_shape)).cuda()).cpu().numpy()
    want = signal.forward(g, rho)
    zero = np.arange(g.n_lines) == 2
    assert not got.reshape(g.n_lines, -1)[zero].any()
    ef = _line_errors(got.reshape(g.n_lines, -1)[~zero], want.reshape(g.n_lines, -1)[~zero]).max()
    y = np.asarray(random_data(g, 14)).reshape(g.n_lines, -1).astype(np.complex64)
    y[1] *= 1e20
    y[2] = 0.0
    got = plan.signal_adj(torch.from_numpy(y.reshape(plan.data_shape)).cuda()).cpu().numpy()
    want = signal.adjoint(g, y)
    assert not got.reshape(g.n_lines, -1)[zero].any()
    ea = _line_errors(got.reshape(g.n_lines, -1)[~zero], want.reshape(g.n_lines, -1)[~zero]).max()
    print("dense split %dx%d M %d T %d raster %d: forward %.2e adjoint %.2e" % (nx, nz, M, T, raster, ef, ea), flush=True)
    assert ef <= TOL and ea <= TOL
