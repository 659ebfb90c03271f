"""Every kernel of the dense FP32 stage on fp16 pairs, each at a scan that takes it.

Each line against the float64 line matrix, at the tolerance of the pair products
(a number to 2^-23, products without lo lo: 8 x 2^-22 = 1.9e-6) relative to the sizes
of the products' terms, |C| |rho| and |C|^T |y|: few bins' random data can cancel
almost wholly, in any arithmetic (100 x 93 x 40, six bins: one line to 1/400 of its
terms).  The kernels that the scan is listed for are held to the profiler's names.
"""
import numpy as np
import pytest

from oracle import signal
from helpers import oracle_geometry, random_data
from test_gpu_routes import _kernels

pytestmark = pytest.mark.gpu

TOL = 1.9e-6

# (n_u, nz, M, T, k_hi, half band), forward and adjoint kernel: padded n_u, column tiles, waves
SCANS = [
    ((40, 1, 1, 2887, 13, 1), (64, 4, 4), (64, 4, 4)),
    ((192, 1, 2, 727, 8, 2), (192, 4, 4), (192, 4, 4)),
    ((128, 5, 1, 725, 29, 0), (128, 4, 4), (128, 4, 4)),
    ((256, 2, 1, 2753, 5, 3), (256, 3, 4), (256, 3, 4)),
    ((192, 1, 2, 1087, 18, 2), (192, 4, 4), (192, 7, 4)),
    ((40, 5, 1, 845, 31, 1), (64, 4, 4), (64, 6, 4)),
    ((192, 4, 1, 887, 23, 1), (192, 4, 4), (192, 5, 4)),
    ((40, 1, 1, 7595, 17, 3), (64, 4, 4), (64, 8, 4)),
    ((100, 1, 8, 737, 20, 3), (128, 4, 4), (128, 6, 4)),
    ((100, 2, 3, 1479, 20, 2), (128, 4, 4), (128, 7, 4)),
    ((128, 12, 1, 727, 23, 2), (128, 4, 4), (128, 8, 4)),
    ((256, 6, 3, 601, 11, 3), (256, 3, 4), (256, 5, 4)),
    ((40, 94, 39, 6309, 7, 0), (64, 4, 8), (64, 4, 8)),
    ((40, 80, 31, 3827, 26, 2), (64, 6, 4), (64, 6, 8)),
    ((100, 93, 40, 8457, 2, 1), (128, 4, 8), (128, 4, 8)),
    ((100, 93, 39, 3315, 20, 3), (128, 6, 8), (128, 6, 8)),
    ((192, 82, 40, 2723, 26, 3), (192, 4, 8), (192, 6, 8)),
    ((64, 50, 27, 8025, 29, 3), (64, 8, 4), (64, 8, 8)),
    ((220, 41, 45, 5265, 23, 3), (256, 4, 8), (256, 4, 8)),
    ((256, 5, 26, 8405, 29, 2), (256, 5, 4), (256, 5, 4)),
    ((128, 71, 33, 4937, 28, 3), (128, 7, 4), (128, 7, 8)),
    ((180, 59, 31, 1127, 23, 1), (192, 5, 4), (192, 5, 4)),
    ((180, 74, 44, 4561, 19, 3), (192, 5, 8), (192, 5, 8)),
    ((256, 63, 43, 5959, 12, 3), (256, 3, 8), (256, 3, 8)),
    ((100, 81, 45, 5509, 25, 2), (128, 8, 4), (128, 8, 8)),
    ((100, 90, 42, 763, 21, 3), (128, 6, 4), (128, 6, 4)),
    ((192, 89, 41, 841, 26, 3), (192, 7, 4), (192, 7, 4)),
    ((40, 72, 47, 8697, 23, 1), (64, 6, 8), (64, 6, 8)),
    ((180, 93, 23, 4823, 25, 3), (192, 6, 8), (192, 7, 4)),
    ((100, 69, 26, 7031, 28, 3), (128, 7, 8), (128, 7, 8)),
    ((180, 60, 40, 7511, 25, 2), (192, 4, 8), (192, 4, 8)),
    ((40, 71, 44, 5973, 29, 3), (64, 8, 8), (64, 8, 8)),
]


def _errors(got, want, terms):
    return float((np.linalg.norm(got - want, axis=1) / np.linalg.norm(terms, axis=1)).max())


@pytest.mark.parametrize("scan,fwd,adj", SCANS)
def test_stage(scan, fwd, adj):
    import torch
    from paper_2511_06627_amd.plan import Plan
    nu, nz, M, T, hi, hb = scan
    args = (nu, 8, nz, M, T, T / 64 + 1 / 3, 2.0, 1, hi, hb)
    g = oracle_geometry(*args)
    plan = Plan(*args, 1.0)
    C = signal.line_matrix(g)
    rho = np.random.default_rng(51).uniform(0, 1, (g.n_lines, nu)).astype(np.float32)
    y = np.asarray(random_data(g, 52)).reshape(g.n_lines, -1).astype(np.complex64)
    x, b = torch.from_numpy(rho.reshape(plan.lines_shape)).cuda(), torch.from_numpy(y.reshape(plan.data_shape)).cuda()
    names = _kernels(lambda: (plan.signal_fwd(x), plan.signal_adj(b)))
    assert "split_fwd_kernel<%d, %d, %d>" % fwd in names and "split_adj_kernel<%d, %d, %d, false>" % adj in names, names
    ef = _errors(plan.signal_fwd(x).cpu().numpy().reshape(g.n_lines, -1), rho.astype(np.float64) @ C.T,
                 rho.astype(np.float64) @ np.abs(C).T)
    ea = _errors(plan.signal_adj(b).cpu().numpy().reshape(g.n_lines, -1), np.real(y.astype(np.complex128) @ np.conj(C)),
                 np.abs(y).astype(np.float64) @ np.abs(C))
    print("%s: forward %.2e adjoint %.2e" % (scan, ef, ea), flush=True)
    assert ef <= TOL and ea <= TOL
