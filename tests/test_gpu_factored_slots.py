"""Factored FP32 stage of scans whose bins bunch into few residues.

With a whole multiple of 64 drive cycles in T over C the residues are 0, +-1, ...
and each pair of them holds two bins a harmonic: from 17 harmonics on more than a
slot takes, so pairs share several slots (in plans that also hold the mixed
operator; others take the dense form on fp16 pairs).  Stage entries against the FP64 oracle,
line by line, with the bound that the stage's fp16 pairs are tested by elsewhere:
three contractions in a row of pairs of 2^-23 stay below 8 x 2^-22 of a line's norm.
"""
import numpy as np
import pytest

from oracle import signal
from helpers import oracle_geometry, random_data

pytestmark = pytest.mark.gpu

TOL = 1.9e-6

# name: (nx, ny, nz, M, T, drive cycles, w, k_lo, k_hi, half band), precisions, C
CASES = {
    "residues_0_32": ((48, 20, 3, 11, 8192, 32.0, 2.0, 1, 34, 0), ("fp32", "mixed"), 64),
    "three_residues_38_bins": ((22, 23, 13, 5, 4096, 64.0, 2.0, 1, 19, 1), ("fp32", "mixed"), 64),
    "six_residues": ((80, 30, 1, 9, 4096, 32.0, 3.0, 1, 35, 1), ("fp32", "mixed"), 64),
    "full_residues": ((64, 20, 2, 17, 16384, 128.0, 2.0, 1, 24, 1), ("fp32", "mixed"), 64),
    "c32": ((33, 20, 4, 9, 2016, 32.0, 2.0, 1, 24, 1), ("fp32", "mixed"), 32),
    # a residue of 50 bins: not split (its rounding would not average out)
    "full_pair_stays_dense": ((64, 20, 2, 17, 16384, 128.0, 2.0, 1, 50, 1), ("fp32", "mixed"), 0),
}


def _line_errors(a, b):
    a, b = np.asarray(a), np.asarray(b)
    a, b = a.reshape(-1, a.shape[-1]), b.reshape(-1, b.shape[-1])
    return np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)


@pytest.mark.parametrize("name", list(CASES))
def test_stages_per_line(name):
    import torch
    from paper_2511_06627_amd.plan import Plan
    dims, precisions, C = CASES[name]
    g = oracle_geometry(*dims)
    plan = Plan(*dims, 1.0, precisions=precisions)
    assert plan.dft_cycles == C, "plan took C = %d" % plan.dft_cycles
    L = g.n_lines
    rho = (np.random.default_rng(7).uniform(0, 1, (L, g.n_u)) ** 3).astype(np.float32)
    got = plan.signal_fwd(torch.from_numpy(rho.reshape(plan.lines_shape)).cuda()).cpu().numpy()
    ef = _line_errors(got, np.asarray(signal.forward(g, rho)).reshape(plan.data_shape))
    y = np.asarray(random_data(g, 8)).reshape(L, -1).astype(np.complex64)
    got = plan.signal_adj(torch.from_numpy(y.reshape(plan.data_shape)).cuda()).cpu().numpy()
    ea = _line_errors(got, np.asarray(signal.adjoint(g, y)).reshape(plan.lines_shape))
    print("%s: A %.2e At %.2e" % (name, ef.max(), ea.max()), flush=True)
    assert ef.max() < TOL and ea.max() < TOL
