"""The dense FP32 stage on fp16 pairs is as accurate as the one on fp32 MFMA.

A plan that also holds the mixed operator keeps the fp32 matrix unit for the same
scan; both are compared with the float64 line matrix.  Tolerance: an rms over
1e5 and more independent roundings is good to well under a percent; 5% covers the
two forms' different numbers of time ranges.
"""
import numpy as np
import pytest

from oracle import signal
from helpers import oracle_geometry, random_data

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,M,T", [(64, 64, 24, 4001), (128, 64, 24, 5001), (224, 64, 24, 6001)])
def test_pairs_against_fp32_products(nx, nz, M, T):
    import torch
    from paper_2511_06627_amd.plan import Plan
    args = (nx, 12, nz, M, T, T / 256 + 1 / 3, 3.0, 1, 31, 3)
    g = oracle_geometry(*args)
    C = signal.line_matrix(g)
    rho = np.random.default_rng(31).uniform(0, 1, (g.n_lines, nx)).astype(np.float32)
    y = np.asarray(random_data(g, 32)).reshape(g.n_lines, -1).astype(np.complex64)
    wf, wa = rho.astype(np.float64) @ C.T, np.real(y.astype(np.complex128) @ np.conj(C))
    err = []
    for precisions in (("fp32",), ("fp32", "mixed")):
        plan = Plan(*args, 1.0, precisions=precisions)
        assert plan.dft_cycles == 0
        got = plan.signal_fwd(torch.from_numpy(rho.reshape(plan.lines_shape)).cuda()).cpu().numpy().reshape(wf.shape)
        ef = np.linalg.norm(got - wf) / np.linalg.norm(wf)
        got = plan.signal_adj(torch.from_numpy(y.reshape(plan.data_shape)).cuda()).cpu().numpy().reshape(wa.shape)
        err.append((ef, np.linalg.norm(got - wa) / np.linalg.norm(wa)))
    print("n_u %d T %d: forward %.2e (pairs) %.2e (fp32), adjoint %.2e %.2e"
          % (nx, T, err[0][0], err[1][0], err[0][1], err[1][1]), flush=True)
    assert err[0][0] <= 1.05 * err[1][0] and err[0][1] <= 1.05 * err[1][1]
