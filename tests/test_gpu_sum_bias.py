"""The FP32 adjoint signal stages' sums have no common sign of error.

The fp16 matrix instructions round their sums down; over a long chain that would
leave every line a little low, which a backprojection adds up over the angles.  A
line's error is at most 2^-22 of its norm, and over L independent lines the mean
error, against the lines' rms, is within 3 x 2^-22 / sqrt(L).
"""
import numpy as np
import pytest

from oracle import signal
from helpers import oracle_geometry, random_data

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz,M,T,C", [(96, 36, 8192, 32), (96, 36, 8101, 0), (50, 30, 6001, 0)])
def test_adjoint_lines_have_no_mean_error(nz, M, T, C):
    import torch
    from paper_2511_06627_amd.plan import Plan
    args = (192, 12, nz, M, T, T / 256 + 1 / 3, 3.0, 1, 31, 3)
    g = oracle_geometry(*args)
    plan = Plan(*args, 1.0)
    assert plan.dft_cycles == C
    y = np.asarray(random_data(g, 21)).reshape(g.n_lines, -1).astype(np.complex64)
    want = np.real(y.astype(np.complex128) @ np.conj(signal.line_matrix(g)))
    got = plan.signal_adj(torch.from_numpy(y.reshape(plan.data_shape)).cuda()).cpu().numpy().reshape(want.shape)
    mean = abs(float(np.mean(got.astype(np.float64) - want))) / float(np.sqrt(np.mean(want ** 2)))
    bound = 3 * 2.0 ** -22 / np.sqrt(g.n_lines)
    print("T %d, %d lines: mean error %.2e of the rms, bound %.2e" % (T, g.n_lines, mean, bound), flush=True)
    assert mean <= bound
