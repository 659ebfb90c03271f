"""The residue DFT's table, held as fp16 pairs, has no gain of its own.

Its few distinct values repeat in every phase and line, so their roundings do not
average out: as they stand they make a forward 1.3e-8 low at these T, alike in every
line.  The gain of the whole stage, <b, b_64> / <b_64, b_64> against the FP64 oracle,
then is one within the roundings of the other tables (2^-23 a value, over more than
10^5 of them) and of the phase sums (2^-23 over 10^4 a line): 8e-9 leaves these four
times their sum, 2^-23 / 300 + 2^-23 / 100.
"""
import numpy as np
import pytest

from oracle import signal
from helpers import oracle_geometry

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k_hi", [(2816, 47), (3008, 47), (5120, 30)])
def test_forward_gain(T, k_hi):
    import torch
    from paper_2511_06627_amd.plan import Plan
    dims = (70, 20, 4, 10, T, T / 256 + 1 / 3, 3.0, 1, k_hi, 3)
    g = oracle_geometry(*dims)
    plan = Plan(*dims, 1.0)
    assert plan.dft_cycles
    rho = np.random.default_rng(3).uniform(0.5, 1.5, (g.n_lines, g.n_u)).astype(np.float32)
    want = np.asarray(signal.forward(g, rho)).reshape(plan.data_shape)
    got = plan.signal_fwd(torch.from_numpy(rho.reshape(plan.lines_shape)).cuda()).cpu().numpy().astype(complex)
    gain = float((got * want.conj()).real.sum() / (want * want.conj()).real.sum())
    print("T = %d, C = %d: gain 1 %+.2e" % (T, plan.dft_cycles, gain - 1), flush=True)
    assert abs(gain - 1) < 8e-9
