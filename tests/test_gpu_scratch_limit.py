"""Scans whose dense FP32 form fits the no-allocation scratch fit it in the factored form.

The factored stage's phase sums would take some of them past it: those take fewer
partial sums, the stage a range of line tiles at a time, or another form.
mpi3d_forward_noalloc has to serve them, in every precision the plan holds, with
mpi3d_forward's bits, and A and A^T have to agree, line by line, with the
precomposed operator (another path: one matrix a line, no phase sums) to the FP32
operators' 1e-5.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MIB = 1 << 20

FP32, MIXED = ("fp32", "precomposed"), ("fp32", "mixed", "precomposed")
# name: (nx, ny, nz, M, T, k_hi, half band), options, precisions, the stage takes ranges of tiles
SCANS = {
    "plain_256": ((256, 16, 145, 13, 12288, 24, 1), {}, FP32, False),
    "plain_192": ((192, 16, 303, 12, 12288, 14, 2), {}, FP32, False),
    "plain_173": ((173, 16, 112, 56, 4096, 19, 2), {}, FP32, False),
    "bunched_160": ((160, 16, 91, 58, 8192, 7, 1), {}, FP32, False),
    "bunched_200": ((200, 16, 80, 34, 16384, 18, 2), {}, FP32, False),
    "raster_64": ((64, 16, 300, 24, 12288, 25, 1), {"raster_sweep": 32.0}, FP32, False),
    "ranges_mixed_192": ((192, 16, 280, 12, 12288, 11, 3), {}, MIXED, True),
    "ranges_plain": ((64, 16, 70, 56, 16384, 11, 1), {}, MIXED, True),
    "ranges_raster": ((64, 16, 114, 52, 12288, 25, 1), {"raster_sweep": 32.0}, MIXED, True),
    "dual_128": ((128, 16, 72, 18, 12288, 18, 2), {"drive_axes": 2}, MIXED, False),
    "ranges_dual": ((96, 16, 20, 47, 16384, 12, 3), {"drive_axes": 2}, MIXED, True),
    "ranges_tensor": ((64, 16, 37, 87, 16384, 24, 0), {"psf_rows": 1}, FP32, True),
}


def _noalloc(plan, prec, x):
    import torch
    from paper_2511_06627_amd import _lib
    from paper_2511_06627_amd.plan import PRECISION
    out = torch.full(plan.data_shape, float("nan"), dtype=torch.complex64, device="cuda")
    rc = _lib.load().mpi3d_forward_noalloc(plan._h, PRECISION[prec], ctypes.c_void_p(x.data_ptr()),
                                           ctypes.c_void_p(out.data_ptr()),
                                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return rc, out


def _rel(a, b, dims):
    import torch
    a, b = (torch.view_as_real(t).double() if t.is_complex() else t.double() for t in (a, b))
    return float(((a - b).pow(2).sum(dims) / b.pow(2).sum(dims).clamp_min(1e-300)).sqrt().max())


# bunched bins whose least phase sums are past the scratch: whole phase sums
@pytest.mark.parametrize("scan", [((32, 33, 152, 54, 6144, 32.0, 22, 1), ("fp32", "mixed")),
                                  ((25, 17, 92, 113, 8192, 128.0, 17, 0), ("fp32",))])
def test_bunched_past_the_scratch_takes_no_ranges(scan):
    from paper_2511_06627_amd import _lib
    from paper_2511_06627_amd.plan import Plan
    (nx, ny, nz, M, T, P, hi, hb), precisions = scan
    plan = Plan(nx, ny, nz, M, T, P, 3.0, 1, hi, hb, 1e-3, precisions=precisions)
    phases = (M * nz + 31) // 32 * 32 * (T // plan.dft_cycles) * 32 * 4
    assert int(plan.info.op_ws_bytes) > max(phases, _lib.NOALLOC_SCRATCH_BYTES)


@pytest.mark.parametrize("name", list(SCANS))
def test_fits_and_agrees(name):
    import torch
    from paper_2511_06627_amd import _lib
    from paper_2511_06627_amd.plan import Plan
    (nx, ny, nz, M, T, hi, hb), opts, precisions, ranges = SCANS[name]
    plan = Plan(nx, ny, nz, M, T, T / 256 + 1 / 3, 3.0, 1, hi, hb, 1e-3, precisions=precisions, **opts)
    ws = int(plan.info.op_ws_bytes)
    rows = max(M * nz // (2 if "raster_sweep" in opts else 1), M * nx if "drive_axes" in opts else 0)
    phases = rows * (T // plan.dft_cycles) * 32 * 4 if plan.dft_cycles else 0      # 16 pairs of columns
    print("%s: workspace %.1f MiB, C %d, phase sums of a line group %.1f MiB"
          % (name, ws / MIB, plan.dft_cycles, phases / MIB), flush=True)
    assert ws <= _lib.NOALLOC_SCRATCH_BYTES
    assert (phases > ws) == ranges
    g = torch.Generator(device="cuda")
    g.manual_seed(41)
    x = torch.rand(plan.shape, generator=g, device="cuda")
    b, ref = plan.forward(x), plan.forward(x, precision="precomposed")
    for prec in precisions:
        rc, out = _noalloc(plan, prec, x)
        assert rc == 0 and torch.equal(torch.view_as_real(out), torch.view_as_real(plan.forward(x, precision=prec)))
    lines = b.reshape(-1, b.shape[-1])
    ef = _rel(lines, ref.reshape(lines.shape), (-1, -2))
    at, aref = plan.signal_adj(ref), plan.signal_adj(ref, precision="precomposed")
    ea = _rel(at.reshape(-1, plan.n_u), aref.reshape(-1, plan.n_u), -1)
    print("  worst line: forward %.2e adjoint %.2e" % (ef, ea), flush=True)
    assert ef <= 1e-5 and ea <= 1e-5


def test_operators_of_a_workspace_follow_one_another():
    """Phase sums lie where the mixed operator has its partial sums; a 192 x 192 x 96
    raster that holds both fits the scratch, and calls in one workspace, in any order,
    give the bits of calls in workspaces of their own (filled with NaN before)."""
    import torch
    from paper_2511_06627_amd import _lib
    from paper_2511_06627_amd.plan import Plan
    plan = Plan(192, 192, 96, 36, 8192, 8192 / 256 + 1 / 3, 3.0, 1, 31, 3, 1e-3, raster_sweep=96.0,
                precisions=("fp32", "mixed"))
    assert plan.dft_cycles == 32 and int(plan.info.op_ws_bytes) <= _lib.NOALLOC_SCRATCH_BYTES
    g = torch.Generator(device="cuda")
    g.manual_seed(43)
    x = torch.rand(plan.shape, generator=g, device="cuda")

    def run(ws):
        out = []
        for prec in ("fp32", "mixed", "fp32"):
            b = plan.forward(x, precision=prec, ws=fresh() if ws is None else ws)
            out += [torch.view_as_real(b), plan.adjoint(b, precision=prec, ws=fresh() if ws is None else ws)]
        return out

    def fresh():
        ws = plan.workspace("op")
        ws.fill_(0xff)
        return ws

    for a, b in zip(run(None), run(plan.workspace("op"))):
        assert torch.equal(a, b)
