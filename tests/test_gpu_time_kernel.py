"""mpi3d_time_kernel's signal contractions cover every line, whatever the stage's form.

Kernels 2 and 3 are one whole contraction: with two line groups (a raster's sweep
directions, two drive axes) the factored stage launches its two kernels for each, or
once for both (variants of several jobs, last template argument true).  Kernels 4 to
7 are those of the first group.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opts", [{}, {"raster_sweep": 24.0}, {"drive_axes": 2}])
def test_signal_kernels_cover_every_line_group(opts):
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_2511_06627_amd.plan import Plan
    plan = Plan(48, 12, 16, 5, 2048, 2048 / 256 + 1 / 3, 2.0, 1, 15, 2, 1e-2, **opts)
    assert plan.dft_cycles == 32
    groups = 2 if opts else 1
    plan.time_kernel("signal_fwd", repeats=1)
    for kernel, want in (("signal_fwd", 2 * groups), ("signal_adj", 2 * groups), ("fac_fwd", 1), ("fac_adj_in", 1)):
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            ms = plan.time_kernel(kernel, repeats=3)
            torch.cuda.synchronize()
        names = [e.name for e in prof.events() if "mpi3d" in e.name]
        if not names:
            pytest.skip("the profiler recorded no kernels")
        count = sum((2 if "true>" in n else 1) for n in names if "fac_" in n)
        print("%s %s: %d groups' launches for 3 repeats, %.4f ms" % (opts, kernel, count, ms), flush=True)
        assert count == 3 * want and ms > 0
