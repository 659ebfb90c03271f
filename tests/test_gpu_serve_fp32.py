"""Served FP32 requests share their signal launches, whatever form the FP32 stage has.

A request's iterates are the same bits alone and in a batch of requests of other
volumes and angle counts of its line class, and the signal kernels of a step are
launched a fixed number of times, not once a request.
"""
import pytest

pytestmark = pytest.mark.gpu

# name: (n_u, T, k_hi, half band), options, signal kernels' name, launches a step
FORMS = {
    "factored": ((48, 2048, 15, 2), {}, "fac_", 4),
    "factored_raster": ((48, 2048, 15, 2), {"raster_sweep": 24.0}, "fac_", 4),
    "factored_tensor": ((48, 2048, 15, 2), {"psf_rows": 2}, "fac_", 4),
    "pairs": ((48, 3001, 15, 2), {}, "split_", 2),
    "pairs_raster": ((48, 3001, 15, 2), {"raster_sweep": 24.0}, "split_", 2),
}
SCANS = ((12, 9, 5), (20, 16, 7), (48, 33, 12), (16, 16, 4), (30, 5, 3), (12, 9, 5))   # ny, nz, angles


def _states(name, which):
    import torch
    from paper_2511_06627_amd.plan import Plan, State
    (nu, T, hi, hb), opts, _, _ = FORMS[name]
    out = []
    for i in which:
        ny, nz, M = SCANS[i]
        plan = Plan(nu, ny, nz, M, T, T / 256 + 1 / 3, 2.0, 1, hi, hb, 1e-2, **opts)
        g = torch.Generator(device="cuda")
        g.manual_seed(100 + i)
        b = torch.view_as_complex(torch.randn(plan.data_shape + (2,), generator=g, device="cuda"))
        out.append(State(plan, b, 1e-3, precision="fp32", iters=4, clamp_every=2))
    return out


def _finish(states):
    from paper_2511_06627_amd.plan import batch_step
    live = states
    while live:
        batch_step(live)
        live = [s for s in live if not s.progress()[1]]
    return [s.x.clone() for s in states]


@pytest.mark.parametrize("name", list(FORMS))
def test_alone_and_batched_are_the_same_bits(name):
    import torch
    batched = _finish(_states(name, range(len(SCANS))))
    for i in range(len(SCANS)):
        alone = _finish(_states(name, [i]))[0]
        assert torch.isfinite(alone).all() and bool(alone.abs().max() > 0)
        assert torch.equal(alone, batched[i]), (name, i)


@pytest.mark.parametrize("name", list(FORMS))
def test_signal_launches_do_not_grow_with_requests(name):
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_2511_06627_amd.plan import batch_step
    _, _, kernel, want = FORMS[name]
    states = _states(name, [0, 0, 0, 0, 0])
    for _ in range(2):
        batch_step(states)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        batch_step(states)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "mpi3d" in e.name]
    if not names:
        pytest.skip("the profiler recorded no kernels")
    count = sum(kernel in n for n in names)
    print("%s: %d signal launches of %d for %d requests" % (name, count, len(names), len(states)), flush=True)
    assert count == want
