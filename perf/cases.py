"""Performance cases: the operator and solver calls a reconstruction makes.

A case is a scan geometry, an operator precision and what is called: A, its
adjoint, A followed by A^T (one application of A^T A, the unit the solvers
spend their time in), a solve, or batched serving steps.  ``listed`` holds the
named cases, ``draw`` makes others of the same ranges, ``prepare`` builds the
plan and the inputs a program has in hand, ``run`` makes the calls, ``work``
counts what the calls cannot do without, and ``exact`` evaluates the same
definition in float64 with plain torch.
"""
import math

import torch

from paper_2511_06627_amd.plan import Plan, State, batch_step

RAYS_PER_GATHER = 1 << 22      # float64 gathers are done this many values at a time


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _scan(name, op, precision, nx, ny, nz, angles, n_t, width, harm_hi, half_band, **extra):
    case = {"name": name, "op": op, "precision": precision, "nx": nx, "ny": ny, "nz": nz, "angles": angles,
            "n_t": n_t, "psf_width": width, "harm_hi": harm_hi, "half_band": half_band, "sweep": 0.0,
            "psf_rows": 0, "axes": 1, "iters": 0, "requests": 1}
    case.update(extra)
    return case


def listed():
    return [
        # The large high-dynamic-range scan: each half of a solver iteration on
        # its own, in FP32 ...
        _scan("hdr256_forward_fp32", "forward", "fp32", 256, 256, 128, 60, 16384, 3.0, 47, 3),
        _scan("hdr256_adjoint_fp32", "adjoint", "fp32", 256, 256, 128, 60, 16384, 3.0, 47, 3),
        # ... and the pair with the mixed operator, as refinement sweeps apply it.
        _scan("hdr256_normal_mixed", "normal", "mixed", 256, 256, 128, 60, 16384, 3.0, 47, 3),
        # The realistic scan, one application of A^T A in each operator precision.
        _scan("real192_normal_fp32", "normal", "fp32", 192, 192, 96, 36, 8192, 3.0, 31, 3),
        _scan("real192_normal_mixed", "normal", "mixed", 192, 192, 96, 36, 8192, 3.0, 31, 3),
        _scan("real192_normal_precomposed", "normal", "precomposed", 192, 192, 96, 36, 8192, 3.0, 31, 3),
        # The same scan with the tensor PSF coupling three rows on each side.
        _scan("tensor192_normal_fp32", "normal", "fp32", 192, 192, 96, 36, 8192, 3.0, 31, 3, psf_rows=3),
        # A zig-zag raster scan of odd sizes (no size a multiple of a tile).
        _scan("raster_odd_normal_fp32", "normal", "fp32", 131, 117, 37, 23, 6001, 3.0, 31, 3, sweep=65.5),
        # The smallest scan: one application of A^T A, bound by launches.
        _scan("small32_normal_fp32", "normal", "fp32", 32, 32, 32, 8, 2048, 2.0, 15, 2),
        # A small request solved by itself: the first CGLS iterations (later
        # iterates of a CGLS run depend on every rounding before them).
        _scan("cgls64_fp32", "cgls", "fp32", 64, 64, 64, 24, 4096, 3.0, 31, 3, iters=3),
        # The momentum iteration with the finite-difference regulariser.
        _scan("momentum128_fp32", "momentum", "fp32", 128, 128, 64, 24, 6144, 3.0, 31, 3, iters=8),
        # Serving: batched mixed refinement steps of requests of two volume sizes.
        _scan("serve_mixed", "serve", "mixed", 128, 128, 64, 24, 4096, 3.0, 31, 3, iters=2, requests=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: scans of any size in the listed range, any T."""
    kind = rng.choice(("forward", "adjoint", "normal", "normal", "normal", "cgls", "momentum", "serve"))
    big = kind in ("forward", "adjoint", "normal")
    nx = _log_int(rng, 32, 256 if big else 128)
    ny = min(256, max(32, int(round(nx * rng.uniform(0.75, 1.3)))))
    nz = _log_int(rng, 16, 128 if big else 64)
    angles = _log_int(rng, 8, 60 if big else 24)
    n_t = rng.choice((2048, 4096, 6144, 8192, 16384, rng.randint(2048, 12000), 64 * rng.randint(40, 200)))
    if not big:
        n_t = min(n_t, 8192)
    half_band = rng.choice((2, 3))
    harm_hi = rng.randint(15, 47)
    precision, extra = "fp32", {}
    if big:
        precision = rng.choice(("fp32", "fp32", "mixed", "mixed", "precomposed"))
        variant = rng.choice(("plain", "plain", "plain", "plain", "raster", "tensor"))
        if variant == "raster":
            extra["sweep"] = 0.5 * nx
        elif variant == "tensor" and nx <= 192 and angles * nz <= 3456:
            extra["psf_rows"] = rng.choice((1, 2, 3))
    elif kind == "serve":
        precision = "mixed"
        extra.update(iters=rng.randint(1, 2), requests=rng.randint(2, 5))
    else:
        extra["iters"] = rng.randint(2, 3) if kind == "cgls" else rng.randint(4, 10)
    if precision == "precomposed":
        n_t = min(n_t, 8192)          # its plan forms F^T K on the host: what such a scan keeps small
    width = rng.choice((2.0, 3.0))
    case = _scan("", kind, precision, nx, ny, nz, angles, n_t, width, harm_hi, half_band, **extra)
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _requests(case):
    """The scans of a case: one, or for serving every second request at half
    the volume size with half the angles."""
    out = []
    for i in range(case["requests"]):
        c = dict(case)
        if i % 2:
            c.update(nx=max(32, case["nx"] // 2), ny=max(32, case["ny"] // 2), nz=max(16, case["nz"] // 2),
                     angles=max(8, case["angles"] // 2))
        out.append(c)
    return out


def _n_bins(case):
    return case["harm_hi"] * (2 * case["half_band"] + 1)


def _phantom(case, gen):
    """Nonnegative volume: one large ellipsoid and Gaussian blobs whose
    amplitudes span three decades (float32, on the GPU)."""
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    ax = [torch.arange(n, dtype=torch.float64, device="cuda") for n in (nz, ny, nx)]
    u = torch.rand(24, 5, generator=gen, dtype=torch.float64).tolist()
    x = torch.zeros(nz, ny, nx, dtype=torch.float64, device="cuda")
    c = [(0.3 + 0.4 * u[0][d]) * (n - 1) for d, n in enumerate((nz, ny, nx))]
    r = [max(1.5, (0.12 + 0.13 * u[1][d]) * n) for d, n in enumerate((nz, ny, nx))]
    q = [((a - c[d]) / r[d]) ** 2 for d, a in enumerate(ax)]
    x += (q[0][:, None, None] + q[1][None, :, None] + q[2][None, None, :] <= 1.0)
    for b in u[2:]:
        sig = 1.0 + b[3] * max(0.5, min(nx, 160) / 20.0)
        g = [torch.exp(-0.5 * ((a - (0.1 + 0.8 * b[d]) * (a.numel() - 1)) / sig) ** 2) for d, a in enumerate(ax)]
        x += 10.0 ** (-3.0 * b[4]) * g[0][:, None, None] * g[1][None, :, None] * g[2][None, None, :]
    return x.to(torch.float32).contiguous()


def _data(case, gen):
    """Compressed data as a residual has them: complex noise whose level falls
    with the harmonic, above a floor (complex64, on the GPU)."""
    per = 2 * case["half_band"] + 1
    k = torch.arange(case["harm_hi"], dtype=torch.float64).repeat_interleave(per)
    env = (torch.exp(-k / 8.0) + 0.01).to(torch.float32).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(int(torch.randint(1 << 40, (1,), generator=gen)))
    re_im = torch.randn(case["angles"], case["nz"], _n_bins(case), 2, generator=g, device="cuda", dtype=torch.float32)
    return torch.view_as_complex((re_im * env[:, None]).contiguous())


def _host_gen(case, seed, i=0):
    g = torch.Generator()
    g.manual_seed(1000003 * int(seed) + i)
    return g


def _solve_inputs(case, seed, i):
    """Data b = A x + 0.5% noise of a phantom and the scale c_A that makes the
    operator's norm about 1, both from the float64 definition."""
    gen = _host_gen(case, seed, i)
    x = _phantom(case, gen)
    ref = _Reference(case, 1.0)
    one = dict(case, nz=1)
    ref1 = _Reference(one, 1.0)
    v = torch.ones(1, case["ny"], case["nx"], dtype=torch.float64, device="cuda")
    lam = 1.0
    for _ in range(12):
        w = ref1.adjoint(ref1.forward(v))
        lam = float(torch.linalg.vector_norm(w) / torch.linalg.vector_norm(v))
        v = w / torch.linalg.vector_norm(w)
    scale = float("%.3g" % (0.97 / math.sqrt(lam)))
    b = ref.forward(x.double()) * scale
    g = torch.Generator(device="cuda")
    g.manual_seed(int(torch.randint(1 << 40, (1,), generator=gen)))
    noise = torch.randn(b.shape + (2,), generator=g, device="cuda", dtype=torch.float64)
    b = b + torch.view_as_complex(noise) * (0.005 * float(b.abs().max()))
    return b.to(torch.complex64).contiguous(), scale


def _plan(case, op_scale):
    return Plan(case["nx"], case["ny"], case["nz"], case["angles"], case["n_t"], case["n_t"] / 256.0 + 1.0 / 3.0,
                case["psf_width"], 1, case["harm_hi"], case["half_band"], op_scale,
                precisions=("fp32",) if case["precision"] == "fp32" else ("fp32", case["precision"]),
                raster_sweep=case["sweep"], psf_rows=case["psf_rows"], drive_axes=case["axes"])


LAMBDA = 1e-3
TAU = 0.9          # momentum step: the operator norm is at most about 1


def prepare(case, seed):
    op = case["op"]
    if op in ("forward", "adjoint", "normal"):
        gen = _host_gen(case, seed)
        plan = _plan(case, 1.0)
        state = {"case": case, "plan": plan, "ws": plan.workspace("op"),
                 "b": torch.empty(plan.data_shape, dtype=torch.complex64, device="cuda"),
                 "x": torch.empty(plan.shape, dtype=torch.float32, device="cuda")}
        if op == "adjoint":
            state["in"] = _data(case, gen)
        else:
            state["in"] = _phantom(case, gen)
        return state
    reqs = []
    for i, c in enumerate(_requests(case)):
        b, scale = _solve_inputs(c, seed, i)
        plan = _plan(c, scale)
        reqs.append({"plan": plan, "b": b, "x": torch.empty(plan.shape, dtype=torch.float32, device="cuda"),
                     "ws": plan.workspace("solve")})
    return {"case": case, "reqs": reqs}


def run(state):
    case = state["case"]
    op, prec = case["op"], case["precision"]
    if op == "forward":
        return state["plan"].forward(state["in"], precision=prec, out=state["b"], ws=state["ws"])
    if op == "adjoint":
        return state["plan"].adjoint(state["in"], precision=prec, out=state["x"], ws=state["ws"])
    if op == "normal":
        p = state["plan"]
        p.forward(state["in"], precision=prec, out=state["b"], ws=state["ws"])
        p.adjoint(state["b"], precision=prec, out=state["x"], ws=state["ws"])
        return [state["b"], state["x"]]
    if op == "cgls":
        q = state["reqs"][0]
        x, _ = q["plan"].solve(q["b"], LAMBDA, iters=case["iters"], ws=q["ws"], report=False)
        return x
    if op == "momentum":
        q = state["reqs"][0]
        x, _ = q["plan"].solve(q["b"], LAMBDA, iters=case["iters"], clamp_every=1, solver="momentum", reg="fd",
                               tau=TAU, ws=q["ws"], report=False)
        return x
    # serving: one refinement sweep of every request, a batched step at a time
    states = [State(q["plan"], q["b"], LAMBDA, precision="mixed", refine_sweeps=1, inner_iters=case["iters"],
                    ws=q["ws"]) for q in state["reqs"]]
    live = states
    while live:
        batch_step(live)
        live = [s for s in live if not s.progress()[1]]
    xs = [s.x for s in states]
    for s in states:
        s.close()
    return xs


# ---------------------------------------------------------------------------
# Work a pass cannot do without
# ---------------------------------------------------------------------------
def _apply_work(c):
    """(floating-point operations, volume bytes, data bytes) of one application
    of A or A^T: ray samples inside the grid times the four-corner sum, the
    time signals of the lines and their transform (an FFT, or the kept columns
    alone where that is less); precomposed lines are one product each."""
    lines = c["angles"] * c["nz"]
    cols = 2 * _n_bins(c)
    vol, data = 4 * c["nx"] * c["ny"] * c["nz"], 4 * lines * cols
    flops = 8.0 * c["angles"] * c["nx"] * c["ny"] * c["nz"]
    if c["precision"] == "precomposed":
        flops += 2.0 * lines * c["nx"] * cols * (1 + c["psf_rows"])
    else:
        per_t = 2.0 * c["nx"] * (1 + c["psf_rows"]) + min(2.0 * cols, 2.5 * math.log2(c["n_t"]))
        flops += lines * c["n_t"] * per_t
    return flops, vol, data


def work(case):
    total = {"bytes": 0.0, "flops": 0.0}
    for c in _requests(case):
        flops, vol, data = _apply_work(c)
        op = case["op"]
        if op in ("forward", "adjoint"):
            n, byts = 1, vol + data
        elif op == "normal":
            n, byts = 2, 2 * vol + data
        else:
            # the data are read and the solution written once; every iteration
            # applies A and A^T, and the start one more of each kind
            n = 2 * case["iters"] + 1
            byts = vol + data + case["iters"] * (vol + data)
        total["flops"] += n * flops
        total["bytes"] += byts
    return total


# ---------------------------------------------------------------------------
# The definition in float64
# ---------------------------------------------------------------------------
def _langevin_deriv(x):
    """1/x^2 - 1/sinh^2 x; below 0.5 by the Maclaurin series."""
    x = x.abs()
    small = x < 0.5
    s = torch.where(small, x, torch.zeros_like(x)) ** 2
    # coefficients 2^{2n} B_{2n} (2n-1) / (2n)!
    bern = (1 / 6, -1 / 30, 1 / 42, -1 / 30, 5 / 66, -691 / 2730, 7 / 6, -3617 / 510, 43867 / 798, -174611 / 330)
    ser = torch.zeros_like(x)
    for n in range(len(bern), 0, -1):
        ser = ser * s + 4.0 ** n * bern[n - 1] * (2 * n - 1) / math.factorial(2 * n)
    big = torch.where(small, torch.ones_like(x), x)
    e = torch.exp(-2.0 * big)
    return torch.where(small, ser, 1.0 / (big * big) - 4.0 * e / (1.0 - e) ** 2)


def _langevin(x):
    """coth x - 1/x for x > 0 away from 0 (tensor PSF offsets are at least 1/w)."""
    return 1.0 / torch.tanh(x) - 1.0 / x


class _Reference:
    """A and A^T of a scan in float64: projection by bilinear ray samples, then
    per line the matrix C = F^T K (time signal and kept DFT bins in one)."""

    def __init__(self, c, op_scale):
        self.c = c
        f64 = dict(dtype=torch.float64, device="cuda")
        nx, ny, n_t = c["nx"], c["ny"], c["n_t"]
        nr = math.isqrt(nx * nx + ny * ny)
        if nr * nr < nx * nx + ny * ny:
            nr += 1
        nr += (nr - ny) % 2
        self.u = torch.arange(nx, **f64) - (nx - 1) / 2.0
        self.y = torch.arange(nr, **f64) - (nr - 1) / 2.0
        cycles = n_t / 256.0 + 1.0 / 3.0
        n = torch.arange(n_t, **f64)
        om = 2.0 * math.pi * cycles / n_t
        per = range(-c["half_band"], c["half_band"] + 1)
        bins = torch.tensor([math.floor(k * cycles + 0.5) + d for k in range(1, c["harm_hi"] + 1) for d in per],
                            dtype=torch.int64, device="cuda")
        ph = (torch.arange(n_t, dtype=torch.int64, device="cuda")[:, None] * bins[None, :]) % n_t
        ang = ph.double() * (2.0 * math.pi / n_t)
        f_re, f_im = torch.cos(ang) / math.sqrt(n_t), torch.sin(ang) / math.sqrt(n_t)
        self.mats = []           # [class or row offset] real (2 n_bins, n_u), re rows then im rows
        w, amp = c["psf_width"], nx / 2.0
        for sweep in ((c["sweep"], -c["sweep"]) if c["sweep"] else (0.0,)):
            xi = amp * torch.sin(om * n) + sweep * (n / n_t - 0.5)
            v = amp * om * torch.cos(om * n) + sweep / n_t
            du = xi[:, None] - self.u[None, :]
            for dz in range(min(c["psf_rows"], c["nz"] - 1) + 1):
                if dz == 0:
                    h = _langevin_deriv(du / w) / w
                else:
                    r2 = du * du + float(dz * dz)
                    r = torch.sqrt(r2)
                    h = _langevin_deriv(r / w) / w * (du * du / r2) + _langevin(r / w) * (dz * dz / (r2 * r))
                k = op_scale * v[:, None] * h
                self.mats.append(torch.cat([f_re.t().contiguous() @ k, f_im.t().contiguous() @ k]))

    def _samples(self, m):
        """Corner index (into the zero-bordered slice) and weight of every ray sample of angle m."""
        c = self.c
        th = m * math.pi / c["angles"]
        cs, sn = math.cos(th), math.sin(th)
        fx = (self.u[:, None] * cs + self.y[None, :] * sn + (c["nx"] - 1) / 2.0).reshape(-1)
        fy = (-self.u[:, None] * sn + self.y[None, :] * cs + (c["ny"] - 1) / 2.0).reshape(-1)
        i0, j0 = torch.floor(fx), torch.floor(fy)
        ax, ay = fx - i0, fy - j0
        inside = (i0 >= -1) & (i0 <= c["nx"] - 1) & (j0 >= -1) & (j0 <= c["ny"] - 1)
        i = torch.where(inside, i0, torch.zeros_like(i0)).long() + 1
        j = torch.where(inside, j0, torch.zeros_like(j0)).long() + 1
        pitch = c["nx"] + 2
        keep = inside.double()
        return [(j * pitch + i, (1 - ax) * (1 - ay) * keep), (j * pitch + i + 1, ax * (1 - ay) * keep),
                (j * pitch + pitch + i, (1 - ax) * ay * keep), (j * pitch + pitch + i + 1, ax * ay * keep)]

    def _groups(self, rays):
        """Runs of rays whose samples' values of all slices stay a bounded size."""
        per = max(1, RAYS_PER_GATHER * 8 // (self.c["nz"] * self.y.numel()))
        return [(a, min(rays, a + per)) for a in range(0, rays, per)]

    def project(self, x):
        c, nu, nr = self.c, self.u.numel(), self.y.numel()
        # voxels first, slices fastest
        pad = torch.zeros(c["ny"] + 2, c["nx"] + 2, c["nz"], dtype=torch.float64, device="cuda")
        pad[1:-1, 1:-1] = x.permute(1, 2, 0)
        pad = pad.reshape(-1, c["nz"])
        out = torch.empty(c["angles"], c["nz"], nu, dtype=torch.float64, device="cuda")
        for m in range(c["angles"]):
            corners = self._samples(m)
            for a, b in self._groups(nu):
                acc = 0.0
                for idx, wt in corners:
                    part = pad[idx[a * nr:b * nr]] * wt[a * nr:b * nr, None]
                    acc = acc + part.reshape(b - a, nr, c["nz"]).sum(1)
                out[m, :, a:b] = acc.t()
        return out

    def backproject(self, rho):
        c, nu, nr = self.c, self.u.numel(), self.y.numel()
        pad = torch.zeros((c["ny"] + 2) * (c["nx"] + 2), c["nz"], dtype=torch.float64, device="cuda")
        for m in range(c["angles"]):
            lines = rho[m].t().contiguous()
            corners = self._samples(m)
            for a, b in self._groups(nu):
                for idx, wt in corners:
                    vals = wt[a * nr:b * nr].reshape(b - a, nr, 1) * lines[a:b, None, :]
                    pad.index_add_(0, idx[a * nr:b * nr], vals.reshape(-1, c["nz"]))
        vol = pad.reshape(c["ny"] + 2, c["nx"] + 2, c["nz"])[1:-1, 1:-1]
        return vol.permute(2, 0, 1).contiguous()

    def _rows(self):
        """(matrix index, output rows, input rows) of every coupling of z-rows."""
        nz = self.c["nz"]
        if self.c["sweep"]:
            return [(0, slice(0, nz, 2), slice(0, nz, 2))] + ([(1, slice(1, nz, 2), slice(1, nz, 2))] if nz > 1 else [])
        out = [(0, slice(0, nz), slice(0, nz))]
        for e in range(1, len(self.mats)):
            out += [(e, slice(0, nz - e), slice(e, nz)), (e, slice(e, nz), slice(0, nz - e))]
        return out

    def forward(self, x):
        c = self.c
        rho = self.project(x)
        both = torch.zeros(c["angles"], c["nz"], 2 * _n_bins(c), dtype=torch.float64, device="cuda")
        for e, dst, src in self._rows():
            r = rho[:, src].contiguous()
            both[:, dst] += (r.reshape(-1, r.shape[-1]) @ self.mats[e].t().contiguous()).reshape(r.shape[0], r.shape[1], -1)
        nb = _n_bins(c)
        return torch.complex(both[..., :nb].contiguous(), both[..., nb:].contiguous())

    def adjoint(self, b):
        c = self.c
        both = torch.cat([b.real, b.imag], -1).double()
        rho = torch.zeros(c["angles"], c["nz"], c["nx"], dtype=torch.float64, device="cuda")
        for e, src, dst in self._rows():
            r = both[:, src].contiguous()
            rho[:, dst] += (r.reshape(-1, r.shape[-1]) @ self.mats[e]).reshape(r.shape[0], r.shape[1], -1)
        return self.backproject(rho)


def _exact_cgls(ref, b, iters):
    x = torch.zeros(ref.c["nz"], ref.c["ny"], ref.c["nx"], dtype=torch.float64, device="cuda")
    r = b.to(torch.complex128)
    s = ref.adjoint(r)
    p = s.clone()
    gamma = float((s * s).sum())
    for _ in range(iters):
        q = ref.forward(p)
        alpha = gamma / (float((q.real ** 2).sum() + (q.imag ** 2).sum()) + LAMBDA * float((p * p).sum()))
        x = x + alpha * p
        r = r - alpha * q
        s = ref.adjoint(r) - LAMBDA * x
        g1 = float((s * s).sum())
        p = s + (g1 / gamma) * p
        gamma = g1
    return x


def _laplacian(x):
    out = torch.zeros_like(x)
    for d in range(3):
        n = x.shape[d]
        if n < 2:
            continue
        diff = x.narrow(d, 1, n - 1) - x.narrow(d, 0, n - 1)
        out.narrow(d, 0, n - 1).sub_(diff)
        out.narrow(d, 1, n - 1).add_(diff)
    return out


def _exact_momentum(ref, b, iters):
    x = torch.zeros(ref.c["nz"], ref.c["ny"], ref.c["nx"], dtype=torch.float64, device="cuda")
    prev = x
    b = b.to(torch.complex128)
    for k in range(1, iters + 1):
        y = x + (k - 1.0) / (k + 2.0) * (x - prev)
        g = ref.adjoint(ref.forward(y) - b) + LAMBDA * _laplacian(y)
        prev, x = x, torch.clamp(y - TAU * g, min=0.0)
    return x


def exact(case, seed):
    op = case["op"]
    if op in ("forward", "adjoint", "normal"):
        gen = _host_gen(case, seed)
        ref = _Reference(case, 1.0)
        if op == "adjoint":
            return ref.adjoint(_data(case, gen))
        b = ref.forward(_phantom(case, gen).double())
        return b if op == "forward" else [b, ref.adjoint(b)]
    outs = []
    for i, c in enumerate(_requests(case)):
        b, scale = _solve_inputs(c, seed, i)
        ref = _Reference(c, scale)
        outs.append(_exact_momentum(ref, b, case["iters"]) if op == "momentum" else _exact_cgls(ref, b, case["iters"]))
    return outs if op == "serve" else outs[0]
