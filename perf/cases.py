"""The work that users of this library have it do, as timed and compared cases.

Five kinds of call, all through the public classes:

  cycle     one Wave-ADR cycle u <- C(u, g) (the preconditioner application, and the layer
            that unrolled training stacks)
  solve     the outer solve to a relative residual of 1e-6: FGMRES in FP64, or FP32 cycles
            inside FP64 refinement
  batch     independent problems of mixed sizes solved together
  adjoint   a training step: K unrolled cycles, the residual loss, and the gradients with
            respect to the phase and the level weights
  eikonal   the travel-time phase of point sources

Media, sources and phases are made on the GPU with plain torch from the seed; `exact`
evaluates a cycle and a training step in complex128 with plain torch operations.
"""
import math

import torch

DEV = "cuda:0"


# ---------------------------------------------------------------------------- the cases
def listed():
    return [
        # the constant-medium 128^2 problem of the parity tests (FP64): the smallest call, all latency
        dict(name="cycle_c128_128", kind="cycle", n=128, ny=128, prec="c128", kh=0.625, levels=4, medium="const"),
        # one problem of the size of the batched workload's small members
        dict(name="cycle_c64_256", kind="cycle", n=256, ny=256, prec="c64", kh=0.625, levels=5, medium="grf"),
        # the differentiation workload's grid, forward only
        dict(name="cycle_c64_1024", kind="cycle", n=1024, ny=1024, prec="c64", kh=0.625, levels=7, medium="grf"),
        # the same grid in FP64 (FGMRES in FP64, gradients to full precision)
        dict(name="cycle_c128_1024", kind="cycle", n=1024, ny=1024, prec="c128", kh=0.625, levels=7, medium="grf"),
        # a non-square domain of aspect 4 (seismic sections are wider than deep)
        dict(name="cycle_c64_4096x1024", kind="cycle", n=4096, ny=1024, prec="c64", kh=0.513, levels=7,
             medium="layered"),
        # the benchmark's grid: the preconditioner application of the 4096^2 solve
        dict(name="cycle_c64_4096", kind="cycle", n=4096, ny=4096, prec="c64", kh=0.513, levels=7, medium="layered"),
        # a heterogeneous problem solved in FP64
        dict(name="solve_c128_512", kind="solve", n=512, ny=512, prec="c128", kh=0.625, levels=6, medium="grf"),
        # a layered medium with FP32 cycles and FP64 refinement, the benchmark's method
        dict(name="solve_c64_2048", kind="solve", n=2048, ny=2048, prec="c64", kh=0.513, levels=7, medium="layered"),
        # many small problems at once: eleven problems of mixed size on four lanes
        dict(name="batch_c64_11", kind="batch", count=11, small=256, large=512, prec="c64", kh=0.625, lanes=4),
        # a training step on the differentiation workload (FP32, ten cycles)
        dict(name="adjoint_c64_1024_k10", kind="adjoint", n=1024, ny=1024, prec="c64", kh=0.625, levels=7,
             medium="grf", cycles=10),
        # gradients in FP64 on a small grid (gradient checks, inversion with few cycles)
        dict(name="adjoint_c128_256_k3", kind="adjoint", n=256, ny=256, prec="c128", kh=0.625, levels=5,
             medium="grf", cycles=3),
        # the phase of a new shot
        dict(name="eikonal_2048", kind="eikonal", n=2048, ny=2048, nsrc=1, medium="layered"),
    ]


def draw(rng):
    kind = rng.choices(["cycle", "solve", "batch", "adjoint", "eikonal"], [8, 3, 2, 3, 2])[0]
    kh = round(rng.uniform(0.35, 0.65), 4)  # k h: about ten to twenty-seven nodes per shortest unit-speed wavelength

    def sides(lo, hi):
        n = 1 << rng.randint(lo, hi)
        ny = n
        if rng.random() < 0.4:  # wide and tall domains, aspect 2 to 8
            ny = max(32, n >> rng.randint(1, 3))
            if rng.random() < 0.5:
                n, ny = ny, n
        return n, ny

    def levels(n, ny):
        top = max(2, min(7, int(math.log2(min(n, ny))) - 3))
        return top if rng.random() < 0.7 else rng.randint(min(3, top), top)

    if kind == "cycle":
        prec = rng.choice(["c64", "c64", "c128"])
        n, ny = sides(6, 12 if prec == "c64" else 11)
        return dict(kind=kind, n=n, ny=ny, prec=prec, kh=kh, levels=levels(n, ny),
                    medium=rng.choice(["const", "grf", "layered"]))
    if kind == "solve":
        prec = rng.choice(["c64", "c128"])
        n, ny = sides(6, 10)
        return dict(kind=kind, n=n, ny=ny, prec=prec, kh=kh, levels=max(2, min(7, int(math.log2(min(n, ny))) - 3)),
                    medium=rng.choice(["const", "grf"]))
    if kind == "batch":
        small = 1 << rng.randint(6, 8)
        return dict(kind=kind, count=rng.randint(2, 13), small=small, large=2 * small, prec="c64", kh=kh,
                    lanes=rng.randint(1, 4))
    if kind == "adjoint":
        prec = rng.choice(["c64", "c128"])
        n, ny = sides(6, 9)
        return dict(kind=kind, n=n, ny=ny, prec=prec, kh=kh, levels=levels(n, ny),
                    medium=rng.choice(["const", "grf"]), cycles=rng.randint(1, 6))
    n, ny = sides(6, 11)
    return dict(kind=kind, n=n, ny=ny, nsrc=rng.randint(1, 3), medium=rng.choice(["const", "grf", "layered"]))


# ---------------------------------------------------------------------------- inputs (plain torch)
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(gen, count, lo, hi):
    return (lo + (hi - lo) * torch.rand(count, generator=gen, device=DEV, dtype=torch.float64)).tolist()


def _smooth(field, sigma):
    """Gaussian filter of standard deviation sigma (cells), edge values extended."""
    p = int(4 * sigma) + 1
    v = torch.nn.functional.pad(field[None, None], (p, p, p, p), mode="replicate")[0, 0]
    fy = torch.fft.fftfreq(v.shape[0], device=DEV, dtype=torch.float64)[:, None]
    fx = torch.fft.rfftfreq(v.shape[1], device=DEV, dtype=torch.float64)[None, :]
    v = torch.fft.irfft2(torch.fft.rfft2(v) * torch.exp(-2 * (math.pi * sigma) ** 2 * (fy * fy + fx * fx)), s=v.shape)
    return v[p:-p, p:-p].contiguous()


def _velocity(n, ny, medium, gen):
    """Wave speeds in [1.5, 4.5] (const: 1): a smooth random field of correlation length
    0.1, or layers with elliptical inclusions smoothed over about one wavelength."""
    big = max(n, ny)
    if medium == "const":
        return torch.ones((ny, n), device=DEV, dtype=torch.float64)
    if medium == "grf":
        v = torch.randn((ny, n), generator=gen, device=DEV, dtype=torch.float64)
        fy = torch.fft.fftfreq(ny, d=1.0 / big, device=DEV, dtype=torch.float64)[:, None]
        fx = torch.fft.rfftfreq(n, d=1.0 / big, device=DEV, dtype=torch.float64)[None, :]
        v = torch.fft.irfft2(torch.fft.rfft2(v) * torch.exp(-(math.pi * 0.1) ** 2 * (fy * fy + fx * fx)), s=v.shape)
        return 1.5 + 3.0 * (v - v.min()) / (v.max() - v.min())
    y = torch.arange(ny, device=DEV, dtype=torch.float64) / big
    x = torch.arange(n, device=DEV, dtype=torch.float64) / big
    ex, ey = n / big, ny / big
    depths = torch.tensor(sorted(_uniform(gen, 7, 0.0, ey)), device=DEV, dtype=torch.float64)
    speeds = torch.tensor(_uniform(gen, 8, 1.5, 4.5), device=DEV, dtype=torch.float64)
    c = speeds[torch.searchsorted(depths, y, right=True)][:, None].expand(ny, n).clone()
    for _ in range(20):
        cx, cy, a, b, th, sg = _uniform(gen, 6, 0.0, 1.0)
        cx, cy, a, b, th = (0.05 + 0.9 * cx) * ex, (0.05 + 0.9 * cy) * ey, 0.02 + 0.06 * a, 0.02 + 0.06 * b, th * math.pi
        dx, dy = x[None, :] - cx, y[:, None] - cy
        u, v = dx * math.cos(th) + dy * math.sin(th), dy * math.cos(th) - dx * math.sin(th)
        c = torch.where((u / a) ** 2 + (v / b) ** 2 <= 1.0, c * (1.3 if sg < 0.5 else 0.7), c)
    return _smooth(c, 0.01 * big)


def _sponge(n, ny, k, vel):
    return max(16, math.ceil(2 * math.pi * float(vel.max()) * max(n, ny) / k))


def _sources(n, ny, count, margin, gen):
    big = max(n, ny)
    m = min(margin, min(n, ny) // 2 - 2)
    return [(_uniform(gen, 1, m, n - m)[0] / big, _uniform(gen, 1, m, ny - m)[0] / big) for _ in range(count)]


def _source_field(n, ny, xy):
    """Unit-mass Gaussians of two cells' width, zero on the ring."""
    h = 1.0 / max(n, ny)
    y = torch.arange(ny, device=DEV, dtype=torch.float64) * h
    x = torch.arange(n, device=DEV, dtype=torch.float64) * h
    s = 2 * h
    g = torch.zeros((ny, n), device=DEV, dtype=torch.float64)
    for x0, y0 in xy:
        g += torch.outer(torch.exp(-((y - y0) ** 2) / (2 * s * s)), torch.exp(-((x - x0) ** 2) / (2 * s * s)))
    g /= 2 * math.pi * s * s
    g[0, :] = 0
    g[:, 0] = 0
    return g.to(torch.complex128)


def _straight_ray_phase(vel, xy):
    """Travel time along straight rays: the distance to the source times the mean slowness
    of sixteen points between them, the smallest over the sources."""
    ny, n = vel.shape
    h = 1.0 / max(n, ny)
    y = torch.arange(ny, device=DEV, dtype=torch.float64)[:, None] * h
    x = torch.arange(n, device=DEV, dtype=torch.float64)[None, :] * h
    best = None
    for x0, y0 in xy:
        mean = torch.zeros_like(vel)
        for q in range(16):
            t = (q + 0.5) / 16
            i = ((y0 + t * (y - y0)) / h).round().long().clamp(0, ny - 1)
            j = ((x0 + t * (x - x0)) / h).round().long().clamp(0, n - 1)
            mean += 1.0 / vel[i, j]
        tau = torch.sqrt((x - x0) ** 2 + (y - y0) ** 2) * _smooth(mean / 16, 4.0)
        best = tau if best is None else torch.minimum(best, tau)
    return best.contiguous()


def _noise(shape, gen, dtype):
    v = torch.randn((*shape, 2), generator=gen, device=DEV, dtype=torch.float64)
    v = torch.view_as_complex(v)
    v[0, :] = 0
    v[:, 0] = 0
    return v.to(dtype)


def _cycle_inputs(case, seed):
    """velocity, sponge width, phase and, per kind, the right-hand side and first iterate."""
    gen = _gen(seed)
    n, ny = case["n"], case["ny"]
    k = case["kh"] * max(n, ny)
    vel = _velocity(n, ny, case["medium"], gen)
    W = _sponge(n, ny, k, vel)
    xy = _sources(n, ny, 1, W + 4, gen)
    phi = _straight_ray_phase(vel, xy)
    cdt = torch.complex64 if case["prec"] == "c64" else torch.complex128
    if case["kind"] == "adjoint":
        if case["prec"] == "c64":
            phi = phi.to(torch.float32)
        g, u0 = _source_field(n, ny, xy).to(cdt), None
    else:
        # a Krylov vector and an iterate of its size
        g = _noise((ny, n), gen, cdt)
        u0 = (_noise((ny, n), gen, torch.complex128) / (8.0 * max(n, ny) ** 2)).to(cdt)
    return vel, k, W, phi, g, u0


# ---------------------------------------------------------------------------- prepare and run
def prepare(case, seed):
    from paper_2404_02493_amd import Helmholtz, HelmholtzBatch

    kind = case["kind"]
    if kind in ("cycle", "adjoint"):
        vel, k, W, phi, g, u0 = _cycle_inputs(case, seed)
        helm = Helmholtz(vel, k, levels=case["levels"], precision=case["prec"], damping_cells=W)
        helm.set_phase(phi)
        if kind == "cycle":
            return dict(kind=kind, helm=helm, g=g, u0=u0, u=torch.empty_like(u0))
        w = torch.as_tensor(helm.weights, dtype=torch.float64)
        return dict(kind=kind, helm=helm, g=g, phi=phi.requires_grad_(True), w=w.requires_grad_(True),
                    cycles=case["cycles"])
    gen = _gen(seed)
    if kind == "solve":
        n, ny = case["n"], case["ny"]
        k = case["kh"] * max(n, ny)
        # one medium per case, a new shot per seed
        vel = _velocity(n, ny, case["medium"], _gen(7))
        W = _sponge(n, ny, k, vel)
        xy = _sources(n, ny, 1, W + 4, gen)
        helm = Helmholtz(vel, k, levels=case["levels"], precision=case["prec"], damping_cells=W)
        helm.eikonal(xy)
        return dict(kind=kind, helm=helm, g=_source_field(n, ny, xy), mode=1 if case["prec"] == "c64" else 0)
    if kind == "batch":
        probs, gs = [], []
        for p in range(case["count"]):
            n = case["small"] if p % 3 else case["large"]
            k = case["kh"] * n
            vel = _velocity(n, n, "grf", gen)
            W = max(16, math.ceil(2 * math.pi * 4.5 * n / k))
            xy = _sources(n, n, 1 + p % 4, W + 4, gen)
            probs.append(dict(velocity=vel.cpu().numpy(), k=k, phi=_straight_ray_phase(vel, xy).cpu().numpy(),
                              damping_cells=W))
            gs.append(_source_field(n, n, xy))
        return dict(kind=kind, batch=HelmholtzBatch(probs, precision=case["prec"], lanes=case["lanes"]), gs=gs)
    n, ny = case["n"], case["ny"]
    vel = _velocity(n, ny, case["medium"], gen)
    helm = Helmholtz(vel, 0.5 * max(n, ny), precision="c64")
    out = [torch.empty((ny, n), device=DEV, dtype=torch.float64) for _ in range(2)]
    return dict(kind=kind, helm=helm, xy=_sources(n, ny, case["nsrc"], 4, gen), tau1=out[0], phi=out[1])


def run(state):
    kind = state["kind"]
    if kind == "cycle":
        u = state["u"]
        u.copy_(state["u0"])
        return state["helm"].cycle(state["g"], u)
    if kind == "solve":
        u, _, _, _ = state["helm"].solve(state["g"], tol=1e-6, maxit=600, mode=state["mode"])
        # with FP32 cycles the user keeps the field in FP32
        return u if state["mode"] == 0 else u.to(torch.complex64)
    if kind == "batch":
        us, _, _, _ = state["batch"].solve(state["gs"], tol=1e-6, maxit=400, mode=1)
        return [u.to(torch.complex64) for u in us]
    if kind == "adjoint":
        helm, phi, w = state["helm"], state["phi"], state["w"]
        u = helm.unrolled(phi, w, state["g"], state["cycles"])
        loss = helm.residual_loss(state["g"], u)
        gphi, gw = torch.autograd.grad(loss, (phi, w))
        return dict(u=u.detach(), grad_phi=gphi, grad_w=gw)
    rounds, _ = state["helm"].eikonal(state["xy"], tau1_out=state["tau1"], phi_out=state["phi"])
    return dict(tau1=state["tau1"], phi=state["phi"], rounds=rounds)


# ---------------------------------------------------------------------------- the work of a pass
def _cycle_work(n, ny, levels, prec):
    """(bytes, flops) of one cycle: every input, coefficient and output once; the flops of
    the smoothers, the eight ADR V-cycles on levels 2..4 and the transfers."""
    b, c = (8, 4) if prec == "c64" else (16, 8)
    N = n * ny
    by = (3 * b + c) * N
    fl = 2 * 45.0 * N
    for lv in range(2, levels + 1):
        Nl = N / 4 ** (lv - 1)
        by += c * Nl
        fl += (0 if lv == 3 else (10 if lv == levels else 12) * 2 * 28.0) * Nl + 30 * Nl
        if levels >= 3 and lv <= min(levels, 4):
            by += (2 * c + 2 * b if lv == 2 else 2 * c + b) * Nl
            smoothings = 1 if lv == min(levels, 4) else 2
            fl += 8 * (smoothings * (3.5 * 42 + 10 * 8 + 3 * 8) + (50 if lv == 2 else 0)) * Nl
    return by, fl


def work(case):
    kind = case["kind"]
    if kind == "cycle":
        by, fl = _cycle_work(case["n"], case["ny"], case["levels"], case["prec"])
        return dict(bytes=by, flops=fl)
    if kind == "solve":
        # iterations as measured on these media, the FGMRES basis (ten vectors deep on
        # average, each read twice) and one cycle per iteration
        N, its = case["n"] * case["ny"], 0.15 * case["kh"] * max(case["n"], case["ny"])
        by, fl = _cycle_work(case["n"], case["ny"], case["levels"], case["prec"])
        b = 8 if case["prec"] == "c64" else 16
        return dict(bytes=its * (by + 2 * 12 * b * N), flops=its * (fl + 2 * 2 * 10 * 8 * N))
    if kind == "batch":
        by = fl = 0.0
        for p in range(case["count"]):
            n = case["small"] if p % 3 else case["large"]
            w = work(dict(kind="solve", n=n, ny=n, prec="c64", kh=case["kh"], levels=max(2, int(math.log2(n)) - 3)))
            by, fl = by + w["bytes"], fl + w["flops"]
        return dict(bytes=by, flops=fl)
    if kind == "adjoint":
        by, fl = _cycle_work(case["n"], case["ny"], case["levels"], case["prec"])
        return dict(bytes=3 * case["cycles"] * by, flops=3 * case["cycles"] * fl)
    N = case["n"] * case["ny"]
    return dict(bytes=24.0 * N, flops=case["nsrc"] * 8 * 60.0 * N)  # two rounds of four sweeps


# ---------------------------------------------------------------------------- exact values (plain torch, 64 bits)
class _Exact:
    """Algorithm 1 in complex128 with plain torch operations (differentiable in phi and w)."""

    def __init__(self, vel, k, W, levels, phi, w=None):
        self.k, self.L, self.LA = k, levels, min(levels, 4)
        ny, n = vel.shape
        big = max(n, ny)
        n2 = 1.0 / (vel * vel)
        self.ih2, self.kap, self.lam, self.mask = {}, {}, {}, {}
        self.n2, self.delta = {}, {}
        alpha = [0.0] * levels
        for lv in range(1, levels + 1):
            s = 1 << (lv - 1)
            m = n2[::s, ::s]
            ti = torch.arange(m.shape[0], device=DEV, dtype=torch.float64) * s
            tj = torch.arange(m.shape[1], device=DEV, dtype=torch.float64) * s
            ri = (1 - torch.minimum(ti, ny - ti) / W).clamp(min=0)
            rj = (1 - torch.minimum(tj, n - tj) / W).clamp(min=0)
            self.delta[lv] = 0.5 * torch.maximum(ri[:, None], rj[None, :]) ** 2
            self.n2[lv] = m
            self.kap[lv] = k * k * m * torch.complex(torch.ones_like(m), self.delta[lv])
            self.ih2[lv] = (big / s) ** 2
            mask = torch.ones_like(m)
            mask[0, :] = 0
            mask[:, 0] = 0
            self.mask[lv] = mask
            inner = self.kap[lv][1:, 1:]
            self.lam[lv] = (float((4 * self.ih2[lv] - inner).abs().max()) + 4 * self.ih2[lv]) ** 2
            if w is None:
                q = m[1:, 1:]
                if lv == 1:
                    K = k * k * float(q.max()) / self.ih2[1]
                    alpha[0] = (4 - K) / (5 - K)
                else:
                    sy, sx = ((torch.arange(1, a, device=DEV, dtype=torch.float64) * math.pi / (2 * a)).sin() ** 2
                              for a in m.shape)
                    vals = (4 * self.ih2[lv] * (sy[:, None] + sx[None, :]) - k * k * float(q.mean())).square()
                    vals = vals.flatten().sort().values
                    mid = (vals.numel() - 1) // 2
                    med = vals[mid] if vals.numel() % 2 else 0.5 * (vals[mid] + vals[mid + 1])
                    alpha[lv - 1] = max(1.0, self.lam[lv] / float(med))
        self.w = alpha if w is None else w
        self.adr = {}
        if levels >= 3:
            for lv in range(2, self.LA + 1):
                self.adr[lv] = self._adr(lv, phi[:: 1 << (lv - 1), :: 1 << (lv - 1)])
            t = k * phi[::2, ::2]
            self.car = torch.complex(torch.cos(t), torch.sin(t))

    def _adr(self, lv, p):
        h = self.ih2[lv] ** -0.5

        def diff(f):  # first and second derivative along the rows of f (one-sided at the last)
            lo, c, hi = f[:-2], f[1:-1], f[2:]
            d1 = torch.cat([f[:1] * 0, (hi - lo) / (2 * h), (f[-1:] - f[-2:-1]) / h])
            d2 = torch.cat([f[:1] * 0, (hi - 2 * c + lo) / h ** 2, (f[-1:] - 2 * f[-2:-1] + f[-3:-2]) / h ** 2])
            return d1, d2

        py, pyy = diff(p)
        px, pxx = (v.T for v in diff(p.T))
        re = self.k ** 2 * (px * px + py * py - self.n2[lv])
        im = -self.k * (pxx + pyy) - self.k ** 2 * self.n2[lv] * self.delta[lv]
        m = self.mask[lv]
        return px * m, py * m, torch.complex(re, im) * m

    @staticmethod
    def _nb(u):
        v = torch.nn.functional.pad(u, (1, 1, 1, 1))
        return v[1:-1, :-2], v[1:-1, 2:], v[:-2, 1:-1], v[2:, 1:-1]  # west, east, south, north

    def A(self, lv, u, adj=False):
        w, e, s, n = self._nb(u)
        kap = self.kap[lv].conj() if adj else self.kap[lv]
        return self.mask[lv] * (self.ih2[lv] * (4 * u - (w + e + s + n)) - kap * u)

    def M(self, lv, x):
        px, py, c0 = self.adr[lv]
        w, e, s, n = self._nb(x)
        U = 0.5 * self.ih2[lv] ** 0.5 * (2 * (px.abs() + py.abs()) * x - (px + px.abs()) * w + (px - px.abs()) * e
                                        - (py + py.abs()) * s + (py - py.abs()) * n)
        return self.mask[lv] * (self.ih2[lv] * (4 * x - (w + e + s + n)) - 2j * self.k * U + c0 * x)

    def R(self, lv, r):
        w, e, s, n = self._nb(r)
        v = torch.nn.functional.pad(r, (1, 1, 1, 1))
        diag = v[:-2, :-2] + v[:-2, 2:] + v[2:, :-2] + v[2:, 2:]
        return ((4 * r + 2 * (w + e + s + n) + diag) / 16)[::2, ::2] * self.mask[lv + 1]

    def P(self, lv, e):
        v = torch.nn.functional.pad(e, (0, 1, 0, 1))
        ee, eo = e, 0.5 * (v[:-1, :-1] + v[:-1, 1:])
        oe = 0.5 * (v[:-1, :-1] + v[1:, :-1])
        oo = 0.25 * (v[:-1, :-1] + v[1:, :-1] + v[:-1, 1:] + v[1:, 1:])
        out = torch.stack([torch.stack([ee, eo], -1), torch.stack([oe, oo], -1)], 1)  # (I, 2, J, 2)
        return out.reshape(2 * e.shape[0], 2 * e.shape[1]) * self.mask[lv]

    def jacobi(self, u, g):
        return u + self.mask[1] * self.w[0] * (g - self.A(1, u)) / (4 * self.ih2[1] - self.kap[1])

    def cheb(self, lv, u, g, m):
        lam, a = self.lam[lv], self.lam[lv] / self.w[lv - 1]
        theta, dc = 0.5 * (lam + a), 0.5 * (lam - a)
        r = self.A(lv, g - self.A(lv, u), adj=True)
        d, rho = r / theta, dc / theta
        for step in range(1, m + 1):
            u = u + d
            if step < m:
                r = r - self.A(lv, self.A(lv, d), adj=True)
                den = 2 * theta - dc * rho
                d = (dc / den) * rho * d + (2 / den) * r
                rho = dc / den
        return u

    def gmres(self, lv, b, x, m):
        r = b - self.M(lv, x)
        beta = r.abs().square().sum().sqrt()
        V, H = [r / beta], []
        for j in range(m):
            v, col = self.M(lv, V[j]), []
            for q in V:
                col.append((q.conj() * v).sum())
                v = v - col[-1] * q
            nv = v.abs().square().sum().sqrt()
            col.append(nv.to(torch.complex128))
            H.append(torch.stack(col + [torch.zeros_like(col[0])] * (m - 1 - j)))
            V.append(v / nv)
        Hm = torch.stack(H, 1)
        y = torch.linalg.solve(Hm.mH @ Hm, Hm.mH[:, 0] * beta)
        return x + sum(y[j] * V[j] for j in range(m))

    def vcycle(self, lv, b):
        x = self.gmres(lv, b, torch.zeros_like(b), 3)
        if lv == self.LA:
            return x
        x = x + self.P(lv, self.vcycle(lv + 1, self.R(lv, b - self.M(lv, x))))
        return self.gmres(lv, b, x, 3)

    def cycle(self, lv, g, u):
        if lv == self.L:
            return self.cheb(lv, u, g, 10)
        if lv == 1:
            u = self.jacobi(u, g)
        elif lv != 3:
            u = self.cheb(lv, u, g, 5)
        rc = self.R(lv, g - self.A(lv, u))
        u = u + self.P(lv, self.cycle(lv + 1, rc, torch.zeros_like(rc)))
        if lv == 1:
            return self.jacobi(u, g)
        if lv == 3:
            return u
        u = self.cheb(lv, u, g, 5)
        if lv == 2 and self.L >= 3:
            for _ in range(8):
                u = u + self.vcycle(2, (g - self.A(2, u)) * self.car.conj()) * self.car
        return u


def exact(case, seed):
    if case["kind"] == "cycle":
        vel, k, W, phi, g, u0 = _cycle_inputs(case, seed)
        return _Exact(vel, k, W, case["levels"], phi).cycle(1, g.to(torch.complex128), u0.to(torch.complex128))
    if case["kind"] == "adjoint":
        vel, k, W, phi, g, _ = _cycle_inputs(case, seed)
        w = torch.tensor([float(v) for v in _Exact(vel, k, W, case["levels"], phi.to(torch.float64)).w],
                         dtype=torch.float64, device=DEV, requires_grad=True)
        p = phi.to(torch.float64).requires_grad_(True)
        ex = _Exact(vel, k, W, case["levels"], p, w)
        g = g.to(torch.complex128)
        u = torch.zeros_like(g)
        for _ in range(case["cycles"]):
            u = ex.cycle(1, g, u)
        loss = (g - ex.A(1, u)).abs().square().sum()
        gphi, gw = torch.autograd.grad(loss, (p, w))
        return dict(u=u.detach(), grad_phi=gphi, grad_w=gw)
    return None  # solves stop at a tolerance; the sweeps' result is the same double precision numbers
