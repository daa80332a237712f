"""What a user of the solver has it do: the cases whose speed is measured.

Every case is a plain dict.  ``kind`` names the public entry point that a pass
goes through:

``solve``      ``Solver.solve`` on fields that live on the device, from p = 0
               (``warm`` false) or from the solution of a nearby density, as a
               time step has it (``warm`` true);
``project``    ``poisson_project``, one pressure projection of a predicted face
               momentum, starting from the previous pressure;
``particles``  the coupling of particles and grid in one time step:
               ``poisson_interpolate`` of a field at the particles, then
               ``poisson_deposit`` of a particle value;
``serve``      a batch of independent requests of mixed sizes through ``Server``.

Grids are (nz, ny, nx); lengths of 2^a or 3 * 2^a.  Inputs are drawn from the
seed on the device, with the distributions of this package's workloads: band-
limited lognormal densities, hot-particle densities from a trilinear deposit,
band-limited right-hand sides and momenta, uniform particle positions.
"""
import math

import torch

from paper_1601_05448_amd import poisson as P
from paper_1601_05448_amd.serve import Server

TWO_PI = 2.0 * math.pi
C_DT = 5e-4
TOL = 1e-10
SERVED = (64, 96, 128, 192)


def _solve(name, shape, fp32, **over):
    case = {"name": name, "kind": "solve", "nz": shape[0], "ny": shape[1], "nx": shape[2], "fp32": fp32,
            "box": "cube", "walls": False, "density": "lognormal", "ratio": 4.0, "coef": P.POISSON_COEF_RHO_FACE_MEAN,
            "weight": P.POISSON_W_RHO, "warm": False}
    case.update(over)
    return case


def listed():
    return [
        # the smallest grid of the tests and of smoke(): launches and latency
        _solve("solve_f64_32", (32, 32, 32), False, density="sine"),
        # a small box in the mixed path, as a caller that runs many of them in a loop has
        _solve("solve_f32_64", (64, 64, 64), True),
        # an anisotropic box with lengths 3 * 2^a and the other weight
        _solve("solve_f64_96x192x48", (96, 192, 48), False, box="aniso", weight=P.POISSON_W_DIAG),
        # an ordinary box of a time-stepping code: warm start from the previous pressure
        _solve("solve_f64_128_warm", (128, 128, 128), False, warm=True),
        # the largest served size, mixed path
        _solve("solve_f32_192", (192, 192, 192), True),
        # the headline workload, both paths
        _solve("solve_f64_256", (256, 256, 256), False),
        _solve("solve_f32_256", (256, 256, 256), True),
        # the inflow-outflow duct (walls in x)
        _solve("duct_f32_512x256x256", (256, 256, 512), True, box="cells", walls=True),
        # fields beyond the memory-side cache: a hot-particle density, FP64
        _solve("solve_f64_512", (512, 512, 512), False, density="particles", ratio=10.0),
        # one projection of a time step
        {"name": "project_f32_256", "kind": "project", "nz": 256, "ny": 256, "nx": 256, "fp32": True, "box": "cube",
         "walls": False, "density": "lognormal", "ratio": 4.0, "coef": P.POISSON_COEF_RHO_FACE_MEAN,
         "weight": P.POISSON_W_RHO},
        # particles and the grid: the 10^6 particles and the grid of the particle-density workload
        {"name": "particles_1e6_512", "kind": "particles", "nz": 512, "ny": 512, "nx": 512, "particles": 10**6},
        # a served batch over the served sizes, FP64
        {"name": "serve_f64_24", "kind": "serve", "requests": 24, "fp32": False, "mix": "served"},
    ]


# ---- more cases of the same ranges ------------------------------------------------

_AXIS = (16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024)


def _draw_shape(rng, lo, hi):
    """A grid with lo..hi cells (uniform in the logarithm), sides within a factor of eight."""
    while True:
        want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        side = want ** (1.0 / 3.0)
        s = [rng.choice([a for a in _AXIS if side / 3.0 <= a <= side * 3.0]) for _ in range(3)]
        n = s[0] * s[1] * s[2]
        if want / 1.6 <= n <= want * 1.6 and lo <= n <= hi and max(s) <= 8 * min(s):
            return tuple(s)


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["duct"] * 2 + ["project", "particles", "serve"])
    if kind == "particles":
        nz, ny, nx = _draw_shape(rng, 2**15, 2**26)
        return {"kind": kind, "nz": nz, "ny": ny, "nx": nx,
                "particles": int(math.exp(rng.uniform(math.log(2e3), math.log(2e6))))}
    if kind == "serve":
        return {"kind": kind, "requests": rng.randint(2, 40), "fp32": rng.random() < 0.5,
                "mix": rng.choice(["served", "served", "64", "128"])}
    fp32 = rng.random() < 0.5
    nz, ny, nx = _draw_shape(rng, 2**14, 2**25 if not fp32 else 2**26)
    if kind == "project":
        return {"kind": kind, "nz": nz, "ny": ny, "nx": nx, "fp32": fp32, "box": "cells", "walls": rng.random() < 0.3,
                "density": "lognormal", "ratio": round(rng.uniform(2.0, 8.0), 2), "coef": P.POISSON_COEF_RHO_FACE_MEAN,
                "weight": P.POISSON_W_RHO}
    return {"kind": "solve", "nz": nz, "ny": ny, "nx": nx, "fp32": fp32,
            "box": rng.choice(["cube", "cells", "cells", "aniso"]), "walls": kind == "duct", "density": "lognormal",
            "ratio": round(rng.uniform(2.0, 8.0), 2),
            "coef": rng.choice([P.POISSON_COEF_RHO_FACE_MEAN] * 3 + [P.POISSON_COEF_INVRHO_FACE_MEAN]),
            "weight": rng.choice([P.POISSON_W_RHO] * 3 + [P.POISSON_W_DIAG]), "warm": rng.random() < 0.3}


# ---- inputs -----------------------------------------------------------------------


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _lengths(case):
    """(lx, ly, lz): a cube, equal cell sizes, or an anisotropic box."""
    if case.get("box", "cube") == "cube":
        return (TWO_PI, TWO_PI, TWO_PI)
    if case["box"] == "aniso":
        return (TWO_PI, 3.0, 5.0)
    h = TWO_PI / min(case["nx"], case["ny"], case["nz"])
    return (case["nx"] * h, case["ny"] * h, case["nz"] * h)


def _band_limited(shape, lengths, gen, kmax=8.0, shift=0.0):
    """Random field of the physical wavenumbers 0 < |k| <= kmax, zero mean, unit
    RMS, synthesised one direction after the other; `shift` carries the same
    field along x by that many cells."""
    dev = _device()
    nz, ny, nx = shape
    modes, phases = [], []
    for n, length in zip((nx, ny, nz), lengths):
        m = max(1, min(int(kmax * length / TWO_PI), n // 6, 16))
        a = torch.arange(-m, m + 1, dtype=torch.float64)
        x = (torch.arange(n, dtype=torch.float64) + 0.5) / n
        modes.append(a * (TWO_PI / length))
        phases.append(torch.exp(1j * TWO_PI * torch.outer(a, x)).to(dev))
    kx, ky, kz = modes
    k2 = kz[:, None, None] ** 2 + ky[None, :, None] ** 2 + kx[None, None, :] ** 2
    # a box whose smallest wavenumbers already exceed kmax keeps its first ones
    cut = max(kmax * kmax, 4.0 * float(k2[k2 > 0].min()))
    mask = (k2 > 0) & (k2 <= cut)
    coef = torch.complex(torch.randn(mask.shape, generator=gen, dtype=torch.float64),
                         torch.randn(mask.shape, generator=gen, dtype=torch.float64)) * mask
    if shift:
        coef = coef * torch.exp(-1j * kx * (shift * lengths[0] / nx))[None, None, :]
    t = (coef.reshape(-1, len(kx)).to(dev) @ phases[0]).reshape(len(kz), len(ky), nx)
    t = torch.stack([phases[1].T @ t[c] for c in range(len(kz))]).reshape(len(kz), ny * nx)
    ez = phases[2].T.contiguous()
    f = (ez.real.contiguous() @ t.real.contiguous() - ez.imag.contiguous() @ t.imag.contiguous()).reshape(shape)
    f -= f.mean()
    f /= f.square().mean().sqrt()
    return f.contiguous()


def _hot_particles(shape, gen, ratio, particles=10**6):
    """rho = 1 / (1 + (ratio - 1) d / max d), d the trilinear deposit of uniform
    particles, accumulated in whole numbers so that its order plays no part."""
    dev = _device()
    nz, ny, nx = shape
    pos = torch.rand(particles, 3, generator=gen, dtype=torch.float64).to(dev)
    i0, w = [], []
    for d, n in enumerate((nx, ny, nz)):
        s = pos[:, d] * n - 0.5
        fl = torch.floor(s)
        i0.append(torch.remainder(fl.to(torch.int64), n))
        w.append(((1.0 - (s - fl)), s - fl))
    d = torch.zeros(nz * ny * nx, dtype=torch.int64, device=dev)
    for c in range(8):
        a, b, e = c & 1, (c >> 1) & 1, c >> 2
        flat = ((torch.remainder(i0[2] + e, nz) * ny + torch.remainder(i0[1] + b, ny)) * nx
                + torch.remainder(i0[0] + a, nx))
        d.index_add_(0, flat, torch.round(w[0][a] * w[1][b] * w[2][e] * 2.0**30).to(torch.int64))
    d = d.to(torch.float64)
    return (1.0 / (1.0 + (ratio - 1.0) * (d / d.max()))).reshape(shape)


def _density(case, gen, shift=0.0):
    shape, lengths = (case["nz"], case["ny"], case["nx"]), _lengths(case)
    if case["density"] == "particles":
        return _hot_particles(shape, gen, case["ratio"])
    if case["density"] == "sine":
        at = []
        for n in shape:
            phase = float(torch.rand((), generator=gen, dtype=torch.float64))
            at.append(torch.sin(TWO_PI * ((torch.arange(n, dtype=torch.float64) + 0.5) / n + phase)))
        sz, sy, sx = at
        return (1.0 + 0.5 * sz[:, None, None] * sy[None, :, None] * sx[None, None, :]).to(_device()).contiguous()
    s = _band_limited(shape, lengths, gen, shift=shift)
    return torch.exp(s * (math.log(case["ratio"]) / float(s.max() - s.min()))).contiguous()


def _gen(seed, stream):
    return torch.Generator().manual_seed(1000003 * int(seed) + stream)


def _solve_fields(case, seed):
    """rho, b and, for a warm start, the density of the step before."""
    rho = _density(case, _gen(seed, 1))
    b = _band_limited((case["nz"], case["ny"], case["nx"]), _lengths(case), _gen(seed, 2))
    before = _density(case, _gen(seed, 1), shift=-0.5) if case.get("warm") else None
    return rho, b, before


def _momentum(case, seed):
    shape, lengths = (case["nz"], case["ny"], case["nx"]), _lengths(case)
    gen = _gen(seed, 3)
    m = [_band_limited(shape, lengths, gen) for _ in range(3)]
    return m, 0.1 * _band_limited(shape, lengths, gen)


def _positions(case, seed):
    return (torch.rand(case["particles"], 3, generator=_gen(seed, 4), dtype=torch.float64) * TWO_PI).to(_device())


def _particle_inputs(case, seed):
    pos = _positions(case, seed)
    q = (1.0 + 0.1 * torch.randn(case["particles"], generator=_gen(seed, 5), dtype=torch.float64)).to(_device())
    field = _band_limited((case["nz"], case["ny"], case["nx"]), _lengths(case), _gen(seed, 6))
    return pos, q, field


def _requests(case, seed):
    """The served requests as solve cases: sizes and density ratios of the
    request stream."""
    gen = _gen(seed, 7)
    sizes = SERVED if case["mix"] == "served" else (int(case["mix"]),)
    out = []
    for r in range(case["requests"]):
        # every size of the mix in turn, so that a batch costs the same for every seed
        n = sizes[r % len(sizes)]
        ratio = 2.0 + 6.0 * float(torch.rand((), generator=gen, dtype=torch.float64))
        out.append(_solve("", (n, n, n), case["fp32"], ratio=ratio))
    return out


def _solver(case):
    return P.Solver((case["nz"], case["ny"], case["nx"]), _lengths(case),
                    precision=P.POISSON_FP32_REFINE if case.get("fp32") else P.POISSON_FP64,
                    coef=case.get("coef", P.POISSON_COEF_RHO_FACE_MEAN), weight=case.get("weight", P.POISSON_W_RHO),
                    bc_x=P.POISSON_BC_WALLS_X if case.get("walls") else P.POISSON_BC_PERIODIC)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        jobs = []
        for k, c in enumerate(_requests(case, seed)):
            rho, b, _ = _solve_fields(c, 1000 * seed + k)
            jobs.append((c, rho, b, torch.zeros_like(b)))
        server = Server(16 << 30, 64, precision=P.POISSON_FP32_REFINE if case["fp32"] else P.POISSON_FP64)
        return {"case": case, "server": server, "jobs": jobs}
    solver = _solver(case)
    if kind == "particles":
        pos, q, field = _particle_inputs(case, seed)
        return {"case": case, "solver": solver, "pos": pos, "q": q, "field": field, "at": torch.empty_like(q),
                "grid": torch.empty_like(field)}
    if kind == "project":
        m, div = _momentum(case, seed)
        rho = _density(case, _gen(seed, 1))
        return {"case": case, "solver": solver, "rho": rho, "predicted": m, "m": [torch.empty_like(x) for x in m],
                "div": div, "p": torch.zeros_like(rho)}
    rho, b, before = _solve_fields(case, seed)
    p = torch.zeros_like(rho)
    p0 = None
    if before is not None:
        solver.solve(before, b, p, TOL)
        p0 = p.clone()
    return {"case": case, "solver": solver, "rho": rho, "b": b, "p": p, "p0": p0}


def run(state):
    kind = state["case"]["kind"]
    if kind == "serve":
        server, todo = state["server"], {}
        for c, rho, b, p in state["jobs"]:
            p.zero_()
            todo[server.submit(tuple(rho.shape), _lengths(c), rho, b, p, TOL)] = p
        while server.tick() > 0:
            pass
        codes = [server.poll(rid)["status"] for rid in todo]
        return {"p": list(todo.values()), "status": codes}
    h = state["solver"].h
    if kind == "particles":
        P.poisson_interpolate(h, state["pos"], state["field"], state["at"])
        P.poisson_deposit(h, state["pos"], state["q"], state["grid"])
        return {"at": state["at"], "grid": state["grid"]}
    if kind == "project":
        for m, new in zip(state["m"], state["predicted"]):
            m.copy_(new)
        state["p"].zero_()
        status, chi = P.poisson_project(h, state["rho"], *state["m"], state["div"], C_DT, state["p"], TOL)
        return {"m": state["m"], "p": state["p"], "status": status}
    if state["p0"] is None:
        state["p"].zero_()
    else:
        state["p"].copy_(state["p0"])
    stats = state["solver"].solve(state["rho"], state["b"], state["p"], TOL)
    return {"p": state["p"], "status": stats["code"]}


# ---- what a pass cannot do without ----------------------------------------------------


def _iterations(case):
    """About how many iterations the method takes at 1e-10 on these densities."""
    if case.get("density") == "particles":
        return 66
    return 8 if case.get("warm") else 10


def work(case):
    """Bytes: every FP64 input read once and every output written once.  Flops:
    per iteration the stencil (about 60 a cell) and the transforms there and
    back (2.5 log2 N a cell and direction each), and the multiples of a cell or
    particle that the other steps take."""
    if case["kind"] == "serve":
        parts = [work(c) for c in _requests(case, 0)]
        return {k: sum(w[k] for w in parts) for k in ("bytes", "flops")}
    n = case["nz"] * case["ny"] * case["nx"]
    if case["kind"] == "particles":
        np_ = case["particles"]
        # positions (read by both steps), values in and out, the grid written;
        # the field is read where there are particles
        return {"bytes": 8.0 * (n + 8 * np_ + min(n, 8 * np_)), "flops": 60.0 * np_}
    per_cell = 60.0 + 5.0 * math.log2(n)
    solve = {"bytes": 32.0 * n, "flops": _iterations(case) * per_cell * n}
    if case["kind"] == "project":
        # rho, three momenta and the target read, three momenta and p written, p read
        return {"bytes": 8.0 * 10 * n, "flops": solve["flops"] + 40.0 * n}
    return solve


# ---- the same in 64 bits, in plain torch --------------------------------------------------


class _Operator:
    """A p = div(beta grad p) on the staggered grid, and the exact inverse of
    the constant-coefficient operator, both from torch's own functions."""

    def __init__(self, rho, lengths, coef, walls):
        nz, ny, nx = rho.shape
        self.walls = walls
        self.inv_h = [n / length for n, length in zip((nz, ny, nx), (lengths[2], lengths[1], lengths[0]))]
        self.beta = []
        for ax in range(3):
            up = torch.roll(rho, -1, dims=ax)
            be = 2.0 / (rho + up) if coef == P.POISSON_COEF_RHO_FACE_MEAN else 0.5 * (1.0 / rho + 1.0 / up)
            if ax == 2 and walls:
                be[:, :, -1] = 0.0
            self.beta.append(be)
        lam = []
        for ax, n in enumerate((nz, ny, nx)):
            k = torch.arange(n, dtype=torch.float64, device=rho.device)
            arg = math.pi * k / (2 * n if ax == 2 and walls else n)
            lam.append(-4.0 * torch.sin(arg) ** 2 * self.inv_h[ax] ** 2)
        if not walls:
            lam[2] = lam[2][: nx // 2 + 1]
        self.lam = lam

    def apply(self, p):
        out = torch.zeros_like(p)
        for ax in range(3):
            flux = self.beta[ax] * (torch.roll(p, -1, dims=ax) - p) * self.inv_h[ax] ** 2
            out += flux - torch.roll(flux, 1, dims=ax)
        return out

    def lap_inverse(self, q):
        lam = self.lam[0][:, None, None] + self.lam[1][None, :, None] + self.lam[2][None, None, :]
        lam[0, 0, 0] = 1.0
        nx = q.shape[2]
        if self.walls:
            # even extension along x: its real transform of length 2 nx holds the cosine transform
            f = torch.fft.rfft(torch.cat([q, q.flip(2)], dim=2), dim=2)[:, :, :nx]
            f = torch.fft.fft2(f, dim=(0, 1)) / lam
            f[0, 0, 0] = 0.0
            f = torch.fft.ifft2(f, dim=(0, 1))
            f = torch.cat([f, torch.zeros_like(f[:, :, :1])], dim=2)
            return torch.fft.irfft(f, n=2 * nx, dim=2)[:, :, :nx].contiguous()
        f = torch.fft.rfftn(q) / lam
        f[0, 0, 0] = 0.0
        return torch.fft.irfftn(f, s=q.shape)


def _exact_solve(rho, b, lengths, coef, walls, smooth=True):
    """Conjugate gradients on -A, zero-mean, preconditioned by
    sqrt(rho) L^+ sqrt(rho) (by L^+ alone where the density is rough from cell
    to cell), down to the rounding floor."""
    op = _Operator(rho, lengths, coef, walls)
    root = torch.sqrt(rho) if smooth else torch.ones_like(rho)
    r = -(b - b.mean())
    p = torch.zeros_like(b)
    norm = float(r.norm())
    d, rz, best = None, 1.0, float("inf")
    since = 0
    for it in range(400):
        z = -root * op.lap_inverse(root * r)
        z -= z.mean()
        new = float((r * z).sum())
        d = z if d is None else z + (new / rz) * d
        rz = new
        ad = -op.apply(d)
        step = rz / float((d * ad).sum())
        p += step * d
        # the residual itself every few steps, so that it does not drift
        r = -(b - b.mean()) + op.apply(p) if it % 8 == 7 else r - step * ad
        rel = float(r.norm()) / norm
        if rel < 0.5 * best:
            best, since = rel, 0
        else:
            since += 1
        if rel < 3e-14 or (since > 12 and best < 1e-11):
            break
    return p - p.mean()


def _exact_particles(case, seed):
    pos, q, field = _particle_inputs(case, seed)
    shape, lengths = (case["nz"], case["ny"], case["nx"]), _lengths(case)
    dev = pos.device
    i0, w = [], []
    for d, n in enumerate((shape[2], shape[1], shape[0])):
        s = pos[:, d] * (n / lengths[d]) - 0.5
        fl = torch.floor(s)
        i0.append(torch.remainder(fl.to(torch.int64), n))
        w.append((1.0 - (s - fl), s - fl))
    at = torch.zeros_like(q)
    grid = torch.zeros(field.numel(), dtype=torch.float64, device=dev)
    cell = lengths[0] * lengths[1] * lengths[2] / field.numel()
    for c in range(8):
        a, b, e = c & 1, (c >> 1) & 1, c >> 2
        flat = ((torch.remainder(i0[2] + e, shape[0]) * shape[1] + torch.remainder(i0[1] + b, shape[1])) * shape[2]
                + torch.remainder(i0[0] + a, shape[2]))
        wt = w[0][a] * w[1][b] * w[2][e]
        at += wt * field.reshape(-1)[flat]
        grid.index_add_(0, flat, q * wt / cell)
    return {"at": at, "grid": grid.reshape(shape)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "particles":
        return _exact_particles(case, seed)
    if kind == "serve":
        ps = []
        for k, c in enumerate(_requests(case, seed)):
            rho, b, _ = _solve_fields(c, 1000 * seed + k)
            ps.append(_exact_solve(rho, b, _lengths(c), c["coef"], False))
        return {"p": ps, "status": None}
    lengths = _lengths(case)
    if kind == "project":
        m, div = _momentum(case, seed)
        rho = _density(case, _gen(seed, 1))
        op = _Operator(rho, lengths, case["coef"], case["walls"])
        rhs = -div
        for ax in range(3):
            u = op.beta[ax] * m[2 - ax] * op.inv_h[ax]
            rhs = rhs + (u - torch.roll(u, 1, dims=ax))
        p = _exact_solve(rho, rhs / C_DT, lengths, case["coef"], case["walls"])
        new = []
        for d in range(3):
            ax = 2 - d
            grad = (torch.roll(p, -1, dims=ax) - p) * op.inv_h[ax]
            if ax == 2 and case["walls"]:
                grad[:, :, -1] = 0.0
            new.append(m[d] - C_DT * grad)
        return {"m": new, "p": p, "status": None}
    rho, b, _ = _solve_fields(case, seed)
    smooth = case["density"] != "particles"
    return {"p": _exact_solve(rho, b, lengths, case["coef"], case["walls"], smooth), "status": None}
