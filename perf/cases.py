"""Timed cases of the hybrid lattice-Boltzmann library: whole calls through its
public Python entry points, on seeded flows of the kinds and sizes that the
studies, the learned closure, the tests and the benchmark run.

A case is a dict of plain values; ``path`` names what it runs:

* ``solver``   one domain: ``Solver.step`` and ``Solver.moments``
               (``populations``, ``totals`` and ``status`` where asked for)
* ``batch``    independent domains: ``BatchSolver.step`` on the shape that
               ``autotune`` picked, ``BatchSolver.moments_cat``
* ``data``     training data of the learned closure: fine batched steps,
               moments and their restriction to the coarse grid
* ``closure``  corrected coarse steps: ``BatchSolver.closure_step``
* ``train``    one Adam step of the closure network on a minibatch

``exact`` is the same computation in 64-bit torch, written from the method
(moments, upwind correction, regularised collision, streaming, entropy
update) on ghost-padded fields, without the library.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2002_03644_amd import CNN, BatchSolver, Params, Solver, restrict

CS2 = 1.0 / 3.0
GAMMA = 1.4
PRANDTL = 0.71
THETA = 240.0 / 1183.0           # temperature of the paper's air at 300 K
SGN_EPS = 1e-12
CX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
CY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
FIELDS = ("rho", "ux", "uy", "s", "theta")
COARSE = ("rho", "ux", "uy", "theta")


def device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


# ------------------------------------------------------------------- cases
def listed():
    return [
        # the headline run: decaying turbulence on the benchmark's grid
        solver("turbulence_8192_f32", "turbulence", 8192, 8192, "f32", steps=20),
        # an ordinary production run on a grid that is no multiple of any tile
        solver("turbulence_1500x1100_f32", "turbulence", 1500, 1100, "f32", steps=20,
               sigma=0.3),
        # a small study: the convected vortex, its state checked after each leg
        solver("vortex_200_f32", "vortex", 200, 200, "f32", steps=50, sigma=0.5, mu=1e-4,
               check=True),
        # the double-precision reference run that the single-precision one is
        # judged by, its populations kept
        solver("turbulence_2048_f64", "turbulence", 2048, 2048, "f64", steps=10,
               populations=True),
        # a shock tube between open ends, viscous heat by finite differences
        solver("tube_2048x512_f32", "tube", 2048, 512, "f32", steps=20, sigma=0.4, bc_x=1,
               phi_fd=True),
        # the paper's thermal Couette channel: the smallest domain, with walls
        solver("couette_2x100_f64", "channel", 2, 100, "f64", steps=50, sigma=0.9, mu=0.1,
               bc_y=2),
        # the coarse runs of the learned closure's evaluation
        batch("batch_8x256_f32", "turbulence", 8, 256, 256, "f32", steps=50, mu=1e-3),
        # a batch of uneven domains
        batch("batch_48_mixed_f32", "mixed", 48, 64, 1024, "f32", steps=20, mu=1e-3),
        # one Mach number of the sigma map: blends and the original model
        batch("batch_12x200_f64", "map", 12, 200, 200, "f64", steps=50, mu=1.5e-6),
        # one coarse step of the closure's training data
        dict(name="data_16x1024", path="data", domains=16, n=1024, factor=4, mu=4e-3),
        # corrected coarse steps up to the next checkpoint of an evaluation
        dict(name="closure_8x256", path="closure", domains=8, n=256, cycles=5, every=10, mu=1e-3),
        # a training step of the closure network, minibatch of the training driver
        dict(name="train_32x256", path="train", batch=32, pool=48, ny=256, nx=256),
    ]


def solver(name, flow, nx, ny, dtype, steps, sigma=0.0, mu=1e-3, bc_x=0, bc_y=0, phi_fd=False,
           original=False, precise=False, populations=False, check=False):
    c = dict(path="solver", flow=flow, nx=nx, ny=ny, dtype=dtype, steps=steps, sigma=sigma, mu=mu,
             bc_x=bc_x, bc_y=bc_y, phi_fd=phi_fd, original=original, precise=precise,
             populations=populations, check=check)
    return dict(c, name=name) if name else c


def batch(name, flow, domains, nmin, nmax, dtype, steps, mu, sizes=1):
    c = dict(path="batch", flow=flow, domains=domains, nmin=nmin, nmax=nmax, dtype=dtype,
             steps=steps, mu=mu, sizes=sizes)
    return dict(c, name=name) if name else c


def draw(rng: random.Random):
    def logint(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    def steps(nodes, most=50):
        return max(2, min(most, int(4e8 / nodes))) + rng.randint(0, 1)

    kind = rng.choice(("turbulence", "turbulence", "turbulence", "vortex", "double", "tube",
                       "channel", "batch", "batch", "map", "data", "closure", "train"))
    if kind == "turbulence":
        nx, ny = logint(128, 8000), logint(128, 8000)
        return solver("", "turbulence", nx, ny, "f32", steps(nx * ny),
                      sigma=round(rng.uniform(0.0, 0.5), 2))
    if kind == "vortex":
        n = logint(64, 900)
        dtype = rng.choice(("f32", "f32", "f64"))
        return solver("", "vortex", n, n + rng.randint(0, 9), dtype, steps(n * n),
                      sigma=rng.choice((0.0, 0.3, 0.5)), mu=1e-4,
                      original=rng.random() < 0.2, check=True)
    if kind == "double":
        nx, ny = logint(128, 3000), logint(128, 3000)
        return solver("", "turbulence", nx, ny, "f64", min(20, steps(nx * ny)),
                      sigma=round(rng.uniform(0.0, 0.5), 2), populations=rng.random() < 0.5)
    if kind == "tube":
        nx, ny = logint(400, 4096), logint(2, 1024)
        return solver("", "tube", nx, ny, rng.choice(("f32", "f64")), steps(nx * ny), sigma=0.4,
                      bc_x=1, bc_y=rng.randint(0, 1), phi_fd=True)
    if kind == "channel":
        nx, ny = logint(2, 512), logint(32, 512)
        dtype = rng.choice(("f32", "f64"))
        return solver("", "channel", nx, ny, dtype, steps(nx * ny), sigma=0.9, mu=0.1, bc_y=2,
                      precise=dtype == "f32")
    if kind == "batch":
        if rng.random() < 0.5:
            n = logint(64, 768)
            return batch("", "turbulence", rng.randint(2, 16), n, n, "f32", rng.randint(10, 50),
                         1e-3)
        return batch("", "mixed", rng.randint(8, 64), 64, logint(256, 1024), "f32",
                     rng.randint(5, 20), 1e-3, sizes=rng.randint(2, 9999))
    if kind == "map":
        n = logint(64, 300)
        return batch("", "map", 12, n, n, rng.choice(("f32", "f64", "f64")), rng.randint(10, 50),
                     1.5e-6)
    if kind == "data":
        factor = rng.choice((2, 4))
        return dict(path="data", domains=rng.randint(2, 16), n=32 * factor * rng.randint(2, 8),
                    factor=factor, mu=4e-3)
    if kind == "closure":
        return dict(path="closure", domains=rng.randint(2, 16), n=64 * rng.randint(1, 5),
                    cycles=rng.randint(2, 6), every=rng.choice((1, 2, 5, 10)), mu=1e-3)
    return dict(path="train", batch=rng.randint(4, 32), pool=48, ny=4 * rng.randint(8, 64),
                nx=32 * rng.randint(1, 8))


# ------------------------------------------------------------------- flows
def generator(seed):
    g = torch.Generator(device=device())
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFF)
    return g


def uniform(g, *shape):
    return torch.rand(*shape, generator=g, device=device(), dtype=torch.float64)


def spread(rows, g, ny, nx):
    """Smooth seeded perturbation of order one."""
    y = torch.arange(ny, device=device(), dtype=torch.float64)[:, None] / ny
    x = torch.arange(nx, device=device(), dtype=torch.float64)[None, :] / nx
    out = torch.zeros(ny, nx, device=device(), dtype=torch.float64)
    a = uniform(g, rows, 2).cpu()
    for k in range(rows):
        out += (2 * float(a[k, 0]) - 1) * torch.sin(
            2 * math.pi * (float(1 + k % 3) * x + float(1 + (k + 1) % 3) * y + float(a[k, 1])))
    return out


def theta_for(mach_max, cfl=0.7):
    return min(THETA, (cfl / (1.0 + mach_max)) ** 2 / (GAMMA * CS2))


def turbulence(nx, ny, mach, theta, g):
    """Random-phase solenoidal velocity, E(k) ~ k^4 exp(-2 (k / kp)^2)."""
    kx = torch.fft.rfftfreq(nx, d=1.0 / nx, device=device(), dtype=torch.float64)[None, :]
    ky = torch.fft.fftfreq(ny, d=1.0 / ny, device=device(), dtype=torch.float64)[:, None]
    kp = min(8.0, min(nx, ny) / 16.0)
    K = torch.sqrt(kx * kx + ky * ky)
    K[0, 0] = 1.0
    amp = torch.sqrt(K * torch.exp(-2.0 * (K / kp) ** 2))
    amp[0, 0] = 0.0
    psi = torch.polar(amp, 2 * math.pi * uniform(g, ny, nx // 2 + 1))
    del K, amp
    u = torch.fft.irfft2(1j * (ky / ny) * psi, s=(ny, nx))
    v = torch.fft.irfft2(-1j * (kx / nx) * psi, s=(ny, nx))
    del psi
    scale = mach * math.sqrt(GAMMA * CS2 * theta) / float((u * u + v * v).mean().sqrt())
    return torch.ones_like(u), u * scale, v * scale, torch.full_like(u, theta)


def vortex(nx, ny, mach, mach_v, theta, g, angle=0.3):
    """Isentropic vortex in a uniform stream, at a seeded place."""
    a = uniform(g, 2).cpu()
    R = min(nx, ny) / 12.0
    x = torch.arange(nx, device=device(), dtype=torch.float64)[None, :]
    y = torch.arange(ny, device=device(), dtype=torch.float64)[:, None]
    dx = (x - nx * float(a[0]) + nx / 2) % nx - nx / 2
    dy = (y - ny * float(a[1]) + ny / 2) % ny - ny / 2
    r2 = (dx * dx + dy * dy) / (R * R)
    c = math.sqrt(GAMMA * CS2 * theta)
    w = c * mach_v * torch.exp((1.0 - r2) / 2.0) / R
    t = 1.0 - 0.5 * (GAMMA - 1.0) * mach_v ** 2 * torch.exp(1.0 - r2)
    return (t ** (1.0 / (GAMMA - 1.0)), mach * c * math.cos(angle) - w * dy,
            mach * c * math.sin(angle) + w * dx, theta * t)


def tube(nx, ny, g):
    """Two states of one temperature in a slow oblique stream, the jump
    smoothed over a few nodes, with a weak seeded perturbation."""
    x = torch.arange(nx, device=device(), dtype=torch.float64)[None, :]
    one = torch.ones(ny, nx, device=device(), dtype=torch.float64)
    p = 1e-3 * spread(4, g, ny, nx)
    rho = (2.0 - torch.tanh((x - nx / 2) / 3.0)) * one * (1.0 + p)
    return rho, (0.05 + p) * one, (0.02 - p) * one, THETA * one * (1.0 + p)


def channel(nx, ny, theta, U, g):
    """Sheared channel between walls with a weak seeded perturbation."""
    y = torch.arange(ny, device=device(), dtype=torch.float64)[:, None] / (ny - 1)
    one = torch.ones(ny, nx, device=device(), dtype=torch.float64)
    p = 1e-3 * spread(4, g, ny, nx) * torch.sin(math.pi * y)
    return one * (1.0 + p), (U * y + 0.1 * p) * one, (0.02 * p) * one, theta * one * (1.0 + p)


WALL_THETA = 0.2


def wall_speed():
    return 0.8 * math.sqrt(GAMMA * CS2 * WALL_THETA)


def domains_of(case, seed):
    """[(params, (rho, ux, uy, theta))] of a case, fields in its precision."""
    g = generator(seed)
    dtype = case.get("dtype", "f32")
    td = torch.float64 if dtype == "f64" else torch.float32
    out = []

    def add(p, f):
        out.append((Params(dtype=dtype, gamma=GAMMA, prandtl=PRANDTL, mu=case["mu"],
                           sgn_eps=SGN_EPS, **p), tuple(a.to(td).contiguous() for a in f)))

    if case["path"] == "solver":
        nx, ny, flow = case["nx"], case["ny"], case["flow"]
        model = dict(e1_centred=True, e2_off=True, feq_order=3) if case["original"] else {}
        p = dict(nx=nx, ny=ny, sigma=case["sigma"], theta_ref=THETA,
                 bc_x=("periodic", "extrapolate")[case["bc_x"]],
                 bc_y=("periodic", "extrapolate", "wall")[case["bc_y"]],
                 phi_mode="fd" if case["phi_fd"] else "lbm", precise_theta=case["precise"],
                 **model)
        if flow == "turbulence":
            f = turbulence(nx, ny, 0.4, THETA, g)
        elif flow == "vortex":
            f = vortex(nx, ny, 0.5, 0.05, THETA, g)
        elif flow == "tube":
            f = tube(nx, ny, g)
        else:
            f = channel(nx, ny, WALL_THETA, wall_speed(), g)
            p.update(theta_ref=WALL_THETA, wall_theta=WALL_THETA, wall_ux_hi=wall_speed())
        add(p, f)
    elif case["path"] == "batch" and case["flow"] == "map":
        n, c = case["nmin"], case["domains"]
        f = vortex(n, n, 0.6, 0.06, THETA, g)
        for k in range(c):
            model = dict(e1_centred=True, e2_off=True, feq_order=3) if k == c - 1 else {}
            add(dict(nx=n, ny=n, theta_ref=THETA, sigma=0.0 if model else 0.3 * k / c, **model), f)
    else:
        r = random.Random(case.get("sizes", 0))
        for k in range(case["domains"]):
            lo, hi = case.get("nmin", case.get("n")), case.get("nmax", case.get("n"))
            n = int(round(math.exp(r.uniform(math.log(lo), math.log(hi)))))
            mach = r.uniform(0.25, 0.4)
            th = theta_for(3.0 * mach)
            if case.get("flow") == "mixed" and r.random() < 0.5:
                f = vortex(n, n, 0.5 + mach, 0.05, th, g, angle=6.0 * mach)
            else:
                f = turbulence(n, n, mach, th, g)
            add(dict(nx=n, ny=n, sigma=0.0, theta_ref=th), f)
    return out


# ----------------------------------------------------------------- network
def network(g, scale):
    """Seeded parameters in the canonical order and the standardisation."""
    def layer(cin, cout, gain):
        w = torch.randn(9, cin, cout, generator=g, device=device(), dtype=torch.float64)
        b = torch.randn(cout, generator=g, device=device(), dtype=torch.float64)
        return [(w * gain * math.sqrt(2.0 / (9 * cin))).float(), (0.05 * b).float()]
    layers = layer(4, 32, 1.0) + layer(32, 32, 1.0) + layer(32, 4, 0.5)
    norm = [(1.0, 0.0, 0.0, 0.17), (0.02, 0.06, 0.06, 0.02), (0.0, 0.0, 0.0, 0.0), scale]
    return torch.cat([a.reshape(-1) for a in layers]), norm


def smooth_samples(g, count, ny, nx, mean, std):
    """[count][4][ny][nx] float32 low-pass fields of given channel moments."""
    z = torch.fft.rfft2(torch.randn(count, 4, ny, nx, generator=g, device=device()))
    kx = torch.fft.rfftfreq(nx, d=1.0 / nx, device=device())[None, :]
    ky = torch.fft.fftfreq(ny, d=1.0 / ny, device=device())[:, None]
    a = torch.fft.irfft2(z * torch.exp(-(kx * kx + ky * ky) / 200.0), s=(ny, nx))
    a = a / a.std(dim=(2, 3), keepdim=True)
    shape = (1, 4, 1, 1)
    return (a * torch.tensor(std, device=device()).view(shape)
            + torch.tensor(mean, device=device()).view(shape)).contiguous()


def train_inputs(case, seed):
    g = generator(seed)
    params, norm = network(g, (2e-4, 1e-3, 1e-3, 2e-4))
    x = smooth_samples(g, case["pool"], case["ny"], case["nx"], norm[0], norm[1])
    t = smooth_samples(g, case["pool"], case["ny"], case["nx"], norm[2], norm[3])
    idx = torch.randperm(case["pool"], generator=g, device=device())[:case["batch"]]
    return params, norm, x, t, idx.to(torch.int32)


# --------------------------------------------------------- prepare and run
def prepare(case, seed):
    path = case["path"]
    st = {"case": case}
    if path == "train":
        params, norm, st["x"], st["t"], st["idx"] = train_inputs(case, seed)
        st["net"] = CNN(case["batch"], case["ny"], case["nx"], params)
        st["net"].set_norm(*norm)
        st["loss"] = torch.zeros(1, device=device())
        return st
    doms = domains_of(case, seed)
    if path == "solver":
        p, (rho, ux, uy, theta) = doms[0]
        st["S"] = Solver(p, rho, ux, uy, theta=theta)
        return st
    B = st["B"] = BatchSolver([p for p, _ in doms], [f for _, f in doms])
    if path == "batch":
        B.autotune(steps=10)
    elif path == "data":
        n, c = case["n"], case["domains"]
        st["fine"] = torch.empty(4, c * n * n, dtype=torch.float32, device=device())
    else:
        B.set_tile(32, 16, kernel="tiles")
        st["start"] = B.save_state()
        params, norm = network(generator(seed + 1), (2e-5, 1e-4, 1e-4, 1e-5))
        st["net"] = CNN(case["domains"], case["n"], case["n"], params)
        st["net"].set_norm(*norm)
        st["net"].set_output_clip(4.0)
    return st


def run(st):
    case = st["case"]
    path = case["path"]
    if path == "solver":
        S = st["S"]
        S.step(case["steps"])
        out = S.moments()
        if case["populations"]:
            out["populations"] = S.populations()
        if case["check"]:
            out["code"], out["cfl"] = S.status()
            out["totals"] = torch.tensor(S.totals(), dtype=S.p.torch_dtype)
        return out
    if path == "batch":
        return st["B"].step(case["steps"], graph=True).moments_cat()
    if path == "data":
        B, n, c = st["B"], case["n"], case["domains"]
        B.step(case["factor"], graph=True)
        cat = B.moments_cat(out=st["fine"], keys=COARSE)
        f = [cat[k].view(c, n, n) for k in COARSE]
        return {"fine": st["fine"], "coarse": restrict(*f, case["factor"], batch=c)}
    if path == "closure":
        B = st["B"]
        B.load_state(st["start"])
        B.closure_step(st["net"], case["cycles"], every=case["every"], conserve=True, graph=True)
        return B.moments_cat(keys=COARSE)
    net = st["net"]
    net.train_step(st["x"], st["t"], 1e-4, idx=st["idx"], loss=st["loss"])
    return {"loss": st["loss"], "grads": net.grads()}


# -------------------------------------------------------------------- work
UPDATE_FLOPS = 300      # of one lattice update: collision, streaming, entropy
NET_MACS = 9 * (4 * 32 + 32 * 32 + 32 * 4)


def nodes_of(case):
    if case["path"] == "solver":
        return case["nx"] * case["ny"]
    if case["path"] == "batch" and case["flow"] != "map":
        r, n = random.Random(case["sizes"]), 0
        for _ in range(case["domains"]):
            m = int(round(math.exp(r.uniform(math.log(case["nmin"]), math.log(case["nmax"])))))
            r.uniform(0.25, 0.4)
            if case["flow"] == "mixed":
                r.random()
            n += m * m
        return n
    m = case.get("n", case.get("nmin"))
    return case["domains"] * m * m


def work(case):
    """The state read and written once in a pass and its outputs written once;
    the arithmetic of its lattice updates and network evaluations."""
    if case["path"] == "train":
        px = case["batch"] * case["ny"] * case["nx"]
        return {"bytes": 4 * 8 * px, "flops": 2 * (3 * NET_MACS - 9 * 4 * 32) * px}
    n = nodes_of(case)
    es = 8 if case.get("dtype") == "f64" else 4
    if case["path"] == "data":
        return {"bytes": es * n * (24 + 4 / case["factor"] ** 2),
                "flops": UPDATE_FLOPS * case["factor"] * n}
    if case["path"] == "closure":
        return {"bytes": es * n * 24, "flops": n * case["cycles"] * (
            UPDATE_FLOPS * case["every"] + 2 * NET_MACS)}
    out = 5 + (9 if case.get("populations") else 0)
    return {"bytes": es * n * (20 + out), "flops": UPDATE_FLOPS * case["steps"] * n}


# ------------------------------------------------- the method in 64-bit torch
def ghosts(a, bc_x, bc_y):
    """Two ghost nodes on every side: wrapped (0) or clamped."""
    def index(n, bc):
        i = torch.arange(-2, n + 2, device=a.device)
        return i % n if bc == 0 else i.clamp(0, n - 1)
    return a[..., index(a.shape[-2], bc_y), :][..., index(a.shape[-1], bc_x)]


def at(a, dx, dy, r):
    """The field seen from neighbour (dx, dy), cut by r on every side."""
    H, W = a.shape[-2:]
    return a[..., r + dy:H - r + dy, r + dx:W - r + dx]


class Exact:
    """One domain: absolute populations F[9] and entropy s in 64 bits."""

    def __init__(self, p: Params, fields):
        self.p = p
        self.cv = CS2 / (p.gamma - 1.0)
        self.lam = p.mu * p.gamma * self.cv / p.prandtl
        self.bcx = 0 if p.bc_x == "periodic" else 1
        self.bcy = 0 if p.bc_y == "periodic" else 1
        rho, ux, uy, th = (a.double() for a in fields)
        self.s = self.cv * (torch.log(th) - (p.gamma - 1.0) * torch.log(rho))
        pad = [ghosts(a, self.bcx, self.bcy) for a in (rho, ux, uy, th)]
        m = self.collide(*pad, None, first=True)
        self.F = [at(f, 0, 0, 1).clone() for f in m["f"]]
        self.walls()

    def collide(self, rho, ux, uy, th, P2, first=False):
        """Populations on the ring of radius one: after the collision, or (first)
        the consistent initial ones with psi taken off."""
        p, e = self.p, SGN_EPS
        gx, gy = rho * ux * (1 - th - ux * ux), rho * uy * (1 - th - uy * uy)
        dxux, dxuy = [0.5 * (at(q, 1, 0, 1) - at(q, -1, 0, 1)) for q in (ux, uy)]
        dyux, dyuy = [0.5 * (at(q, 0, 1, 1) - at(q, 0, -1, 1)) for q in (ux, uy)]
        r, u, v, t = (at(q, 0, 0, 1) for q in (rho, ux, uy, th))

        def upwind(q, w, dx, dy):
            c, hi, lo = at(q, 0, 0, 1), at(q, dx, dy, 1), at(q, -dx, -dy, 1)
            mid = 0.5 * (hi - lo)
            if p.e1_centred:
                return mid
            return torch.where(w > e, c - lo, torch.where(w < -e, hi - c, mid))

        pr = r * CS2 * t
        e2 = 0.0 if p.e2_off else pr * (2.0 - p.gamma) * (dxux + dyuy)
        Ex, Ey = upwind(gx, u, 1, 0) + e2, upwind(gy, v, 0, 1) + e2
        del gx, gy
        taup = p.mu + 0.5 * pr                       # (tau + 1/2) p
        fxx, fxy = -taup * (dxux - dyuy), -taup * (dyux + dxuy)
        keep = 1.0 - pr / taup
        if first:
            axx, ayy, axy, keep, half = fxx, -fxx, fxy, 1.0, -0.5
        else:
            sg = torch.full((r.shape[-2], 1), float(p.sigma), device=r.device, dtype=r.dtype)
            if p.bc_y == "wall":
                sg[1], sg[-2] = 1.0, 1.0
            pxx, pyy, pxy = (at(q, 0, 0, 1) for q in P2)
            axx = sg * (pxx - pr - r * u * u + 0.5 * Ex) + (1 - sg) * fxx
            ayy = sg * (pyy - pr - r * v * v + 0.5 * Ey) - (1 - sg) * fxx
            axy = sg * (pxy - r * u * v) + (1 - sg) * fxy
            half = 0.5
        if p.phi_mode == "fd":
            phi = p.mu * ((dxux - dyuy) ** 2 + (dyux + dxuy) ** 2)
        else:
            phi = -(p.mu / taup) * (axx * dxux + axy * (dyux + dxuy) + ayy * dyuy)
        del dxux, dxuy, dyux, dyuy, fxx, fxy
        axx, ayy, axy = keep * axx, keep * ayy, keep * axy
        c = CS2 * (t - 1.0)
        A = {"xx": r * u * u + r * c + axx + half * Ex, "yy": r * v * v + r * c + ayy + half * Ey,
             "xy": r * u * v + axy}
        bxxy, bxyy = v * axx + 2 * u * axy, u * ayy + 2 * v * axy
        A["xxy"] = r * u * u * v + r * c * v + bxxy
        A["xyy"] = r * u * v * v + r * c * u + bxyy
        A["xxyy"] = (torch.zeros_like(r) if p.feq_order == 3 else
                     r * u * u * v * v + r * c * (u * u + v * v) + r * c * c
                     + 2 * (u * bxyy + v * bxxy) + (c - u * u) * ayy + (c - v * v) * axx
                     - 4 * u * v * axy)
        f = populations(r, r * u, r * v, A)
        return {"f": f, "phi": phi, "rho": r, "u": u, "v": v, "th": t}

    def theta(self, rho, s):
        return torch.exp(s / self.cv + (self.p.gamma - 1.0) * torch.log(rho))

    def step(self):
        F = [ghosts(f, self.bcx, self.bcy) for f in self.F]
        self.F = None
        s = ghosts(self.s, self.bcx, self.bcy)
        rho, jx, jy = moments(F)
        ux, uy = jx / rho, jy / rho
        th = self.theta(rho, s)
        P2 = (sum(f for k, f in enumerate(F) if CX[k]), sum(f for k, f in enumerate(F) if CY[k]),
              F[5] - F[6] + F[7] - F[8])
        del F, jx, jy
        m = self.collide(rho, ux, uy, th, P2)
        del P2, rho, ux, uy
        u, v = at(m["u"], 0, 0, 1), at(m["v"], 0, 0, 1)
        lap = (at(th, 1, 0, 2) + at(th, -1, 0, 2) + at(th, 0, 1, 2) + at(th, 0, -1, 2)
               - 4 * at(th, 0, 0, 2))
        adv = advect(u, *(at(s, k, 0, 2) for k in range(-2, 3)))
        adv = adv + advect(v, *(at(s, 0, k, 2) for k in range(-2, 3)))
        heat = (self.lam * lap + at(m["phi"], 0, 0, 1)) / at(m["rho"] * m["th"], 0, 0, 1)
        self.s = at(s, 0, 0, 2) - adv + heat
        self.F = [at(m["f"][k], -CX[k], -CY[k], 1).clone() for k in range(9)]
        self.walls()

    def walls(self):
        """Isothermal moving walls on the first and last rows."""
        p = self.p
        if p.bc_y != "wall":
            return
        for row, d, U, inward in ((0, 1, p.wall_ux_lo, (4, 7, 8)), (-1, -1, p.wall_ux_hi,
                                                                     (2, 5, 6))):
            F = self.F
            rho = sum(F[k][row] for k in (0, 1, 3)) + 2 * sum(F[k][row] for k in inward)
            n1, n2 = (1, 2) if d > 0 else (-2, -3)
            w = []
            for n in (n1, n2):
                r, jx, jy = moments([f[n] for f in F])
                w.append((jx / r, jy / r))
            dux = 0.5 * d * (4 * w[0][0] - w[1][0] - 3 * U)
            duy = 0.5 * d * (4 * w[0][1] - w[1][1])
            th, u = p.wall_theta, U * torch.ones_like(rho)
            taup = p.mu + 0.5 * rho * CS2 * th
            axx, ayy, axy = taup * duy, -taup * duy, -taup * dux
            c = CS2 * (th - 1.0)
            A = {"xx": rho * u * u + rho * c + axx, "yy": rho * c + ayy, "xy": axy,
                 "xxy": 2 * u * axy, "xyy": rho * c * u + u * ayy}
            A["xxyy"] = (torch.zeros_like(rho) if p.feq_order == 3 else
                         rho * c * u * u + rho * c * c + 2 * u * u * ayy
                         + (c - u * u) * ayy + c * axx)
            for k, f in enumerate(populations(rho, rho * u, 0 * rho, A)):
                F[k][row] = f
            self.s[row] = self.cv * (math.log(th) - (p.gamma - 1.0) * torch.log(rho))

    def fields(self):
        rho, jx, jy = moments(self.F)
        return {"rho": rho, "ux": jx / rho, "uy": jy / rho, "s": self.s,
                "theta": self.theta(rho, self.s)}

    def correct(self, delta):
        """The network's increments with the domain's mass and momentum kept."""
        m = self.fields()
        r, u, v, t = (m[k] for k in COARSE)
        r1, u1, v1 = r + delta[0], u + delta[1], v + delta[2]
        r2 = r1 - delta[0].mean()
        jx, jy = r2 * u1, r2 * v1
        u2 = (jx - (jx - r * u).mean()) / r2
        v2 = (jy - (jy - r * v).mean()) / r2
        t2 = t + delta[3]
        for k, (a, b) in enumerate(zip(equilibrium(r2, u2, v2, t2), equilibrium(r, u, v, t))):
            self.F[k] = self.F[k] + a - b
        self.s = self.s + self.cv * (torch.log(t2 / t)
                                     - (self.p.gamma - 1.0) * torch.log(r2 / r))


def moments(F):
    rho = sum(F)
    return rho, sum(CX[k] * F[k] for k in range(9) if CX[k]), sum(
        CY[k] * F[k] for k in range(9) if CY[k])


def populations(A0, Ax, Ay, A):
    """Sum of the Hermite polynomials of each lattice velocity."""
    out = []
    for k in range(9):
        cx, cy = CX[k], CY[k]
        w = (4 / 9, 1 / 9, 1 / 36)[abs(cx) + abs(cy)]
        hx, hy = cx * cx - CS2, cy * cy - CS2
        f = A0 + (hx * A["xx"] + hy * A["yy"]) * 4.5 + (hx * hy * 20.25) * A["xxyy"]
        if cx:
            f = f + 3.0 * cx * Ax + 13.5 * cx * hy * A["xyy"]
        if cy:
            f = f + 3.0 * cy * Ay + 13.5 * cy * hx * A["xxy"]
        if cx and cy:
            f = f + 9.0 * cx * cy * A["xy"]
        out.append(w * f)
    return out


def equilibrium(r, u, v, t):
    rc = r * CS2 * (t - 1.0)
    c = CS2 * (t - 1.0)
    return populations(r, r * u, r * v, {
        "xx": r * u * u + rc, "yy": r * v * v + rc, "xy": r * u * v, "xxy": r * u * u * v + rc * v,
        "xyy": r * u * v * v + rc * u,
        "xxyy": r * u * u * v * v + rc * (u * u + v * v) + rc * c})


def limited(a, b):
    """van Albada slope."""
    den = a * a + b * b
    ok = (a * b > 0) & (den > 1e-300)
    return torch.where(ok, a * b * (a + b) / torch.where(ok, den, torch.ones_like(den)),
                       torch.zeros_like(a))


def advect(u, m2, m1, c, p1, p2):
    """Upwind MUSCL u ds/dx."""
    here = limited(c - m1, p1 - c)
    back = (c - m1) + 0.5 * (here - limited(m1 - m2, c - m1))
    fore = (p1 - c) + 0.5 * (here - limited(p2 - p1, p1 - c))
    return torch.where(u > 0, u * back, u * fore)


def forward(params, norm, x, leaves=None):
    """The network in 64 bits: raw increments of x [B][4][ny][nx]."""
    if leaves is None:
        leaves = split(params.double())
    mean, std, om, os_ = (torch.tensor(v, device=x.device, dtype=torch.float32).double()
                          for v in norm)
    h = ((x.double().permute(0, 2, 3, 1) - mean) / std).contiguous()
    for k in range(3):
        w, b = leaves[2 * k], leaves[2 * k + 1]
        acc = b
        for t in range(9):
            q = torch.roll(h, (1 - t // 3, 1 - t % 3), (1, 2))
            acc = acc + (q.reshape(-1, q.shape[-1]) @ w[t]).view(*q.shape[:3], -1)
        h = torch.relu(acc) if k < 2 else acc
    return h, om, os_


def split(flat):
    out, at_ = [], 0
    for cin, cout in ((4, 32), (32, 32), (32, 4)):
        out.append(flat[at_:at_ + 9 * cin * cout].view(9, cin, cout))
        at_ += 9 * cin * cout
        out.append(flat[at_:at_ + cout])
        at_ += cout
    return out


def exact(case, seed):
    path = case["path"]
    if path == "train":
        params, norm, x, t, idx = train_inputs(case, seed)
        x, t = x[idx.long()], t[idx.long()]
        leaves = [a.clone().requires_grad_(True) for a in split(params.double())]
        total, loss = x.shape[0] * x.shape[2] * x.shape[3] * 4, 0.0
        for k in range(x.shape[0]):                  # one sample at a time: memory
            h, om, os_ = forward(None, norm, x[k:k + 1], leaves)
            want = (t[k:k + 1].double().permute(0, 2, 3, 1) - om) / os_
            part = (h - want).square().sum() / total
            part.backward()
            loss += float(part.detach())
        return {"loss": torch.tensor([loss], dtype=torch.float64),
                "grads": torch.cat([a.grad.reshape(-1) for a in leaves])}
    doms = [Exact(p, f) for p, f in domains_of(case, seed)]
    if path == "closure":
        params, norm = network(generator(seed + 1), (2e-5, 1e-4, 1e-4, 1e-5))
        for _ in range(case["cycles"]):
            for D in doms:
                for _ in range(case["every"]):
                    D.step()
                m = D.fields()
                h, om, os_ = forward(params, norm, torch.stack([m[k] for k in COARSE])[None])
                D.correct((h.clamp(-4.0, 4.0) * os_ + om)[0].permute(2, 0, 1))
    else:
        for D in doms:
            for _ in range(case.get("steps", case.get("factor"))):
                D.step()
    if path == "solver":
        D = doms[0]
        out = D.fields()
        if case["populations"]:
            out["populations"] = torch.stack(D.F)
        if case["check"]:
            r, u, v, t = (out[k] for k in COARSE)
            ke = u * u + v * v
            out["code"] = None
            out["cfl"] = float((ke.sqrt() + torch.sqrt(GAMMA * CS2 * t)).max())
            out["totals"] = torch.stack([r.sum(), (r * u).sum(), (r * v).sum(),
                                         (r * D.cv * t + 0.5 * r * ke).sum()]).cpu()
        return out
    all_ = [D.fields() for D in doms]
    if path == "data":
        n, f = case["n"], case["factor"]
        fine = [torch.stack([m[k] for m in all_]) for k in COARSE]
        cells = [a.view(-1, n // f, f, n // f, f) for a in fine]
        mass = cells[0].sum((2, 4))
        coarse = [mass / (f * f)] + [(cells[0] * q).sum((2, 4)) / mass for q in cells[1:]]
        return {"fine": torch.stack([a.reshape(-1) for a in fine]),
                "coarse": torch.stack(coarse, dim=1)}
    keys = COARSE if path == "closure" else FIELDS
    return {k: torch.cat([m[k].reshape(-1) for m in all_]) for k in keys}
