"""What the framework is timed on: calls that its users make, through the public
entry points, over the range of grids, particle numbers and options in use.

Kinds of case
  slices      a run of xi-slices from a saved state (particles, fields, xi, dxi),
              as a program does that restarts from a checkpoint: set_state, run,
              get_state.  Linear or blowout plasma, the Boris-like or a
              Runge-Kutta pusher, the FP64 or the mixed form.
  adjoint     a taped run and the reverse sweep: the gradient of a probe and of
              a linear functional of the final particles with respect to the
              driver's radial bins and the initial particles.
  driver      one step of the time loop with driver macroparticles.
  laser       one step of the time loop with a laser envelope.
  poisson,    one multigrid solve (1 or 2 right-hand sides), the solver of the
  helmholtz   slice on its own.
  noalloc     the solve that allocates nothing, a fixed number of V-cycles.
  nonuniform  the multigrid solve on a non-uniform grid.

Inputs are made from the seed on the GPU; exact() is the same computation in
plain torch in 64 bits (dense sine transforms, Krylov iterations, autograd).
"""
import math

import numpy as np
import torch

from paper_2012_00881_amd import Simulation, mg_solve_noalloc

F64 = torch.float64


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


# ------------------------------------------------------------------ cases --

def listed():
    return [
        # the linear wake on the smallest configured grid: latency and launches
        dict(name="slices_64_linear", kind="slices", n=64, half_width=6.0, ppc=1, slices=8,
             regime="linear", precision="fp64", pusher="boris", adaptive=False, dxi0=0.0625),
        # the blowout workload at 256^2 with adaptive steps
        dict(name="slices_256_blowout", kind="slices", n=256, half_width=8.0, ppc=2, slices=16,
             regime="blowout", precision="fp64", pusher="boris", adaptive=True, dxi0=0.02),
        # driver and witness at 512^2 in the mixed form
        dict(name="slices_512_mixed", kind="slices", n=512, half_width=8.0, ppc=2, slices=12,
             regime="blowout", precision="mixed", pusher="boris", adaptive=True, dxi0=0.01),
        # nine particles a cell and the four-stage pusher, fixed steps
        dict(name="slices_512_rk4", kind="slices", n=512, half_width=10.0, ppc=3, slices=9,
             regime="blowout", precision="fp64", pusher="rk4", adaptive=False, dxi0=0.01),
        # the production run: 1024^2, 4.2 million particles
        dict(name="slices_1024_blowout", kind="slices", n=1024, half_width=10.0, ppc=2, slices=12,
             regime="blowout", precision="fp64", pusher="boris", adaptive=True, dxi0=0.005),
        # gradient of a probe with respect to 32 radial bins of the driver
        dict(name="adjoint_256_bins", kind="adjoint", n=256, half_width=8.0, ppc=2, slices=20,
             every=8, bins=32, dxi0=0.02),
        # one time step of a sampled electron driver
        dict(name="driver_256", kind="driver", n=256, half_width=8.0, ppc=2, slices=40,
             particles=50021, nsub=4, dxi0=0.05, dt=10.0),
        # one time step of a laser pulse and the plasma behind its front
        dict(name="laser_512", kind="laser", n=512, half_width=8.0, ppc=2, slices=20, k0=20.0,
             a0=2.0, dxi0=0.04, dt=10.0),
        # a single small solve
        dict(name="poisson_128", kind="poisson", n=128, half_width=6.0, nrhs=1),
        # the B_perp system of the production grid
        dict(name="helmholtz_1024", kind="helmholtz", n=1024, half_width=10.0, nrhs=2),
        # a serving loop's solve: no allocation, no host synchronisation
        dict(name="noalloc_256", kind="noalloc", n=256, half_width=8.0, nrhs=2, helm=True,
             cycles=14),
        # three-region grid of the bubble, the Helmholtz form
        dict(name="nonuniform_1024", kind="nonuniform", n=1024, half_width=10.0, axis="regions",
             helm=True),
    ]


def draw(rng):
    kind = rng.choice(["slices", "slices", "slices", "adjoint", "driver", "laser", "poisson",
                       "helmholtz", "noalloc", "nonuniform"])
    L = rng.choice([6.0, 8.0, 10.0]) * (1.0 + 0.01 * rng.randrange(10))
    if kind == "slices":
        n = rng.choice([64, 128, 256, 512, 1024])
        return dict(kind=kind, n=n, half_width=L, ppc=rng.choice([1, 2, 3] if n <= 512 else [1, 2]),
                    slices=rng.randrange(5, 13), regime=rng.choice(["linear", "blowout"]),
                    precision=rng.choice(["fp64", "fp64", "mixed"]),
                    pusher=rng.choice(["boris", "boris", "rk1", "rk2", "rk4"]),
                    adaptive=rng.choice([False, True]),
                    dxi0=round(rng.uniform(0.2, 0.5) * 2.0 * L / n, 5))
    if kind == "adjoint":
        return dict(kind=kind, n=rng.choice([64, 128, 256]), half_width=L, ppc=rng.choice([1, 2, 3]),
                    slices=rng.randrange(9, 21), every=rng.choice([4, 7, 16]),
                    bins=rng.randrange(5, 41), dxi0=round(rng.uniform(0.01, 0.03), 4))
    if kind == "driver":
        return dict(kind=kind, n=rng.choice([64, 128, 256, 512]), half_width=L,
                    ppc=rng.choice([1, 2]), slices=rng.randrange(17, 41),
                    particles=int(math.exp(rng.uniform(math.log(2000), math.log(100000)))),
                    nsub=rng.choice([1, 4]), dxi0=round(rng.uniform(0.03, 0.06), 4),
                    dt=round(rng.uniform(5.0, 15.0), 2))
    if kind == "laser":
        n = rng.choice([64, 128, 256, 512])
        return dict(kind=kind, n=n, half_width=L, ppc=rng.choice([1, 2]),
                    slices=rng.randrange(8, 21), k0=round(rng.uniform(8.0, 25.0), 2),
                    a0=round(rng.uniform(0.5, 2.0), 2), dxi0=round(rng.uniform(0.02, 0.06), 4),
                    dt=round(rng.uniform(4.0, 12.0), 2))
    if kind in ("poisson", "helmholtz"):
        return dict(kind=kind, n=rng.choice([32, 64, 128, 256, 512, 1024]), half_width=L,
                    nrhs=rng.choice([1, 2]))
    if kind == "noalloc":
        return dict(kind=kind, n=rng.choice([64, 128, 256]), half_width=L, nrhs=rng.choice([1, 2]),
                    helm=rng.choice([False, True]), cycles=rng.randrange(12, 17))
    return dict(kind=kind, n=rng.choice([64, 128, 256, 512, 1024]), half_width=L,
                axis=rng.choice(["regions", "smooth"]), helm=rng.choice([False, True]))


# ----------------------------------------------------------------- inputs --

def _config(case, seed):
    """The configuration a program hands to Simulation for this case."""
    cfg = dict(n_cells=case["n"], half_width=case["half_width"], ppc_side=case.get("ppc", 1),
               jitter=0.0, seed=int(seed) & 0xFFFFFFFF, n0=1.0, dxi0=case.get("dxi0", 0.02),
               adaptive=int(case.get("adaptive", False)), refine_k=8,
               precision=case.get("precision", "fp64"), mg_rtol=1e-14, mg_atol=0.0,
               mg_max_cycles=50, nu_pre=2, nu_post=2, beams=[], probes=[], checkpoint_every=0,
               pusher=case.get("pusher", "boris"))
    kind = case["kind"]
    if cfg["ppc_side"] > 1:
        cfg["jitter"] = 0.25 if cfg["ppc_side"] == 2 else 0.1
    gauss = lambda a, sr, sz, xc: dict(kind="gauss", amp=a, sigma_r=sr, sigma_z=sz, xi_c=xc,  # noqa: E731
                                       x0=0.0, y0=0.0)
    if kind == "slices":
        if case["regime"] == "linear":
            cfg["beams"] = [gauss(0.1, 0.5, 1.0, 2.0)]
        else:
            cfg["beams"] = [gauss(5.0, 0.4, 0.8, 2.0), gauss(2.0, 0.2, 0.3, 6.5)]
    if kind == "adjoint":
        u = np.random.RandomState(seed % (1 << 31)).uniform(0.5, 2.0, case["bins"])
        h = 2.0 * case["half_width"] / case["n"]
        r_max = max(1.0, case["bins"] * h)
        cfg["beams"] = [dict(kind="radial_bins", bin_amp=u, r_max=r_max, sigma_z=0.8, xi_c=2.0,
                             x0=0.0, y0=0.0, amp=1.0, sigma_r=1.0)]
        cfg["probes"] = [dict(field=1, slice_begin=case["slices"] // 2, slice_end=case["slices"],
                              r_max=0.5, x0=0.0, y0=0.0)]
        cfg["checkpoint_every"] = case["every"]
    if kind == "driver":
        cfg.update(driver_max=case["particles"], driver_nz=int(case["slices"]) + 8,
                   driver_xi0=-2.0 * case["dxi0"], driver_dz=case["dxi0"], driver_nsub=case["nsub"])
    if kind == "laser":
        cfg.update(laser_nz=case["slices"], laser_k0=case["k0"])
    if kind == "noalloc":
        cfg.update(mg_rtol=0.0, mg_max_cycles=case["cycles"])
    if kind == "nonuniform":
        cfg.update(mg_max_cycles=200)
    return cfg


def _gen(seed):
    return torch.Generator(device=_dev()).manual_seed(int(seed))


def _plasma(case, seed):
    """Mid-run particles [4][P]: the lattice (jittered), displaced and set in
    motion as behind the driver -- a small radial oscillation (linear), or a
    cavity of radius about 1.5 with the electrons piled up in its sheath
    (blowout) -- with a weak swirl and a little spread in momentum."""
    n, L, s = case["n"], case["half_width"], case["ppc"]
    h, dev, g = 2.0 * L / n, _dev(), _gen(seed)
    a = torch.arange(n * s, dtype=F64, device=dev)
    X = -L + h * (a + 0.5) / s
    x = X.repeat(n * s, 1).reshape(n, s, n, s).permute(0, 2, 1, 3).reshape(-1)
    y = X.reshape(-1, 1).repeat(1, n * s).reshape(n, s, n, s).permute(0, 2, 1, 3).reshape(-1)
    P = x.numel()
    amp = 1.0 + 0.1 * torch.rand(4, dtype=F64, device=dev, generator=g)
    x = x + 0.2 * h / s * (2.0 * torch.rand(P, dtype=F64, device=dev, generator=g) - 1.0)
    y = y + 0.2 * h / s * (2.0 * torch.rand(P, dtype=F64, device=dev, generator=g) - 1.0)
    rx, ry = x - 0.05 * (amp[2] - 1.0), y - 0.05 * (amp[3] - 1.0)
    q = rx * rx + ry * ry
    if case["regime" if "regime" in case else "kind"] == "linear":
        e = torch.exp(-q)
        px, py = 0.03 * amp[0] * rx * e, 0.03 * amp[0] * ry * e
        x, y = x + 0.01 * amp[1] * rx * e, y + 0.01 * amp[1] * ry * e
        spread = 1e-4
    else:
        R = 1.4 * amp[0] if case["kind"] == "slices" else 0.5 * amp[0]
        e = torch.exp(-(q / (R * R)) ** 2)
        r1 = torch.sqrt(q + R * R * e)
        r0 = torch.sqrt(q).clamp_min(1e-12)
        ux, uy = rx / r0, ry / r0
        pr = 0.4 * R * amp[1] * torch.exp(-q / (R * R))
        sw = 0.05 * amp[2] * torch.exp(-q / (4.0 * R * R))
        x, y = x + (r1 - r0) * ux, y + (r1 - r0) * uy
        px, py = pr * ux - sw * ry, pr * uy + sw * rx
        spread = 3e-3
    px = px + spread * torch.randn(P, dtype=F64, device=dev, generator=g)
    py = py + spread * torch.randn(P, dtype=F64, device=dev, generator=g)
    lim = L * (1.0 - 1e-9)
    return torch.stack([x.clamp(-lim, lim), y.clamp(-lim, lim), px, py])


def _driver(case, seed):
    """An electron beam of gamma ~ 2000, sampled from a Gaussian."""
    g, dev, n = _gen(seed), _dev(), case["particles"]
    z = torch.randn(5, n, dtype=F64, device=dev, generator=g)
    xi_c = 0.5 * case["slices"] * case["dxi0"]
    sz = 0.25 * case["slices"] * case["dxi0"]
    d = torch.zeros(8, n, dtype=F64, device=dev)
    d[0], d[1], d[2] = 0.4 * z[0], 0.4 * z[1], xi_c + sz / math.sqrt(2.0) * z[2]
    d[3], d[4] = 0.5 * z[3], 0.5 * z[4]
    d[5] = 2000.0 * (1.0 + 0.01 * torch.rand(n, dtype=F64, device=dev, generator=g))
    d[6] = -1.0
    d[7] = 2.0 * math.pi * 0.32 * math.sqrt(math.pi) * sz / n
    return d


def _laser(case, seed):
    """Envelope planes of a Gaussian pulse with a small chirp."""
    n, L, nz = case["n"], case["half_width"], case["slices"]
    u = torch.rand(4, dtype=F64, device=_dev(), generator=_gen(seed))
    x = torch.linspace(-L, L, n + 1, dtype=F64, device=_dev())
    xi = case["dxi0"] * torch.arange(nz, dtype=F64, device=_dev())
    w0, sz, xc = 2.0 + u[0], (0.3 + 0.1 * u[1]) * nz * case["dxi0"], 0.5 * nz * case["dxi0"]
    r2 = (x[None, :] - 0.1 * u[2]) ** 2 + (x[:, None] + 0.1 * u[3]) ** 2
    ph = 0.3 * (xi - xc)[:, None, None] * (1.0 + 0.05 * r2)
    env = case["a0"] * torch.exp(-r2 / w0 ** 2 - ((xi - xc) / sz)[:, None, None] ** 2)
    env = torch.complex(env * torch.cos(ph), env * torch.sin(ph))
    env[:, 0, :] = env[:, -1, :] = 0.0
    env[:, :, 0] = env[:, :, -1] = 0.0
    return env.contiguous()


def _axis(n, L, kind):
    s = -1.0 + 2.0 * np.arange(n + 1) / n
    if kind == "smooth":
        return L * np.sinh(2.0 * s) / np.sinh(2.0)
    a = np.abs(s)
    x = np.where(a < 0.25, a, np.where(a < 0.5, 0.25 + 2 * (a - 0.25), 0.75 + 3 * (a - 0.5)))
    return np.sign(s) * x * (L / 2.25)


def _sources(case, seed):
    """Right-hand sides and coefficient of a solve: a cavity with its sheath and
    particle noise; f [nrhs][n+1][n+1], k2 [n+1][n+1] = n*/(1 + psi) >= 0."""
    n, L = case["n"], case["half_width"]
    g, dev = _gen(seed), _dev()
    if case["kind"] == "nonuniform":
        X = torch.from_numpy(_axis(n, L, case["axis"])).to(dev)
    else:
        X = torch.linspace(-L, L, n + 1, dtype=F64, device=dev)
    u = torch.rand(4, dtype=F64, device=dev, generator=g)
    r = torch.sqrt((X[None, :] - 0.2 * u[0]) ** 2 + (X[:, None] - 0.2 * u[1]) ** 2)
    R = 1.5 + 0.5 * u[2]
    noise = torch.randn(3, n + 1, n + 1, dtype=F64, device=dev, generator=g)
    dens = 0.5 * (1.0 + torch.tanh((r - R) / 0.2)) + 3.0 * torch.exp(-((r - R) / 0.25) ** 2)
    k2 = (dens * (1.0 + 0.05 * noise[0])).clamp_min(0.0)
    f = [dens - 1.0 + 0.05 * noise[1], X[None, :] * (1.0 - dens) * torch.exp(-r) + 0.05 * noise[2]]
    f = torch.stack(f[: case.get("nrhs", 1)])
    f[:, 0, :] = f[:, -1, :] = 0.0
    f[:, :, 0] = f[:, :, -1] = 0.0
    return f.contiguous(), k2.contiguous()


def prepare(case, seed):
    kind, cfg = case["kind"], _config(case, seed)
    st = dict(case=case, cfg=cfg)
    if kind in ("slices", "adjoint"):
        sim = Simulation(cfg, n_slices=case["slices"])
        st["particles"] = _plasma(case, seed)
        st["xi"], st["dxi"] = 1.9, case["dxi0"]
        # the fields a checkpoint holds: those of the slice the state is at
        sim.set_state(particles=st["particles"], xi=st["xi"], dxi=st["dxi"])
        st["fields"], _ = sim.step(fields=True)
        st["sim"] = sim
        if kind == "adjoint":
            st["pbar"] = torch.randn(4, sim.P, dtype=F64, device=_dev(), generator=_gen(seed + 1))
    elif kind == "driver":
        st["sim"], st["driver"] = Simulation(cfg, n_slices=case["slices"]), _driver(case, seed)
    elif kind == "laser":
        st["sim"], st["env"] = Simulation(cfg, n_slices=case["slices"]), _laser(case, seed)
    else:
        st["f"], st["k2"] = _sources(case, seed)
        if kind == "nonuniform":
            st["x"] = _axis(case["n"], case["half_width"], case["axis"])
            st["M"] = (-st["k2"]).contiguous() if case["helm"] else None
        if kind != "noalloc":
            st["sim"] = Simulation(cfg)
    return st


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "slices":
        sim = st["sim"]
        sim.set_state(particles=st["particles"], fields=st["fields"], xi=st["xi"], dxi=st["dxi"])
        sim.run(case["slices"])
        got = sim.get_state()
        return dict(particles=got["particles"], fields=got["fields"], xi=got["xi"], dxi=got["dxi"])
    if kind == "adjoint":
        sim = st["sim"]
        sim.set_state(particles=st["particles"], fields=st["fields"], xi=st["xi"], dxi=st["dxi"])
        _, probe = sim.run(case["slices"], probes=True)
        theta, p0 = sim.backward(dL_dprobe=[1.0], dL_dparticles=st["pbar"], particles_grad=True)
        return dict(probe=probe, theta=theta, particles0=p0)
    if kind == "driver":
        sim = st["sim"]
        sim.driver_set(st["driver"])
        sim.time_step(case["dt"], case["slices"])
        return dict(driver=sim.driver_get(), fields=sim.get_state()["fields"])
    if kind == "laser":
        sim = st["sim"]
        sim.laser_set(st["env"])
        sim.time_step(case["dt"], case["slices"])
        return dict(env=sim.laser_get(), fields=sim.get_state()["fields"])
    if kind in ("poisson", "helmholtz"):
        _, u, _, _ = st["sim"].mg_solve(st["f"], k2=st["k2"] if kind == "helmholtz" else None)
        return u
    if kind == "noalloc":
        return mg_solve_noalloc(st["cfg"], st["f"], k2=st["k2"] if case["helm"] else None)[1]
    return st["sim"].nu_mg_solve(st["x"], st["x"], st["f"][0], M=st["M"])[1]


def work(case):
    """Inputs read once, outputs written once; per slice the particles and the
    five fields with the six moments between them."""
    nodes, kind = float((case["n"] + 1) ** 2), case["kind"]
    if kind in ("slices", "adjoint", "driver", "laser"):
        P, S = float((case["n"] * case["ppc"]) ** 2), float(case["slices"])
        b = S * (64.0 * P + 8.0 * nodes * (5 + 5 + 6 + 6))
        fl = S * (250.0 * P + 500.0 * nodes)
        if kind == "adjoint":
            b, fl = 3.0 * b, 3.0 * fl
        if kind == "laser":
            b, fl = b + S * nodes * 16.0 * 4, fl + S * nodes * 200.0
        if kind == "driver":
            b, fl = b + 128.0 * case["particles"], fl + 400.0 * case["particles"]
        return dict(bytes=b, flops=fl)
    R = case.get("nrhs", 1)
    helm = kind == "helmholtz" or bool(case.get("helm"))
    return dict(bytes=8.0 * nodes * (2 * R + (1 if helm else 0)), flops=150.0 * nodes * R)


# ------------------------------------------------------------------ exact --

class _Solve(torch.autograd.Function):
    """u with (L_h - k2) u = f (interior), by the reference's Krylov iteration."""

    @staticmethod
    def forward(ctx, ref, f, k2):
        u = ref.helm(f, k2)
        ctx.ref = ref
        ctx.save_for_backward(u, k2)
        return u

    @staticmethod
    def backward(ctx, g):
        u, k2 = ctx.saved_tensors
        lam = ctx.ref.helm(ctx.ref.inside(g), k2)
        return None, lam, (lam * u if ctx.needs_input_grad[2] else None)


class _Ref:
    """The slice of the quasi-static model in plain torch."""

    def __init__(self, cfg):
        self.cfg, self.N, self.L = cfg, cfg["n_cells"], cfg["half_width"]
        self.h, self.dev = 2.0 * self.L / self.N, _dev()
        N = self.N
        k = torch.arange(1, N, device=self.dev)
        self.S = torch.sin(math.pi * ((k[:, None] * k[None, :]) % (2 * N)).to(F64) / N)
        self.mu = -(4.0 / self.h ** 2) * torch.sin(math.pi * k.to(F64) / (2 * N)) ** 2
        self.x = -self.L + self.h * torch.arange(N + 1, dtype=F64, device=self.dev)
        self.wdep = cfg["n0"] / cfg["ppc_side"] ** 2

    def inside(self, a):
        return torch.nn.functional.pad(a[1:-1, 1:-1], (1, 1, 1, 1))

    def const(self, f, shift=0.0):
        """(L_h - shift)^-1 f on interior values."""
        lam = self.mu[:, None] + self.mu[None, :] - shift
        return (2.0 / self.N) ** 2 * (self.S @ ((self.S @ f @ self.S) / lam) @ self.S)

    def poisson(self, f):
        return torch.nn.functional.pad(self.const(f[1:-1, 1:-1]), (1, 1, 1, 1))

    def lap(self, u):
        p = torch.nn.functional.pad(u, (1, 1, 1, 1))
        return (p[1:-1, :-2] + p[1:-1, 2:] + p[:-2, 1:-1] + p[2:, 1:-1] - 4.0 * u) / self.h ** 2

    def helm(self, f, k2):
        b, k = f[1:-1, 1:-1], k2[1:-1, 1:-1]
        s = k.mean() + 0.05
        u = torch.zeros_like(b)
        for _ in range(2):  # conjugate gradients on the residual, twice
            r = b - (self.lap(u) - k * u)
            e, z = torch.zeros_like(b), self.const(r, s)
            p, rz, first = z, (r * z).sum(), float(r.norm())
            if first == 0.0:
                break
            for _ in range(80):
                q = self.lap(p) - k * p
                a = rz / (p * q).sum()
                e, r = e + a * p, r - a * q
                if float(r.norm()) <= 1e-13 * first:
                    break
                z = self.const(r, s)
                rz, old = (r * z).sum(), rz
                p = z + (rz / old) * p
            u = u + e
        return torch.nn.functional.pad(u, (1, 1, 1, 1))

    def cell(self, x, y):
        tx, ty = (x + self.L) / self.h, (y + self.L) / self.h
        a = tx.detach().floor().clamp(0, self.N - 1)
        b = ty.detach().floor().clamp(0, self.N - 1)
        return (b * (self.N + 1) + a).long(), tx - a, ty - b

    def corners(self, dx, dy):
        return (1 - dx) * (1 - dy), dx * (1 - dy), (1 - dx) * dy, dx * dy

    def gather(self, F, at):
        i, dx, dy = at
        v = F.reshape(-1)
        o = (0, 1, self.N + 1, self.N + 2)
        return sum(w * v[i + d] for w, d in zip(self.corners(dx, dy), o))

    def deposit(self, q, at, scale):
        i, dx, dy = at
        out = torch.zeros((self.N + 1) ** 2, dtype=F64, device=self.dev)
        for w, d in zip(self.corners(dx, dy), (0, 1, self.N + 1, self.N + 2)):
            out = out.index_add(0, i + d, w * q)
        return (scale * out).reshape(self.N + 1, self.N + 1)

    def dx(self, F):
        return torch.nn.functional.pad((F[1:-1, 2:] - F[1:-1, :-2]) / (2 * self.h), (1, 1, 1, 1))

    def dy(self, F):
        return torch.nn.functional.pad((F[2:, 1:-1] - F[:-2, 1:-1]) / (2 * self.h), (1, 1, 1, 1))

    def grad(self, F):
        gx = torch.cat([(F[:, 1:2] - F[:, :1]) / self.h, (F[:, 2:] - F[:, :-2]) / (2 * self.h),
                        (F[:, -1:] - F[:, -2:-1]) / self.h], 1)
        gy = torch.cat([(F[1:2] - F[:1]) / self.h, (F[2:] - F[:-2]) / (2 * self.h),
                        (F[-1:] - F[-2:-1]) / self.h], 0)
        return gx, gy

    def beams(self, xi, theta=None):
        out = torch.zeros(self.N + 1, self.N + 1, dtype=F64, device=self.dev)
        for b in self.cfg["beams"]:
            fz = math.exp(-((xi - b["xi_c"]) / b["sigma_z"]) ** 2)
            r2 = (self.x[None, :] - b["x0"]) ** 2 + (self.x[:, None] - b["y0"]) ** 2
            if b["kind"] == "gauss":
                out = out + b["amp"] * fz * torch.exp(-r2 / b["sigma_r"] ** 2)
            else:
                nb = len(b["bin_amp"])
                k = torch.floor(torch.sqrt(r2) / (b["r_max"] / nb)).long()
                ok = (torch.sqrt(r2) < b["r_max"]) & (k < nb)
                out = out + fz * torch.where(ok, theta[k.clamp(0, nb - 1)], torch.zeros_like(out))
        return out

    def fields(self, p, jb, a2=None):
        """psi, Ez, Bz, Bx, By and k2 of the particles p with the driver current jb."""
        at = self.cell(p[0], p[1])
        n = self.deposit(torch.ones_like(p[0]), at, self.wdep)
        psi = self.poisson(n - self.cfg["n0"])
        gi = 1.0 + self.gather(psi, at)
        vx, vy = p[2] / gi, p[3] / gi
        jx, jy, txx, txy, tyy = (self.deposit(q, at, self.wdep)
                                 for q in (vx, vy, vx * vx, vx * vy, vy * vy))
        Ez = self.poisson(-(self.dx(jx) + self.dy(jy)))
        Bz = self.poisson(self.dx(jy) - self.dy(jx))
        g = 1.0 + psi
        half = 0.0 if a2 is None else 0.5 * a2
        G = (n * (1.0 + g * g + half) + g * g * (txx + tyy)) / (2.0 * g)
        jz = torch.where(n > 0, G / g - n, torch.zeros_like(n)) + jb
        k2 = self.inside(torch.where(n > 0, n / g, torch.zeros_like(n)))
        px, py = self.dx(psi), self.dy(psi)
        lx = (jx * Bz - jy * Ez) / g + (G / (g * g) - tyy / g) * py - (txy / g) * px
        ly = (jy * Bz + jx * Ez) / g - (G / (g * g) - txx / g) * px + (txy / g) * py
        if a2 is not None:
            lx = lx - n * 0.25 * self.dy(a2) / (g * g)
            ly = ly + n * 0.25 * self.dx(a2) / (g * g)
        zero = torch.zeros_like(n)
        fx = self.dy(jz - tyy) - self.dx(txy) + torch.where(n > 0, lx, zero)
        fy = self.dx(txx - jz) + self.dy(txy) + torch.where(n > 0, ly, zero)
        Bx = _Solve.apply(self, self.inside(fx), k2)
        By = _Solve.apply(self, self.inside(fy), k2)
        return psi, Ez, Bz, Bx, By, k2

    def force(self, s, F, gp, las):
        at = self.cell(s[0], s[1])
        g = 1.0 + self.gather(F[0], at)
        Gx, Gy = self.gather(gp[0], at), self.gather(gp[1], at)
        bz, bx, by = (self.gather(F[k], at) for k in (2, 3, 4))
        a2, ax, ay = (self.gather(v, at) for v in las) if las else (0.0, 0.0, 0.0)
        gam = (1.0 + s[2] ** 2 + s[3] ** 2 + g * g + 0.5 * a2) / (2.0 * g)
        return g, (gam * Gx - 0.25 * ax) / g - by, (gam * Gy - 0.25 * ay) / g + bx, bz

    def push(self, p, F, d, a2=None):
        gp = self.grad(F[0])
        las = None if a2 is None else (a2,) + tuple(self.grad(a2))
        order = {"boris": 0, "rk1": 1, "rk2": 2, "rk4": 4}[self.cfg["pusher"]]
        x, y, px, py = p[0], p[1], p[2], p[3]
        if order == 0:
            g, Fx, Fy, bz = self.force(p, F, gp, las)
            mx, my = px + 0.5 * d * Fx, py + 0.5 * d * Fy
            t = bz * d / (2.0 * g)
            s = 2.0 * t / (1.0 + t * t)
            qx, qy = mx - t * my, my + t * mx
            px, py = mx - s * qy + 0.5 * d * Fx, my + s * qx + 0.5 * d * Fy
            x, y = x + d * px / g, y + d * py / g
        else:
            def rhs(s):
                gg, Fx, Fy, bz = self.force(s, F, gp, las)
                vx, vy = s[2] / gg, s[3] / gg
                return gg, torch.stack([vx, vy, Fx - vy * bz, Fy + vx * bz])
            g, k1 = rhs(p)
            if order == 1:
                o = p + d * k1
            elif order == 2:
                o = p + d * rhs(p + 0.5 * d * k1)[1]
            else:
                k2 = rhs(p + 0.5 * d * k1)[1]
                k3 = rhs(p + 0.5 * d * k2)[1]
                k4 = rhs(p + d * k3)[1]
                o = p + (d / 6.0) * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
            x, y, px, py = o[0], o[1], o[2], o[3]
        L = self.L
        px = torch.where(x.abs() > L, -px, px)
        py = torch.where(y.abs() > L, -py, py)
        x = torch.where(x > L, 2 * L - x, torch.where(x < -L, -2 * L - x, x))
        y = torch.where(y > L, 2 * L - y, torch.where(y < -L, -2 * L - y, y))
        vmax = float((torch.sqrt(px * px + py * py) / g).detach().max())
        return torch.stack([x, y, px, py]), vmax

    def step_size(self, vmax):
        d0 = self.cfg["dxi0"]
        if not self.cfg["adaptive"] or not vmax > 0.0:
            return d0
        return max(min(d0, self.h / vmax), d0 / self.cfg["refine_k"])


def _lattice(cfg):
    """The cold plasma a time step starts from (the library's own jittered
    lattice: SplitMix64 draws in particle order)."""
    N, L, s, J = cfg["n_cells"], cfg["half_width"], cfg["ppc_side"], cfg["jitter"]
    b, a, sy, sx = (v.reshape(-1).astype(np.float64) for v in
                    np.meshgrid(*(np.arange(k) for k in (N, N, s, s)), indexing="ij"))
    k = np.arange(1, 2 * a.size + 1, dtype=np.uint64)
    with np.errstate(over="ignore"):
        z = np.uint64(cfg["seed"]) + k * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    u = (z >> np.uint64(11)).astype(np.float64) * 2.0 ** -53
    h = 2.0 * L / N
    x = -L + h * ((a + (sx + 0.5) / s) + J * (2.0 * u[0::2] - 1.0))
    y = -L + h * ((b + (sy + 0.5) / s) + J * (2.0 * u[1::2] - 1.0))
    return torch.from_numpy(np.stack([x, y, 0 * x, 0 * x])).to(_dev())


def _exact_slices(case, seed):
    ref = _Ref(_config(case, seed))
    p, xi, d = _plasma(case, seed), 1.9, case["dxi0"]
    for _ in range(case["slices"]):
        F = ref.fields(p, ref.beams(xi))
        p, vmax = ref.push(p, F, d)
        xi, d = xi + d, ref.step_size(vmax)
    return dict(particles=p, fields=torch.stack(F[:5]), xi=xi, dxi=d)


def _exact_adjoint(case, seed):
    cfg = _config(case, seed)
    ref, pr = _Ref(cfg), cfg["probes"][0]
    p0 = _plasma(case, seed).requires_grad_(True)
    theta = torch.from_numpy(cfg["beams"][0]["bin_amp"]).to(_dev()).requires_grad_(True)
    disc = (ref.x[None, :] ** 2 + ref.x[:, None] ** 2 <= pr["r_max"] ** 2).to(F64)
    p, xi, d, probe = p0, 1.9, case["dxi0"], 0.0
    for j in range(case["slices"]):
        F = ref.fields(p, ref.beams(xi, theta))
        if j >= pr["slice_begin"]:
            probe = probe + (F[1] * disc).sum() / disc.sum() / (pr["slice_end"] - pr["slice_begin"])
        p, _ = ref.push(p, F, d)
        xi += d
    pbar = torch.randn(4, p.shape[1], dtype=F64, device=_dev(), generator=_gen(seed + 1))
    (probe + (p * pbar).sum()).backward()
    return dict(probe=probe.detach().reshape(1), theta=theta.grad, particles0=p0.grad)


def _exact_driver(case, seed):
    cfg = _config(case, seed)
    ref, d8, dt = _Ref(cfg), _driver(case, seed), case["dt"]
    N, L, h, nz, dz = ref.N, ref.L, ref.h, cfg["driver_nz"], cfg["driver_dz"]
    x, y, xi = d8[0], d8[1], d8[2]
    gam = torch.sqrt(1.0 + d8[3] ** 2 + d8[4] ** 2 + d8[5] ** 2)
    t = (xi - cfg["driver_xi0"]) / dz
    m = torch.floor(t)
    ok = (x.abs() <= L) & (y.abs() <= L) & (m >= 0) & (m <= nz - 2)
    q = (-d8[6] * d8[7] * (d8[5] / gam) / (h * h * dz))[ok]
    az, m = (t - m)[ok], m[ok].long()
    i, dx, dy = ref.cell(x[ok], y[ok])
    planes = torch.zeros(nz * (N + 1) ** 2, dtype=F64, device=ref.dev)
    for w, o in zip(ref.corners(dx, dy), (0, 1, N + 1, N + 2)):
        for k, wz in ((0, 1.0 - az), (1, az)):
            planes.index_add_(0, (m + k) * (N + 1) ** 2 + i + o, q * w * wz)
    planes = planes.reshape(nz, N + 1, N + 1)
    xh, yh = x + 0.5 * dt * d8[3] / gam, y + 0.5 * dt * d8[4] / gam
    xih = xi + 0.5 * dt * (1.0 - d8[5] / gam)
    E, B = torch.zeros(3, x.numel(), dtype=F64, device=ref.dev), torch.zeros(3, x.numel(), dtype=F64, device=ref.dev)
    p, s, d, before = _lattice(cfg), 0.0, case["dxi0"], None
    for j in range(case["slices"]):
        tm = (s - cfg["driver_xi0"]) / dz
        k = int(math.floor(tm))
        jb = ref.beams(s)
        if 0 <= k <= nz - 2:
            jb = jb + (1.0 - (tm - k)) * planes[k] + (tm - k) * planes[k + 1]
        F = ref.fields(p, jb)
        p, _ = ref.push(p, F, d)
        gp = ref.grad(F[0])
        wake = (-gp[0], -gp[1], F[1], F[2], F[3], F[4])
        if before is not None:
            lo, w0 = before
            sel = (xih >= lo) & (xih < s) & (xh.abs() <= L) & (yh.abs() <= L)
            at, a = ref.cell(xh[sel], yh[sel]), (xih[sel] - lo) / (s - lo)
            v = [(1.0 - a) * ref.gather(f0, at) + a * ref.gather(f1, at) for f0, f1 in zip(w0, wake)]
            E[:, sel] = torch.stack([v[0] + v[5], v[1] - v[4], v[2]])
            B[:, sel] = torch.stack([v[4], v[5], v[3]])
        before = (s, wake)
        s = s + d
    st, sub = d8.clone(), dt / case["nsub"]
    qm = d8[6]
    for _ in range(case["nsub"]):
        P = st[3:6]
        g0 = torch.sqrt(1.0 + (P * P).sum(0))
        mid = torch.stack([st[0] + 0.5 * sub * P[0] / g0, st[1] + 0.5 * sub * P[1] / g0,
                           st[2] + 0.5 * sub * (1.0 - P[2] / g0)])
        k = 0.5 * sub * qm
        m3 = P + k * E
        tv = k * B / torch.sqrt(1.0 + (m3 * m3).sum(0))
        sv = 2.0 * tv / (1.0 + (tv * tv).sum(0))
        pr = m3 + torch.linalg.cross(m3, tv, dim=0)
        P = m3 + torch.linalg.cross(pr, sv, dim=0) + k * E
        g1 = torch.sqrt(1.0 + (P * P).sum(0))
        st[3:6] = P
        st[0], st[1] = mid[0] + 0.5 * sub * P[0] / g1, mid[1] + 0.5 * sub * P[1] / g1
        st[2] = mid[2] + 0.5 * sub * (1.0 - P[2] / g1)
    return dict(driver=st, fields=torch.stack(F[:5]))


def _exact_laser(case, seed):
    cfg = _config(case, seed)
    ref, A0 = _Ref(cfg), _laser(case, seed)
    A1, nz, d, dt = torch.zeros_like(A0), case["slices"], case["dxi0"], case["dt"]
    beta, gam = 4.0 / (dt * d), 4.0 * case["k0"] / dt

    def lap(u):
        return torch.complex(ref.lap(u.real), ref.lap(u.imag))

    def const(f, shift):
        lam = ref.mu[:, None] + ref.mu[None, :] - shift
        S, re, im = ref.S, f.real.contiguous(), f.imag.contiguous()
        v = torch.complex(S @ re @ S, S @ im @ S) / lam
        re, im = v.real.contiguous(), v.imag.contiguous()
        return (2.0 / ref.N) ** 2 * torch.complex(S @ re @ S, S @ im @ S)

    p, xi = _lattice(cfg), 0.0
    for j in range(nz):
        t = xi / d
        m = int(math.floor(t))
        a2 = torch.zeros(ref.N + 1, ref.N + 1, dtype=F64, device=ref.dev)
        for k, w in ((m, 1.0 - (t - m)), (m + 1, t - m)):
            if 0 <= k < nz:
                a2 = a2 + w * (A0[k].real ** 2 + A0[k].imag ** 2)
        F = ref.fields(p, ref.beams(xi), a2)
        p, _ = ref.push(p, F, d, a2)
        # eq. (20) for this plane: complex conjugate-orthogonal conjugate gradients
        chi = F[5][1:-1, 1:-1]
        a0 = A0[j][1:-1, 1:-1]
        dp = (A1[j - 1] - A0[j - 1])[1:-1, 1:-1] if j else torch.zeros_like(a0)
        f = torch.complex(chi - beta, torch.full_like(chi, gam)) * a0 - lap(a0) - beta * dp
        kk = torch.complex(chi + beta, torch.full_like(chi, -gam))
        shift = complex(float(chi.mean()) + beta, -gam)
        u = a0 + dp
        for _ in range(2):
            r = f - (lap(u) - kk * u)
            e, z, first = torch.zeros_like(u), const(r, shift), float(r.norm())
            q, rz = z, (r * z).sum()
            if first == 0.0:
                break
            for _ in range(80):
                Aq = lap(q) - kk * q
                a = rz / (q * Aq).sum()
                e, r = e + a * q, r - a * Aq
                if float(r.norm()) <= 1e-13 * first:
                    break
                z = const(r, shift)
                rz, old = (r * z).sum(), rz
                q = z + (rz / old) * q
            u = u + e
        A1[j, 1:-1, 1:-1] = u
        xi = xi + d
    return dict(env=A1, fields=torch.stack(F[:5]))


def _exact_nonuniform(case, seed):
    """The nine-point system by GMRES, preconditioned with the exact solve of
    the tensor-product operator Dxx + Dyy + mean(M)."""
    n, dev = case["n"], _dev()
    X = _axis(n, case["half_width"], case["axis"])
    hm, hp = X[1:-1] - X[:-2], X[2:] - X[1:-1]
    ha, hb = hm + hp, hp - hm
    w = [torch.from_numpy(v).to(dev) for v in (2.0 / (hm * ha), -2.0 / (hm * hp), 2.0 / (hp * ha))]
    v = [torch.from_numpy(c).to(dev) for c in (-hp / (ha * hm), hp / (ha * hm) - hm / (ha * hp), hm / (ha * hp))]
    b3 = torch.from_numpy(hb / 3.0).to(dev)

    def ax(u, c, dim):  # three-point operator along dim, zero ends
        z = torch.nn.functional.pad(u, (1, 1, 0, 0) if dim == 1 else (0, 0, 1, 1))
        s = (lambda q: q[None, :]) if dim == 1 else (lambda q: q[:, None])
        lo, hi = (z[:, :-2], z[:, 2:]) if dim == 1 else (z[:-2], z[2:])
        return s(c[0]) * lo + s(c[1]) * u + s(c[2]) * hi

    J, k2 = _sources(case, seed)
    J, M = J[0], (-k2 if case["helm"] else torch.zeros_like(k2))

    def third(full):  # (1/3)(hb_x dx + hb_y dy) of values given with their boundary
        fx = v[0][None, :] * full[1:-1, :-2] + v[1][None, :] * full[1:-1, 1:-1] + v[2][None, :] * full[1:-1, 2:]
        fy = v[0][:, None] * full[:-2, 1:-1] + v[1][:, None] * full[1:-1, 1:-1] + v[2][:, None] * full[2:, 1:-1]
        return b3[None, :] * fx + b3[:, None] * fy

    def op(u):
        Mu = M[1:-1, 1:-1] * u
        dxx, dyy = ax(u, w, 1), ax(u, w, 0)
        s = dxx + dyy + b3[None, :] * ax(dyy, v, 1) + b3[:, None] * ax(dxx, v, 0)
        return s + third(torch.nn.functional.pad(Mu, (1, 1, 1, 1))) + Mu

    # Dxx = D^-1 K with D = diag(ha/2), K symmetric: eigenvectors of D^-1/2 K D^-1/2
    D = np.sqrt(0.5 * ha)
    T = np.diag(-2.0 / (hm * hp)) + np.diag((1.0 / hp[:-1]) / (D[:-1] * D[1:]), 1) + np.diag((1.0 / hp[:-1]) / (D[:-1] * D[1:]), -1)
    lam, Q = np.linalg.eigh(T)
    lam, Q, D = (torch.from_numpy(a).to(dev) for a in (lam, Q, D))
    Qt = Q.t().contiguous()
    den = lam[:, None] + lam[None, :] + M.mean()

    def pre(r):
        t = D[:, None] * D[None, :]
        return (Q @ ((Qt @ (r * t) @ Q) / den) @ Qt) / t

    f = J[1:-1, 1:-1] + third(J)
    u = torch.zeros_like(f)
    for _ in range(3):
        r = pre(f - op(u))
        beta = float(r.norm())
        if beta == 0.0:
            break
        V, H = [r / beta], np.zeros((41, 40))
        for j in range(40):
            z = pre(op(V[j]))
            for _ in range(2):
                for i in range(j + 1):
                    c = float((V[i] * z).sum())
                    H[i, j] += c
                    z = z - c * V[i]
            H[j + 1, j] = float(z.norm())
            if H[j + 1, j] <= 1e-14 * abs(H[0, 0]):
                break
            V.append(z / H[j + 1, j])
        k = j + 1
        e1 = np.zeros(k + 1)
        e1[0] = beta
        c = np.linalg.lstsq(H[: k + 1, :k], e1, rcond=None)[0]
        u = u + sum(float(c[i]) * V[i] for i in range(k))
    return torch.nn.functional.pad(u, (1, 1, 1, 1))


def exact(case, seed):
    kind = case["kind"]
    if kind == "adjoint":
        return _exact_adjoint(case, seed)
    with torch.no_grad():
        if kind == "slices":
            return _exact_slices(case, seed)
        if kind == "driver":
            return _exact_driver(case, seed)
        if kind == "laser":
            return _exact_laser(case, seed)
        if kind == "nonuniform":
            return _exact_nonuniform(case, seed)
        f, k2 = _sources(case, seed)
        ref = _Ref(_config(case, seed))
        if kind == "helmholtz" or case.get("helm"):
            return torch.stack([ref.helm(v, k2) for v in f])
        return torch.stack([ref.poisson(v) for v in f])
