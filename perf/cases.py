"""The calls whose speed matters, as a program on top of the package makes them.

A program on this library propagates a two-component order parameter in imaginary time (ground
states: single runs, runs to an energy rule, spin-Hall states, parameter sweeps) or in real time
(dynamics), and reads energies and norms.  `listed` has one case per such use, with the sizes of the
workload presets, of the tests and of the benchmark; `draw` gives further ones of the same ranges.

    case  = {"kind": "step" | "relax" | "sweep" | "energy", ...}
    state = prepare(case, seed)    # a context or batch with a state of this seed, on the GPU
    run(state)                     # one call (or one readout), its results
    exact(case, seed)              # what run() returns, in plain complex128 torch
"""
import math

import numpy as np
import torch

from paper_2010_15069_amd import Batch, Solver

# Physics of the presets: (g_uu, g_dd, g_ud), spin-momentum k_l, uniform Raman coupling, detuning,
# trap, box, step.  "raman": a spatial Raman coupling, "x" Omega(x) = 2 tanh(x / 4), "y" the clamped
# spin-Hall profile along y (full 2x2 real-space exponential), "" none (diagonal exponential).
PHYSICS = {
    # small two-component box without Raman coupling
    "tiny": dict(g=(1.0, 1.0, 0.9), k_l=0.0, omega=0.0, delta=0.0, wy=1.0, box=8.0, dt=1e-3, raman=""),
    # Raman-coupled gas with the coupling in k-space: throughput, dynamics and ground states
    "coupled": dict(g=(10.0, 10.0, 10.0), k_l=2.0, omega=1.0, delta=0.2, wy=1.0, box=8.0, dt=1e-3, raman=""),
    # large ground state: Omega(x) in real space, anisotropic trap
    "ground": dict(g=(50.0, 50.0, 50.0), k_l=2.0, omega=0.0, delta=0.0, wy=1.5, box=8.0, dt=1e-3, raman="x"),
    # spin-Hall system: strong unequal couplings, Omega(y); stepped with the N L N real-space split
    "hall": dict(g=(1.1e3, 1.1e3, 3.3e2), k_l=3.0, omega=0.0, delta=0.0, wy=1.0, box=16.0, dt=1e-3, raman="y"),
}
FIELD = 0.369   # spin-Hall synthetic field


def listed():
    return [
        # the smallest grid the tests and presets use: a few kilobytes per step, launches and latency only
        dict(name="tiny_imag", kind="step", physics="tiny", time="imag", nx=64, ny=64, steps=200, precision="c64", split="krk"),
        # the same grid as the published code computes it, in complex128 and real time
        dict(name="tiny_real_c128", kind="step", physics="tiny", time="real", nx=64, ny=64, steps=200, precision="c128", split="krk"),
        # a ground state run to an energy rule at 256^2, with its energy checks and the final read-out
        dict(name="relax_256", kind="relax", physics="coupled", nx=256, ny=256, steps=2000, every=50),
        # dynamics at 512^2 (the real-time preset)
        dict(name="real_512", kind="step", physics="coupled", time="real", nx=512, ny=512, steps=100, precision="c64", split="krk"),
        # the throughput workload, imaginary and real time
        dict(name="imag_1024", kind="step", physics="coupled", time="imag", nx=1024, ny=1024, steps=50, precision="c64", split="krk"),
        dict(name="real_1024", kind="step", physics="coupled", time="real", nx=1024, ny=1024, steps=50, precision="c64", split="krk"),
        # an elongated grid in real time with a spatial Raman coupling
        dict(name="real_long", kind="step", physics="ground", time="real", nx=2048, ny=256, steps=50, precision="c64", split="krk"),
        # the large ground state, Omega(x) in real space
        dict(name="imag_2048", kind="step", physics="ground", time="imag", nx=2048, ny=2048, steps=20, precision="c64", split="krk"),
        # a stretch of a spin-Hall trial
        dict(name="hall_1024", kind="step", physics="hall", time="imag", nx=1024, ny=1024, steps=50, precision="c64", split="nln"),
        # a parameter sweep: 8 instances of each of three sizes stepped together, energies read at the end
        dict(name="sweep_24", kind="sweep", time="imag", n=128, sizes=3, per_size=8, steps=300),
        # complex128 at the throughput size
        dict(name="imag_1024_c128", kind="step", physics="coupled", time="imag", nx=1024, ny=1024, steps=20, precision="c128", split="krk"),
        # the read-out between steps: energy and norm of a large state
        dict(name="energy_2048", kind="energy", physics="ground", nx=2048, ny=2048, precision="c64"),
    ]


def draw(rng):
    kind = rng.choice(["step"] * 7 + ["relax", "sweep", "energy"])
    if kind == "sweep":
        n = rng.choice([32, 64, 128])
        per = rng.randint(2, 8)
        return dict(kind=kind, time=rng.choice(["imag", "imag", "real"]), n=n, sizes=rng.randint(1, 3), per_size=per,
                    steps=rng.randint(20, 300))
    physics = rng.choice(["tiny", "coupled", "ground", "hall"])
    # power-of-two axes, independently, up to 2^22 points (4096 only with a shorter other axis)
    while True:
        nx, ny = 2 ** rng.randint(4, 12), 2 ** rng.randint(4, 12)
        if 2 ** 9 <= nx * ny <= 2 ** 22:
            break
    if kind == "energy":
        return dict(kind=kind, physics=physics, nx=nx, ny=ny, precision=rng.choice(["c64", "c64", "c128"]))
    most = 2 ** 26 // (nx * ny)   # grid points times steps, at most those of the largest listed case
    if kind == "relax":
        nx, ny = min(nx, 512), min(ny, 512)
        every = rng.randint(7, 100)
        return dict(kind=kind, physics=rng.choice(["tiny", "coupled"]), nx=nx, ny=ny, every=every,
                    steps=every * rng.randint(3, 15))
    precision = rng.choice(["c64", "c64", "c64", "c128"])
    split = "krk" if precision == "c128" else rng.choice(["krk", "krk", "nln", "rkr"])
    steps = max(1, min(int(round(math.exp(rng.uniform(0.0, math.log(300.0))))), most // (2 if precision == "c128" else 1)))
    return dict(kind=kind, physics=physics, time=rng.choice(["imag", "real"]), nx=nx, ny=ny, steps=steps,
                precision=precision, split=split)


# ---- inputs -----------------------------------------------------------------------------------

def params(case):
    f = PHYSICS[case["physics"]]
    p = dict(nx=case["nx"], ny=case["ny"], xmax=f["box"], ymax=f["box"], g_uu=f["g"][0], g_dd=f["g"][1],
             g_ud=f["g"][2], k_l=f["k_l"], omega=f["omega"], delta=f["delta"], wx=1.0, wy=f["wy"], omega_r0=0.0,
             omega_rw=1.0, dt=f["dt"], norm0=1.0)
    if f["raman"] == "x":
        p.update(omega_r0=2.0, omega_rw=4.0)
    if case.get("time") == "real" and case["physics"] == "coupled":
        p["dt"] = 5e-4
    return p


def profile_y(p):
    """The spin-Hall coupling Omega(y_i) for these parameters."""
    y = -p["ymax"] + 2.0 * p["ymax"] / p["ny"] * np.arange(p["ny"])
    u = np.clip(2.0 + y * 4.0 * FIELD / p["k_l"], 0.0, 4.0)
    return 0.5 * p["k_l"] ** 2 * np.sqrt(np.maximum(8.0 * u - u * u, 0.0))


def sweep_params(case, seed):
    rng = np.random.default_rng(seed)
    out = []
    for k in range(case["sizes"]):
        n = case["n"] << k
        for _ in range(case["per_size"]):
            g, om, de = rng.uniform(1.0, 100.0), rng.uniform(0.0, 3.0), rng.uniform(-0.5, 0.5)
            out.append(dict(nx=n, ny=n, xmax=8.0, ymax=8.0, g_uu=g, g_dd=g, g_ud=g, k_l=2.0, omega=om, delta=de, wx=1.0,
                            wy=1.0, omega_r0=0.0, omega_rw=1.0, dt=1e-3, norm0=1.0))
    return out


def axes(p):
    x = -p["xmax"] + 2.0 * p["xmax"] / p["nx"] * torch.arange(p["nx"], dtype=torch.float64, device="cuda")
    y = -p["ymax"] + 2.0 * p["ymax"] / p["ny"] * torch.arange(p["ny"], dtype=torch.float64, device="cuda")
    return x, y


def start_state(p, seed, precision, vortices=0):
    """A Thomas-Fermi cloud with 1e-3 complex noise (and vortices), normalised, in the library's
    layout: (ny, nx, 4) of re_up, im_up, re_dn, im_dn."""
    x, y = axes(p)
    X, Y = x[None, :], y[:, None]
    gu, gd = p["g_uu"] + p["g_ud"], p["g_dd"] + p["g_ud"]
    mu = math.sqrt(p["wx"] * p["wy"] * gu / (2.0 * math.pi))
    n = (mu - 0.5 * ((p["wx"] * X) ** 2 + (p["wy"] * Y) ** 2)).clamp(min=0.0)
    psi = torch.stack([(n / gu).sqrt(), (n / gd).sqrt()]).to(torch.complex128)
    if vortices:
        rng = np.random.default_rng(seed)
        radius, core = 0.8 * math.sqrt(2.0 * mu), 1.0 / math.sqrt(2.0 * mu)
        for c, sign in ((0, 1.0), (1, -1.0)):
            for _ in range(vortices):
                r, a = radius * math.sqrt(rng.uniform()), 2.0 * math.pi * rng.uniform()
                zx, zy = X - r * math.cos(a), Y - r * math.sin(a)
                psi[c] *= torch.complex(zx.expand_as(n), (sign * zy).expand_as(n)) / (zx * zx + zy * zy + core * core).sqrt()
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    noise = torch.randn((2, p["ny"], p["nx"], 2), generator=gen, dtype=torch.float64, device="cuda")
    psi += 1e-3 * psi.abs().max() * torch.view_as_complex(noise)
    w = 4.0 * p["xmax"] * p["ymax"] / (p["nx"] * p["ny"])
    psi *= torch.sqrt(p["norm0"] / (w * (psi.abs() ** 2).sum()))
    out = torch.view_as_real(psi).permute(1, 2, 0, 3).reshape(p["ny"], p["nx"], 4)
    return out.to(torch.float64 if precision == "c128" else torch.float32).contiguous()


def case_state(case, seed):
    p = params(case)
    return p, start_state(p, seed, case.get("precision", "c64"), vortices=10 if case["physics"] == "hall" else 0)


# ---- the calls --------------------------------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "sweep":
        ps = sweep_params(case, seed)
        b = Batch(ps)
        for i, p in enumerate(ps):
            b.set_psi_device(i, start_state(p, seed + i, "c64"))
        return dict(case=case, batch=b)
    p, psi = case_state(case, seed)
    torch.cuda.synchronize()
    # a step or an energy works on the program's own tensor; a relaxation keeps the state in the context
    own = case["kind"] == "relax"
    s = Solver(p, psi_dev=None if own else psi.data_ptr(), precision=case.get("precision", "c64"))
    if PHYSICS[case["physics"]]["raman"] == "y":
        s.set_raman_profile(omega_y=profile_y(p))
    if case.get("split") == "nln":
        s.set_splitting("krk", "nln")
    if case.get("split") == "rkr":
        s.set_splitting("rkr", "frozen")
    s.set_psi_device(psi)
    return dict(case=case, solver=s, psi=psi)


def run(state):
    case = state["case"]
    if case["kind"] == "sweep":
        b = state["batch"]
        (b.step_imag if case["time"] == "imag" else b.step_real)(case["steps"])
        # the energies of a complex64 trajectory carry fp32 rounding
        return dict(energies=b.energies().astype(np.float32), psi=b.get_psi(0).astype(np.complex64))
    s = state["solver"]
    if case["kind"] == "relax":
        r = s.relax_imag(check_every=case["every"], max_steps=case["steps"], rule="delta", tol=0.0, record_energies=True)
        return dict(energies=r["energies"].astype(np.float32), psi=s.get_psi().astype(np.complex64))
    if case["kind"] == "energy":
        return dict(energy=s.energy(), norm=s.norm())
    (s.step_imag if case["time"] == "imag" else s.step_real)(case["steps"])
    return dict(psi=state["psi"])


def work(case):
    """A step reads and writes the state once (each step needs the one before) and takes a forward and
    an inverse 2D transform per component and some 80 operations per point for its 2x2 exponentials."""
    def one(nx, ny, steps, point):
        n = nx * ny
        return 2.0 * point * n * steps, steps * n * (2 * 2 * 5.0 * math.log2(n) + 80.0)
    if case["kind"] == "energy":
        n, point = case["nx"] * case["ny"], 32 if case["precision"] == "c128" else 16
        return dict(bytes=float(point * n), flops=n * (2 * 5.0 * math.log2(n) + 60.0))
    if case["kind"] == "sweep":
        parts = [one(case["n"] << k, case["n"] << k, case["steps"] * case["per_size"], 16) for k in range(case["sizes"])]
    else:
        parts = [one(case["nx"], case["ny"], case["steps"], 32 if case.get("precision") == "c128" else 16)]
    return dict(bytes=sum(b for b, _ in parts), flops=sum(f for _, f in parts))


# ---- the same in complex128 torch ---------------------------------------------------------------

class Reference:
    """K(dt/2) R(dt) K(dt/2) (or R K R) on states of one grid, batched over instances."""

    def __init__(self, ps, raman_y=None, split="krk"):
        self.p, self.split = ps[0], split
        p = self.p
        col = lambda k: torch.tensor([q[k] for q in ps], dtype=torch.float64, device="cuda")[:, None, None]  # noqa: E731
        x, y = axes(p)
        self.dx, self.dy = 2.0 * p["xmax"] / p["nx"], 2.0 * p["ymax"] / p["ny"]
        self.v = 0.5 * ((p["wx"] * x[None, :]) ** 2 + (p["wy"] * y[:, None]) ** 2)
        om = p["omega_r0"] * torch.tanh(x[None, :] / p["omega_rw"]).expand_as(self.v)
        if raman_y is not None:
            om = om + torch.as_tensor(raman_y, device="cuda")[:, None]
        self.bx = 0.5 * om
        self.kx = 2.0 * math.pi * torch.fft.fftfreq(p["nx"], self.dx, dtype=torch.float64, device="cuda")[None, :]
        self.ky = 2.0 * math.pi * torch.fft.fftfreq(p["ny"], self.dy, dtype=torch.float64, device="cuda")[:, None]
        self.ak = 0.5 * (self.kx ** 2 + self.ky ** 2)
        self.omega, self.bzk, self.hd = col("omega"), p["k_l"] * self.kx, 0.5 * col("delta")
        self.guu, self.gdd, self.gud = col("g_uu"), col("g_dd"), col("g_ud")

    @staticmethod
    def exp2(u, d, a, bx, bz, h):
        """exp(-h (a 1 + bx sigma_x + bz sigma_z)) (u, d) for h real (imaginary time) or i times real."""
        b = torch.sqrt(bx * bx + bz * bz)
        z = h * b
        zero = b == 0
        s = torch.where(zero, torch.as_tensor(h, dtype=torch.complex128, device="cuda"), torch.sinh(z) / torch.where(zero, 1.0, b))
        c, e = torch.cosh(z), torch.exp(-h * a)
        return e * ((c - s * bz) * u - s * bx * d), e * ((c + s * bz) * d - s * bx * u)

    def k(self, u, d, h):
        u, d = self.exp2(torch.fft.fft2(u), torch.fft.fft2(d), self.ak + 0.0 * self.omega, 0.5 * self.omega + 0.0 * self.ak,
                         self.bzk + 0.0 * self.ak, h)
        return torch.fft.ifft2(u), torch.fft.ifft2(d)

    def r(self, u, d, h):
        nu, nd = u.abs() ** 2, d.abs() ** 2
        fu, fd = self.guu * nu + self.gud * nd, self.gdd * nd + self.gud * nu
        if self.split == "nln":
            u, d = torch.exp(-0.5 * h * fu) * u, torch.exp(-0.5 * h * fd) * d
            u, d = self.exp2(u, d, self.v, self.bx, self.hd + 0.0 * self.v, h)
            nu, nd = u.abs() ** 2, d.abs() ** 2
            return (torch.exp(-0.5 * h * (self.guu * nu + self.gud * nd)) * u,
                    torch.exp(-0.5 * h * (self.gdd * nd + self.gud * nu)) * d)
        return self.exp2(u, d, self.v + 0.5 * (fu + fd), self.bx, self.hd + 0.5 * (fu - fd), h)

    def steps(self, u, d, n, imag):
        h = self.p["dt"] * (1.0 + 0.0j if imag else 1.0j)
        ends, mid = (self.r, self.k) if self.split == "rkr" else (self.k, self.r)
        for _ in range(n):
            u, d = ends(u, d, 0.5 * h)
            u, d = mid(u, d, h)
            u, d = ends(u, d, 0.5 * h)
            if imag:
                c = torch.sqrt(self.p["norm0"] / self.norm(u, d))[:, None, None]
                u, d = c * u, c * d
        return u, d

    def norm(self, u, d):
        return self.dx * self.dy * (u.abs() ** 2 + d.abs() ** 2).sum((-2, -1))

    def energy(self, u, d):
        w, npts = self.dx * self.dy, self.p["nx"] * self.p["ny"]
        a, b = torch.fft.fft2(u), torch.fft.fft2(d)
        pu, pd = a.abs() ** 2, b.abs() ** 2
        ek = (self.ak * (pu + pd) + self.bzk * (pu - pd) + self.omega * (a.conj() * b).real).sum((-2, -1))
        nu, nd = u.abs() ** 2, d.abs() ** 2
        el = (self.v * (nu + nd) + self.hd * (nu - nd) + 2.0 * self.bx * (u.conj() * d).real).sum((-2, -1))
        ei = (0.5 * self.guu * nu * nu + 0.5 * self.gdd * nd * nd + self.gud * nu * nd).sum((-2, -1))
        nrm = self.norm(u, d)
        return (w / npts * ek + w * el) / nrm + w * ei * self.p["norm0"] / (nrm * nrm)


def components(psi):
    z = torch.view_as_complex(psi.to(torch.float64).reshape(*psi.shape[:-1], 2, 2).contiguous())
    return z[..., 0].contiguous(), z[..., 1].contiguous()


def exact(case, seed):
    if case["kind"] == "sweep":
        ps, energies, first = sweep_params(case, seed), [], None
        m = case["per_size"]
        for k in range(case["sizes"]):
            group = ps[k * m:(k + 1) * m]
            u, d = components(torch.stack([start_state(p, seed + k * m + i, "c64") for i, p in enumerate(group)]))
            ref = Reference(group)
            u, d = ref.steps(u, d, case["steps"], case["time"] == "imag")
            energies.append(ref.energy(u, d))
            first = torch.stack([u[0], d[0]]) if first is None else first
        return dict(energies=torch.cat(energies), psi=first)
    p, psi = case_state(case, seed)
    u, d = components(psi[None])
    ref = Reference([p], profile_y(p) if PHYSICS[case["physics"]]["raman"] == "y" else None, case.get("split", "krk"))
    if case["kind"] == "energy":
        return dict(energy=float(ref.energy(u, d)[0]), norm=float(ref.norm(u, d)[0]))
    if case["kind"] == "relax":
        energies, done = [ref.energy(u, d)], 0
        while done < case["steps"]:
            n = min(case["every"], case["steps"] - done)
            u, d = ref.steps(u, d, n, True)
            done += n
            energies.append(ref.energy(u, d))
        return dict(energies=torch.cat(energies), psi=torch.stack([u[0], d[0]]))
    u, d = ref.steps(u, d, case["steps"], case["time"] == "imag")
    return dict(psi=torch.view_as_real(torch.stack([u[0], d[0]], -1)).reshape(p["ny"], p["nx"], 4))
