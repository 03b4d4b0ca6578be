"""Performance cases of the reacting-flow library: what a program has it do,
through its public entry points, over the sizes and options it is used at.

A case is a dict of plain values:
  kind   "steps" (SSP-RK3 steps of one grid with the in-step CFL dt and the
         heat-release objective), "rhs" (one right-hand side with the heat
         release, as an outer integrator or a sampler calls it), "ensemble"
         (RK3 steps of many members as one captured graph) or "adjoint"
         (objective and its gradient over checkpointed steps)
  field  "hotspot" (1-D Gaussian hot spot in an acoustic wave), "vortex" (multicomponent
         Taylor-Green state) or "layer" (double mixing layer with a laser
         pulse under way)
  nx, ny, nz, ns (species; each has its seeded mechanism), steps
  scheme "hybrid", "weno3z" (in place of TENO6), "inert" (no chemistry)
  grid   "uniform", "stretched" (rectilinear) or "wavy" (curvilinear)
  walls  True: isothermal walls across y, inflow and outflow along x
An ensemble has `members` grids with sides between `lo` and `hi` (steps of
`by`) in the place of nx, ny, nz.

The composition, the noise, the pulse and the members' perturbations come
from the seed; the mechanism and the grid are what a program keeps.
"""
from __future__ import annotations

import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

import synth
from paper_2202_02319_amd import htr
from paper_2202_02319_amd.adjoint import HeatReleaseProblem

RU = 8.31446261815324
KB, NA, P_ATM = 1.380649e-23, 6.02214076e23, 101325.0
DX = 50e-6
FLAGS = {"hybrid": 0, "weno3z": synth.WENO3Z, "inert": synth.CHEM_OFF}
# species -> (reactions, mechanism seed at 1200 K and above, at the layers' 300 K)
MECHS = {5: (4, 1, 1), 9: (20, 0, 3), 12: (30, 18, 18)}
CFL, THETA_C, PSI_C, CT = 0.5, 0.1, 0.05, 1e-5


def _steps(name, field, n, ns, steps, **more):
    c = {"kind": "steps", "field": field, "nx": n[0], "ny": n[1], "nz": n[2], "ns": ns, "steps": steps,
         "scheme": "hybrid", "grid": "uniform", "walls": False, **more}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the 1-D reacting hot spot: the smallest program, a loop of steps over 256 cells
        _steps("hotspot_256", "hotspot", (256, 1, 1), 5, 20),
        # a 2-D diffusion layer with ignition pulse, the shape of a low-fidelity sample
        _steps("layer_2d_384x250", "layer", (384, 250, 1), 9, 4),
        # the headline box: 128^3, 9 species, 20 reactions
        _steps("vortex_128", "vortex", (128, 128, 128), 9, 2),
        # the mixing layer with laser deposition at its full size
        _steps("layer_256x128x128", "layer", (256, 128, 128), 9, 2),
        # a ragged stretched grid, small mechanism, WENO3-Z as the shock-capturing scheme
        _steps("layer_stretched_83x61x37", "layer", (83, 61, 37), 5, 4, scheme="weno3z", grid="stretched"),
        # walls and in/outflow: the boundary conditions of the flame and combustor set-ups
        _steps("channel_100x72x48", "layer", (100, 72, 48), 9, 3, walls=True),
        # curvilinear box of the headline size
        _steps("vortex_wavy_128", "vortex", (128, 128, 128), 9, 2, grid="wavy"),
        # one right-hand side of a large-mechanism box (most species the library takes)
        {"name": "rhs_75_12_species", "kind": "rhs", "field": "vortex", "nx": 75, "ny": 75, "nz": 75, "ns": 12,
         "steps": 1, "scheme": "hybrid", "grid": "uniform", "walls": False},
        # many small samples of an ignition study
        {"name": "ensemble_small_64", "kind": "ensemble", "members": 64, "lo": 12, "hi": 24, "by": 4, "ns": 9, "steps": 5},
        # uneven samples of a sensitivity study
        {"name": "ensemble_mixed_24", "kind": "ensemble", "members": 24, "lo": 32, "hi": 96, "by": 8, "ns": 9, "steps": 2},
        # objective and gradient: checkpointed steps and their reverse
        {"name": "adjoint_64", "kind": "adjoint", "field": "layer", "nx": 64, "ny": 64, "nz": 64, "ns": 9,
         "steps": 4, "every": 2, "scheme": "hybrid", "grid": "uniform", "walls": False},
    ]


def draw(rng):
    def logn(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["steps1", "steps2", "steps3", "steps3", "steps3", "walls", "wavy", "rhs", "ensemble", "adjoint"])
    ns = rng.choice([5, 9, 9, 12])
    scheme = rng.choice(["hybrid", "hybrid", "weno3z", "inert"])
    if kind == "steps1":
        return _steps(None, "hotspot", (logn(100, 4000), 1, 1), 5, rng.randint(5, 20))
    if kind == "steps2":
        return _steps(None, "layer", (logn(64, 800), logn(64, 800), 1), ns, rng.randint(1, 4), scheme=scheme)
    if kind in ("steps3", "walls", "wavy", "rhs"):
        big = 150 if kind == "wavy" else 100 if kind == "walls" else 170
        n = (logn(20, big), logn(20, big), logn(20, big))
        if kind == "walls":
            return _steps(None, "layer", n, ns, rng.randint(1, 3), walls=True)
        field = "vortex" if kind == "wavy" else rng.choice(["vortex", "layer"])
        grid = "wavy" if kind == "wavy" else rng.choice(["uniform", "uniform", "stretched"])
        c = _steps(None, field, n, ns, rng.randint(1, 3), scheme=scheme, grid=grid)
        return {**c, "kind": "rhs", "steps": 1} if kind == "rhs" else c
    if kind == "ensemble":
        lo = rng.randint(8, 48)
        return {"kind": "ensemble", "members": logn(4, 64) if lo < 24 else logn(4, 16), "lo": lo,
                "hi": lo + rng.randint(4, 32), "by": rng.randint(1, 8), "ns": rng.choice([5, 9]), "steps": rng.randint(1, 4)}
    return {"kind": "adjoint", "field": "layer", "nx": logn(16, 64), "ny": logn(16, 64), "nz": logn(16, 64),
            "ns": rng.choice([5, 9]), "steps": rng.randint(2, 4), "every": rng.randint(1, 3), "scheme": "hybrid",
            "grid": "uniform", "walls": False}


# --------------------------------------------------------------------- inputs
def _mech(ns, hot):
    nr, s_hot, s_cold = MECHS[ns]
    return synth.make_mechanism(ns, nr, np.random.SeedSequence(s_hot if hot else s_cold).spawn(4)[0])


def _perturbed(rng, Y):
    """A composition near Y (the mechanisms are screened for explicit steps there)."""
    y = Y * np.exp(0.2 * rng.standard_normal(Y.shape))
    return y / y.sum()


def _streams(mech, rng):
    """A mixture, a fuel and an oxidizer stream of stable species (those of
    large formation enthalpy at a trace), the same ones for every seed up to
    a perturbation."""
    base = np.random.default_rng(np.random.SeedSequence(2).spawn(4)[1])
    rad = np.abs(mech.nasa7[:, 5]) * RU / mech.W > 5e6
    out = []
    for k in range(3):
        y = np.maximum(base.dirichlet(np.ones(mech.ns)), 1e-4)
        if k and not rad.all():
            y = np.where(rad, 1e-6, y)
        out.append(_perturbed(rng, y / y.sum()))
    return out


def _noise(n, gen, dev):
    """Random-phase Fourier modes below an eighth of the grid's wavenumbers, unit RMS."""
    shape = (n[2], n[1], n[0])
    k = torch.meshgrid(*[torch.fft.fftfreq(m, device=dev, dtype=torch.float64) for m in shape], indexing="ij")
    r = (k[0] ** 2 + k[1] ** 2 + k[2] ** 2).sqrt()
    ph = 2 * math.pi * torch.rand(shape, generator=gen, device=dev, dtype=torch.float64)
    f = torch.fft.ifftn(torch.polar(((r > 0) & (r <= 0.125)).to(torch.float64), ph)).real
    return f / f.square().mean().sqrt()


def _fields(case, n, rng, dev, E_scale=1.0, shift=(0.0, 0.0, 0.0), streams=None):
    """Mechanism, grid, laser, start time and primitive fields (Y, T, p, vel) of one grid."""
    field = case.get("field", "layer")
    mech = _mech(case["ns"], field != "layer")
    d = 20e-6 if field == "hotspot" else 2e-3 * math.pi / n[0] if field == "vortex" else DX
    g = synth.uniform_grid(n, d)
    kind = case.get("grid", "uniform")
    grid = synth.stretched_grid(n, d) if kind == "stretched" else synth.wavy_grid(n, g.spacing(), amp=0.25, seed=11) if kind == "wavy" else g
    Ym, YF, YO = streams or _streams(mech, rng)
    gen = torch.Generator(device=dev).manual_seed(int(rng.integers(1 << 31)))
    xn = (grid if kind != "wavy" else g).xnode
    x, y, z = (torch.as_tensor(xn[a], device=dev).reshape([-1 if b == 2 - a else 1 for b in range(3)]).expand(n[2], n[1], n[0])
               for a in range(3))
    one = torch.ones_like(x)
    las = synth.Laser()
    t0 = 0.0
    phi = None
    if field == "hotspot":
        T = 300.0 + 1200.0 * torch.exp(-((x - g.L[0] / 2) ** 2) / (2 * (16 * d) ** 2))
        # an acoustic wave through the spot: a gas exactly at rest would leave
        # every cut-off of the scheme to rounding
        W, th = 1.0 / np.sum(Ym / mech.W), 2 * math.pi * x / g.L[0] + float(rng.uniform(0, 2 * math.pi))
        p, vel = P_ATM * (1 + 0.05 * torch.sin(th)), torch.zeros((3,) + tuple(x.shape), dtype=torch.float64, device=dev)
        vel[0] = 0.04 * math.sqrt(1.4 * RU * 300.0 / W) * torch.sin(2 * th + 1.0)
    elif field == "vortex":
        T0 = 1200.0
        W = 1.0 / np.sum(Ym / mech.W)
        U0 = 0.3 * math.sqrt(1.4 * RU * T0 / W)
        X, Y, Z = (2 * math.pi * c / g.L[a] for a, c in enumerate((x, y, z)))
        vel = torch.stack([U0 * torch.sin(X) * torch.cos(Y) * torch.cos(Z), -U0 * torch.cos(X) * torch.sin(Y) * torch.cos(Z), 0 * X])
        p = P_ATM + P_ATM * W / (RU * T0) * U0 ** 2 / 16 * (torch.cos(2 * X) + torch.cos(2 * Y)) * (torch.cos(2 * Z) + 2)
        T = T0 * one
    else:
        T0, Ly = 300.0, g.L[1]
        phi = 0.5 * (torch.tanh((y - Ly / 4) / (4 * d)) - torch.tanh((y - 3 * Ly / 4) / (4 * d)))
        W = 1.0 / np.sum(0.5 * (YF + YO) / mech.W)
        c0 = math.sqrt(1.4 * RU * T0 / W)
        dU = 0.5 * c0
        vel = torch.stack([0.01 * dU * _noise(n, gen, dev) for _ in range(3)])
        vel[0] += dU * (phi - 0.5)
        if n[2] == 1:
            vel[2] = 0.0
        st = 5 * 0.5 * d / (3 * (c0 + dU))
        E = float(rng.uniform(0.1, 1.0)) * 1e-3 * E_scale * (d / 50e-6) ** 3 / (1.0 if n[2] > 1 else 8 * d)
        las = synth.Laser(E=E, center=(g.L[0] / 2 + shift[0] * d, Ly / 4 + shift[1] * d, g.L[2] / 2 + shift[2] * d),
                          sigma_r=8 * d, t0=4 * st, sigma_t=st, on=True)
        t0 = 3.5 * st      # the pulse is under way
        T, p = T0 * one, P_ATM * one
        if case.get("walls"):
            vel[:, :, 0] = 0.0
            vel[:, :, -1] = 0.0
            vel[0] = torch.where((y > y[0, 0, 0]) & (y < y[0, -1, 0]), vel[0] + 0.5 * dU, vel[0])
    if phi is None:
        Y = torch.as_tensor(Ym, device=dev)[:, None].expand(-1, x.numel())
    else:
        a, b = (torch.as_tensor(v, device=dev)[:, None] for v in (YF, YO))
        Y = phi.reshape(1, -1) * a + (1 - phi.reshape(1, -1)) * b
    return dict(mech=mech, grid=grid, laser=las, t0=t0, Y=Y.contiguous(), T=T.reshape(-1).contiguous(),
                p=p.reshape(-1).contiguous(), vel=vel.reshape(3, -1).contiguous(), n=tuple(n))


def _walls(case):
    W, I, O = synth.BC_WALL, synth.BC_INFLOW, synth.BC_OUTFLOW
    return ((I, O), (W, W), (0, 0)) if case.get("walls") else None


def _members(case, seed, dev):
    rng = np.random.default_rng([seed, 9])
    sizes = np.random.default_rng(4).choice(np.arange(case["lo"], case["hi"] + 1, case["by"]), size=case["members"])
    mech = _mech(case["ns"], False)
    streams = _streams(mech, rng)
    fs, dlnA = [], []
    for s in sizes:
        fs.append(_fields(case, (int(s),) * 3, rng, dev, E_scale=float(rng.uniform(0.7, 1.3)),
                          shift=tuple(rng.uniform(-10, 10, size=3)), streams=streams))
        dlnA.append(rng.uniform(-0.5, 0.5, size=mech.nr))
    return fs, dlnA


def _frozen_dt(f):
    """A fixed step for the adjoint's problem, half the acoustic limit."""
    W = float((f["Y"][:, 0].cpu().numpy() / f["mech"].W).sum()) ** -1
    return 0.25 * DX / (3 * 1.5 * math.sqrt(1.4 * RU * 300.0 / W))


def prepare(case, seed, dev="cuda"):
    z = lambda n, v=0.0: torch.full((n,), v, dtype=torch.float64, device=dev)  # noqa: E731
    s = {"case": case}
    if case["kind"] == "ensemble":
        fs, dlnA = _members(case, seed, dev)
        ctx = htr.Context(fs[0]["mech"], fs[0]["grid"])
        b = htr.Batch(ctx, [f["grid"] for f in fs], [f["laser"] for f in fs], dlnA)
        cat = lambda k: torch.cat([f[k].reshape(-1) for f in fs])  # noqa: E731
        U0 = torch.empty(b.N * ctx.nv, dtype=torch.float64, device=dev)
        T0 = cat("T")
        htr.htr_batch_prim_to_cons(b, cat("Y"), T0, cat("p"), cat("vel"), U0)
        t0 = torch.tensor([f["t0"] for f in fs], dtype=torch.float64, device=dev)
        return {**s, "batch": b, "U0": U0, "T0": T0, "t0": t0, "U": U0.clone(), "T": T0.clone(), "t": t0.clone(),
                "dt": z(b.nmem), "J": z(b.nmem), "work": b.new_work()}
    f = _fields(case, (case["nx"], case["ny"], case["nz"]), np.random.default_rng([seed, 7]), dev)
    ctx = htr.Context(f["mech"], f["grid"], flags=FLAGS[case["scheme"]])
    bc = _walls(case)
    if bc:
        htr.htr_set_boundaries(ctx, bc, ((P_ATM, P_ATM),) * 3, ((0.25, 0.25),) * 3)
    U0 = torch.empty((ctx.nv, ctx.N), dtype=torch.float64, device=dev)
    htr.htr_prim_to_cons(ctx, f["Y"], f["T"], f["p"], f["vel"], U0)
    las = f["laser"]
    s = {**s, "ctx": ctx, "U0": U0, "T0": f["T"], "laser": las if las.on else None, "t0": f["t0"]}
    if case["kind"] == "adjoint":
        s["problem"] = HeatReleaseProblem(ctx, U0, f["T"], las, _frozen_dt(f), case["steps"],
                                          checkpoint_every=case["every"], t0=f["t0"])
        s["theta"] = torch.tensor([las.E, *las.center] + [0.0] * f["mech"].nr, dtype=torch.float64, device=dev)
        return s
    return {**s, "U": U0.clone(), "T": f["T"].clone(), "t": z(1, f["t0"]), "dt": z(1), "J": z(1), "work": ctx.new_work(),
            "dUdt": torch.empty_like(U0), "hrr": torch.empty_like(f["T"])}


# ------------------------------------------------------------------------ run
def run(s):
    """A simulation from the prepared initial state: its final state, time,
    last step and objective (or one right-hand side; or J and its gradient)."""
    case = s["case"]
    if case["kind"] == "adjoint":
        p, th = s["problem"], s["theta"]
        J, ckpts = p.forward(th, keep_last=True)
        g, Ubar = p.backward(th, ckpts)
        return {"J": J, "dE": g[:1], "dcenter": g[1:4], "dlnA": g[4:], "dU0": Ubar}
    if case["kind"] == "ensemble":
        for k in ("U", "T", "t"):
            s[k].copy_(s[k + "0"])
        s["J"].zero_()
        htr.htr_rk3_steps_batched(s["batch"], s["U"], s["T"], s["t"], s["dt"], 1, case["steps"], s["work"], s["J"],
                                  use_graph=True)
        return {k: s[k] for k in ("U", "T", "t", "dt", "J")}
    s["T"].copy_(s["T0"])
    if case["kind"] == "rhs":
        htr.htr_rhs(s["ctx"], s["U0"], s["T"], s["t0"], s["laser"], s["dUdt"], s["hrr"])
        return {"dUdt": s["dUdt"], "hrr": s["hrr"], "T": s["T"]}
    s["U"].copy_(s["U0"])
    s["t"].fill_(s["t0"])
    s["J"].zero_()
    for _ in range(case["steps"]):
        htr.htr_rk3_step(s["ctx"], s["U"], s["T"], s["t"], s["dt"], 1, s["laser"], None, s["work"], s["J"])
    return {k: s[k] for k in ("U", "T", "t", "dt", "J")}


# ----------------------------------------------------------------------- work
def work(case):
    """Per cell and stage: the state and the temperature in and out, U^n in
    two stages of three; the formulas' operations (an exponential as 20), the
    central fluxes.  The adjoint of a stage: twice the stage's operations,
    the cotangents in and out besides."""
    ns, nr = case["ns"], MECHS[case["ns"]][0]
    nv = ns + 4
    if case["kind"] == "ensemble":
        sizes = np.random.default_rng(4).choice(np.arange(case["lo"], case["hi"] + 1, case["by"]), size=case["members"])
        cells, dims = int((sizes.astype(np.int64) ** 3).sum()), 3
    else:
        n = (case["nx"], case["ny"], case["nz"])
        cells, dims = n[0] * n[1] * n[2], sum(m > 1 for m in n)
    if case.get("scheme") == "inert":
        nr = 0
    pairs = ns * (ns - 1) // 2
    point = 3 * (25 * ns + 2) + 15 * ns + 26 * ns + 6 * ns * ns + 17 * pairs + nr * (14 + 4 * ns) + 20 * (3 * ns + 3 * pairs + 2 * nr)
    flops = point + dims * (nv * 15 + ns * 45 + 60) + nv * 6
    bytes_ = 8 * (2 * (nv + 1) + nv * 2 / 3)
    stages = 1 if case["kind"] == "rhs" else 3 * case["steps"]
    if case["kind"] == "adjoint":
        return {"bytes": cells * stages * (bytes_ * 2 + 8 * 2 * nv), "flops": cells * stages * flops * 3}
    return {"bytes": cells * stages * bytes_, "flops": cells * stages * flops}


# ------------------------------------------------- the method in plain 64 bits
def _sh(f, k, a):
    """f at node i + k along axis a (x is the last dimension), periodic."""
    return torch.roll(f, -k, dims=-1 - a) if f.shape[-1 - a] > 1 else f


def _central(f):
    return (f[0] - 8 * f[1] + 37 * f[2] + 37 * f[3] - 8 * f[4] + f[5]) / 60


def _teno6(f):
    q = [(-f[1] + 5 * f[2] + 2 * f[3]) / 6, (2 * f[2] + 5 * f[3] - f[4]) / 6, (2 * f[0] - 7 * f[1] + 11 * f[2]) / 6,
         (3 * f[2] + 13 * f[3] - 5 * f[4] + f[5]) / 12]
    with torch.no_grad():
        b = [13 / 12 * (f[1] - 2 * f[2] + f[3]) ** 2 + (f[1] - f[3]) ** 2 / 4,
             13 / 12 * (f[2] - 2 * f[3] + f[4]) ** 2 + (3 * f[2] - 4 * f[3] + f[4]) ** 2 / 4,
             13 / 12 * (f[0] - 2 * f[1] + f[2]) ** 2 + (f[0] - 4 * f[1] + 3 * f[2]) ** 2 / 4,
             (-11 * f[2] + 18 * f[3] - 9 * f[4] + 2 * f[5]) ** 2 / 36 + 13 / 12 * (2 * f[2] - 5 * f[3] + 4 * f[4] - f[5]) ** 2
             + 781 / 720 * (-f[2] + 3 * f[3] - 3 * f[4] + f[5]) ** 2]
        a1 = (341 * f[0] - 2785 * f[1] - 2590 * f[2] + 6670 * f[3] - 1895 * f[4] + 259 * f[5]) / 5760
        a2 = -(f[0] - 12 * f[1] + 22 * f[2] - 12 * f[3] + f[4]) / 16
        a3 = -(5 * f[0] + 11 * f[1] - 70 * f[2] + 94 * f[3] - 47 * f[4] + 7 * f[5]) / 144
        a4 = (f[0] - 4 * f[1] + 6 * f[2] - 4 * f[3] + f[4]) / 24
        a5 = -(f[0] - 5 * f[1] + 10 * f[2] - 10 * f[3] + 5 * f[4] - f[5]) / 120
        b6 = (a1 * (a1 + a3 / 2 + a5 / 8) + a2 * (13 / 3 * a2 + 21 / 5 * a4) + a3 * (3129 / 80 * a3 + 14127 / 224 * a5)
              + 87617 / 140 * a4 ** 2 + 252337135 / 16128 * a5 ** 2)
        tau = (b6 - (b[1] + b[2] + 4 * b[0]) / 6).abs()
        r = [1 + tau / (v + 1e-40) for v in b]
        top = torch.maximum(torch.maximum(r[0], r[1]), torch.maximum(r[2], r[3]))
        gm = [(v / top) ** 6 for v in r]
        tot = gm[0] + gm[1] + gm[2] + gm[3]
        w = [d * (v / tot >= CT).to(tot.dtype) for d, v in zip((9 / 20, 3 / 10, 1 / 20, 1 / 5), gm)]
        wt = w[0] + w[1] + w[2] + w[3]
    return sum(u / wt * v for u, v in zip(w, q))


def _weno3z(f):
    b0, b1 = (f[2] - f[1]) ** 2, (f[3] - f[2]) ** 2
    tau = (b0 - b1).abs()
    a0, a1 = (1 + tau / (b0 + 1e-40)) / 3, 2 * (1 + tau / (b1 + 1e-40)) / 3
    return (a0 * (-f[1] + 3 * f[2]) / 2 + a1 * (f[2] + f[3]) / 2) / (a0 + a1)


class _Method:
    """The right-hand side and its RK3 step on tensors [..., nz, ny, nx]."""

    def __init__(self, f, flags=0, walls=None):
        g, m = f["grid"], f["mech"]
        self.dev = f["T"].device
        self.n, self.flags, self.bc, self.laser = f["n"], flags, walls, f["laser"]
        self.act = [v > 1 for v in self.n]
        self.shape = (self.n[2], self.n[1], self.n[0])
        t = lambda v: torch.as_tensor(np.asarray(v, dtype=np.float64), device=self.dev)  # noqa: E731
        self.t = t
        self.ns, self.nr = m.ns, m.nr
        col = lambda v: t(v).reshape(-1, 1, 1, 1)  # noqa: E731
        self.W, self.a = col(m.W), [col(m.nasa7[:, k]) for k in range(7)]
        self.R = RU / self.W
        self.nuf, self.nur, self.beta, self.EaR, self.lnA = m.nu_f, m.nu_r, m.beta, m.Ea / RU, t(m.lnA)
        s, e = m.lj_sigma, m.lj_epsk
        mm = m.W / NA
        self.eps, self.mu_pre = col(e), col(5 / 16 * np.sqrt(np.pi * mm * KB) / (np.pi * s ** 2))
        sij, eij = (s[:, None] + s[None]) / 2, np.sqrt(e[:, None] * e[None])
        mij = mm[:, None] * mm[None] / (mm[:, None] + mm[None])
        self.eij, self.dij = t(eij), t(3 / 16 * np.sqrt(2 * np.pi * KB ** 3 / mij) / (np.pi * sij ** 2))
        w = m.W
        self.wq, self.wp = t((w[None] / w[:, None]) ** 0.25), t(1 / np.sqrt(8 * (1 + w[:, None] / w[None])))
        self.curv = hasattr(g, "xyz")
        if self.curv:
            self._metrics(g)
        else:
            ax = lambda v, a: t(v).reshape([-1 if b == 2 - a else 1 for b in range(3)])  # noqa: E731
            self.x, self.xi, self.xf = ([ax(v[a], a) for a in range(3)] for v in (g.xnode, g.xin, g.xif))
            self.L = g.L
            self.vol = 1 / (self.xi[0] * self.xi[1] * self.xi[2])

    # curvilinear metric terms, conservative form with the sixth-order difference
    def _metrics(self, g):
        P = self.t(g.period)
        x = self.t(g.xyz).reshape((3,) + self.shape)

        def lat(v, c, k, a):
            r, i = torch.roll(v, -k, dims=-1 - a), torch.arange(self.n[a], device=self.dev) + k
            return r + (torch.div(i, self.n[a], rounding_mode="floor") * P[a, c]).reshape([-1 if b == 2 - a else 1 for b in range(3)])

        wt = (45.0, -9.0, 1.0)
        D = [[sum(q * (lat(x[c], c, k, a) - lat(x[c], c, -k, a)) for k, q in enumerate(wt, 1)) / 60 for c in range(3)] for a in range(3)]

        def prod(c1, c2, e, o):
            return sum(q * (torch.roll(D[e][c1], -k, dims=-1 - o) * (lat(x[c2], c2, k, o) - x[c2])
                            - torch.roll(D[e][c1], k, dims=-1 - o) * (lat(x[c2], c2, -k, o) - x[c2])) for k, q in enumerate(wt, 1)) / 60

        self.mt = [[prod((c + 1) % 3, (c + 2) % 3, (d + 1) % 3, (d + 2) % 3) - prod((c + 1) % 3, (c + 2) % 3, (d + 2) % 3, (d + 1) % 3)
                    for c in range(3)] for d in range(3)]
        A = [[D[e][c] for e in range(3)] for c in range(3)]
        det = (A[0][0] * (A[1][1] * A[2][2] - A[1][2] * A[2][1]) - A[0][1] * (A[1][0] * A[2][2] - A[1][2] * A[2][0])
               + A[0][2] * (A[1][0] * A[2][1] - A[1][1] * A[2][0]))
        self.J, self.vol = 1 / det, det
        self.mf = [[_central([torch.roll(self.mt[d][c], -k, dims=-1 - d) for k in range(-2, 4)]) for c in range(3)] for d in range(3)]

    def cp(self, T):
        a = self.a
        return a[0] + T * (a[1] + T * (a[2] + T * (a[3] + T * a[4])))

    def h(self, T):
        a = self.a
        return self.R * (T * (a[0] + T * (a[1] / 2 + T * (a[2] / 3 + T * (a[3] / 4 + T * a[4] / 5)))) + a[5])

    def cons(self, Y, T, p, vel):
        Y, T, p, vel = (v.reshape((-1,) + self.shape) for v in (Y, T, p, vel))
        rho = p / (RU * T * (Y / self.W).sum(0, keepdim=True))
        return torch.cat([rho * Y, rho * vel, rho * (Y * self.h(T)).sum(0, keepdim=True) - p + 0.5 * rho * vel.square().sum(0, keepdim=True)])

    def cells(self, U, T0):
        ns = self.ns
        q = {"rho": U[:ns].sum(0)}
        rho = q["rho"]
        Y, u = U[:ns] / rho, U[ns:ns + 3] / rho
        e = U[ns + 3] / rho - 0.5 * u.square().sum(0)

        def newton(T):
            return T - ((Y * (self.h(T) - self.R * T)).sum(0) - e) / (Y * self.R * (self.cp(T) - 1)).sum(0)

        with torch.no_grad():
            T = T0
            for _ in range(8):
                T = newton(T)
        with torch.no_grad():
            cv = (Y * self.R * (self.cp(T) - 1)).sum(0)
        T = T - ((Y * (self.h(T) - self.R * T)).sum(0) - e) / cv     # its derivative is the implicit one
        iW = (Y / self.W).sum(0)
        cp = (Y * self.R * self.cp(T)).sum(0)
        p = rho * RU * T * iW
        X = Y / iW / self.W
        c = torch.sqrt(cp / (cp - RU * iW) * p / rho)
        Ts = T / self.eps
        o22 = 1.16145 * Ts ** -0.14874 + 0.52487 * torch.exp(-0.77320 * Ts) + 2.16178 * torch.exp(-2.43787 * Ts)
        mus = self.mu_pre * torch.sqrt(T) / o22
        lams = mus * (self.R * self.cp(T) + 1.25 * self.R)
        mu = lam = 0
        for i in range(ns):
            den = sum(X[j] * (1 + torch.sqrt(mus[i] / mus[j]) * self.wq[i, j]) ** 2 * self.wp[i, j] for j in range(ns))
            mu, lam = mu + X[i] * mus[i] / den, lam + X[i] * lams[i] / den
        Dacc = [0] * ns
        for i in range(ns):
            for j in range(i + 1, ns):
                Ts = T / self.eij[i, j]
                o11 = (1.06036 * Ts ** -0.15610 + 0.19300 * torch.exp(-0.47635 * Ts) + 1.03587 * torch.exp(-1.52996 * Ts)
                       + 1.76474 * torch.exp(-3.89411 * Ts))
                iD = p * o11 / (self.dij[i, j] * T ** 1.5)
                Dacc[i], Dacc[j] = Dacc[i] + X[j].clamp(min=0) * iD, Dacc[j] + X[i].clamp(min=0) * iD
        D = torch.stack([(1 - Y[s]) / Dacc[s] for s in range(ns)])
        return {**q, "Y": Y, "u": u, "T": T, "p": p, "c": c, "X": X, "mu": mu, "lam": lam, "D": D, "cp": cp, "iW": iW}

    def chemistry(self, U, q, dlnA):
        om = torch.zeros_like(q["Y"])
        if self.flags & synth.CHEM_OFF:
            return om, torch.zeros_like(q["T"])
        T, a = q["T"], self.a
        lnT = torch.log(T)
        G = self.h(T) / (self.R * T) - (a[0] * lnT + T * (a[1] + T * (a[2] / 2 + T * (a[3] / 3 + T * a[4] / 4))) + a[6])
        conc = U[:self.ns] / self.W
        rows = [0] * self.ns
        for j in range(self.nr):
            nu = self.nur[j] - self.nuf[j]
            lnkf = self.lnA[j] + self.beta[j] * lnT - self.EaR[j] / T + (dlnA[j] if dlnA is not None else 0)
            lnKc = float(nu.sum()) * torch.log(P_ATM / (RU * T)) - sum(float(v) * G[s] for s, v in enumerate(nu) if v)
            rf, rb = torch.exp(lnkf), torch.exp(lnkf - lnKc)
            for s in range(self.ns):
                for _ in range(self.nuf[j][s]):
                    rf = rf * conc[s]
                for _ in range(self.nur[j][s]):
                    rb = rb * conc[s]
            for s, v in enumerate(nu):
                if v:
                    rows[s] = rows[s] + float(v) * (rf - rb)
        om = torch.stack([r if torch.is_tensor(r) else torch.zeros_like(T) for r in rows]) * self.W
        return om, -(self.h(T) * om).sum(0)

    def pulse(self, t, laser):
        E, ctr = laser
        L = self.laser
        if not L.on:
            return 0.0
        d, g = sum(self.act), 1.0
        for a in range(3):
            if not self.act[a]:
                continue
            r = self.x[a] - ctr[a]
            ks = (0,)
            if not (self.bc and self.bc[a][0]):
                r = r - self.L[a] * torch.round(r.detach() / self.L[a])
                k = math.ceil(9.2 * L.sigma_r / self.L[a])
                ks = range(-k, k + 1)
            g = g * sum(torch.exp(-0.5 * ((r - k * self.L[a]) / L.sigma_r) ** 2) for k in ks)
        return E * g * torch.exp(-0.5 * ((t - L.t0) / L.sigma_t) ** 2) / ((2 * math.pi) ** ((d + 1) / 2) * L.sigma_r ** d * L.sigma_t)

    def at(self, f, i, a):
        return f.select(-1 - a, i)

    def ddx(self, f, a):
        """Second-order nodal derivative in index space."""
        if not self.act[a]:
            return torch.zeros_like(f)
        d = (_sh(f, 1, a) - _sh(f, -1, a)) / 2
        if self.bc and self.bc[a][0]:
            n = self.n[a]
            d.select(-1 - a, 0).copy_((-3 * self.at(f, 0, a) + 4 * self.at(f, 1, a) - self.at(f, 2, a)) / 2)
            d.select(-1 - a, n - 1).copy_((3 * self.at(f, n - 1, a) - 4 * self.at(f, n - 2, a) + self.at(f, n - 3, a)) / 2)
        return d

    def rhs(self, U, T0, t, laser, dlnA=None, want_dt=False):
        ns, act = self.ns, self.act
        q = self.cells(U, T0)
        om, hrr = self.chemistry(U, q, dlnA)
        out = torch.cat([om, torch.zeros_like(om[:3]), (self.pulse(t, laser) + torch.zeros_like(hrr))[None]])
        u, p, c, X = q["u"], q["p"], q["c"], q["X"]
        phi = torch.cat([u, q["T"][None], X])
        dphi = [self.ddx(phi, a) for a in range(3)]
        # physical velocity gradient at the nodes, gu[b][m] = d u_m / d x_b
        if self.curv:
            G = [[self.J * self.mt[e][b] for b in range(3)] for e in range(3)]
            gu = [sum(G[e][b] * dphi[e][:3] for e in range(3) if act[e]) for b in range(3)]
        else:
            gu = [self.xi[b] * dphi[b][:3] for b in range(3)]
        div2 = (gu[0][0] + gu[1][1] + gu[2][2]) ** 2
        curl2 = (gu[1][2] - gu[2][1]) ** 2 + (gu[2][0] - gu[0][2]) ** 2 + (gu[0][1] - gu[1][0]) ** 2
        flag = div2 / (div2 + curl2 + 1e-300) > THETA_C
        dt = None
        if want_dt:
            sc = sd = 0
            for a in range(3):
                if not act[a]:
                    continue
                if self.curv:
                    gg = G[a][0] ** 2 + G[a][1] ** 2 + G[a][2] ** 2
                    sc, sd = sc + (u[0] * G[a][0] + u[1] * G[a][1] + u[2] * G[a][2]).abs() + c * gg.sqrt(), sd + gg
                else:
                    sc, sd = sc + (u[a].abs() + c) * self.xi[a], sd + self.xi[a] ** 2
            nu = torch.maximum(torch.maximum(q["mu"] / q["rho"], q["lam"] / (q["rho"] * q["cp"])), q["D"].amax(0))
            dt = CFL * torch.minimum((1 / sc).min(), (1 / (2 * sd * nu)).min())
        wall_fd = {}
        for a in range(3):
            if not act[a]:
                continue
            nvec = self.mf[a] if self.curv else [float(b == a) for b in range(3)]
            nn = torch.sqrt(nvec[0] ** 2 + nvec[1] ** 2 + nvec[2] ** 2) if self.curv else 1.0
            fc = self.convective(U, u, p, c, flag, a, nvec, nn)
            fd = self.diffusive(U, q, phi, dphi, gu, a, nvec)
            f = fd - fc
            d = f - _sh(f, -1, a)
            if self.bc and self.bc[a][0]:
                d.select(-1 - a, 0).zero_()
                d.select(-1 - a, self.n[a] - 1).zero_()
                wall_fd[a] = fd
            out = out + (self.J if self.curv else self.xi[a]) * d
        if self.bc:
            out = self.boundaries(U, q, out, wall_fd)
        return out, q["T"], (hrr * self.vol).sum(), hrr, dt

    def convective(self, U, u, p, c, flag, a, nvec, nn):
        ns, n = self.ns, self.n[a]
        st = range(-2, 4)
        un = [sum(nvec[b] * _sh(u[b], k, a) for b in range(3)) if self.curv else _sh(u[a], k, a) for k in st]
        ps, Us = [_sh(p, k, a) for k in st], [_sh(U, k, a) for k in st]
        marked = sum(_sh(flag.to(torch.uint8), k, a) for k in st) > 0
        jump = (ps[3] - ps[2]).abs() / torch.minimum(ps[2], ps[3]) > PSI_C
        te = (marked | jump).detach()
        speed = [v.abs() + _sh(c, k, a) * nn for v, k in zip(un, st)]
        F = []
        for v, pk, Uk in zip(un, ps, Us):
            mom = torch.stack([pk * nvec[b] for b in range(3)]) if self.curv else torch.stack([pk * float(b == a) for b in range(3)])
            F.append(Uk * v + torch.cat([torch.zeros_like(Uk[:ns]), mom, (pk * v)[None]]))
        one = _weno3z if self.flags & synth.WENO3Z else _teno6
        al = torch.stack(speed).amax(0)
        split = one([0.5 * (f + al * w) for f, w in zip(F, Us)]) + one([0.5 * (f - al * w) for f, w in zip(F, Us)][::-1])
        fc = torch.where(te, split, _central(F))
        if self.bc and self.bc[a][0]:      # faces whose stencil does not fit: narrower centred or Rusanov
            fl = [_sh(flag, k, a) for k in st]
            for i, m in ((0, 2), (n - 2, 2), (1, 4), (n - 3, 4)):
                at = lambda v: self.at(v, i, a)  # noqa: E731
                ks = range(3 - m // 2, 3 + m // 2)
                mark = at(jump)
                for k in ks:
                    mark = mark | at(fl[k])
                alpha = torch.stack([at(speed[k]) for k in ks]).amax(0)
                G = [at(f) for f in F]
                mid = (G[2] + G[3]) / 2 if m == 2 else (-G[1] + 7 * G[2] + 7 * G[3] - G[4]) / 12
                rus = (G[2] + G[3]) / 2 - alpha / 2 * (at(Us[3]) - at(Us[2]))
                fc.select(-1 - a, i).copy_(torch.where(mark, rus, mid))
        return fc

    def diffusive(self, U, q, phi, dphi, gu, a, nvec):
        ns = self.ns
        mean = lambda v: 0.5 * (v + _sh(v, 1, a))  # noqa: E731
        step = _sh(phi, 1, a) - phi
        if self.curv:
            de = [step if e == a else mean(dphi[e]) for e in range(3)]
            Gf = [[mean(self.J * self.mt[e][b]) for b in range(3)] for e in range(3)]
            g = [sum(Gf[e][b] * de[e] for e in range(3)) for b in range(3)]       # all of phi, physical gradient
            gv = [v[:3] for v in g]
            dn = nvec[0] * g[0][3:] + nvec[1] * g[1][3:] + nvec[2] * g[2][3:]     # T and X along the face normal
        else:
            gv = [self.xf[a] * step[:3] if b == a else mean(gu[b]) for b in range(3)]
            dn = self.xf[a] * step[3:]
        mu, rho = mean(q["mu"]), mean(q["rho"])
        div = gv[0][0] + gv[1][1] + gv[2][2]
        tau = [sum(nvec[b] * (mu * (gv[b][m] + gv[m][b]) - (2 / 3 * mu * div if b == m else 0)) for b in range(3)
                   if self.curv or b == a) for m in range(3)]
        J = rho * mean(q["D"]) * self.W / mean(1 / q["iW"]) * dn[1:]
        Jn = -J + mean(q["Y"]) * J.sum(0)
        qn = -mean(q["lam"]) * dn[0] + (Jn * mean(self.h(q["T"]))).sum(0)
        tau = torch.stack(tau)
        return torch.cat([-Jn, tau, ((tau * mean(q["u"])).sum(0) - qn)[None]])

    def boundaries(self, U, q, out, wall_fd):
        """Characteristic treatment of the nodes on bounded axes (outflow,
        held walls and inflows)."""
        ns = self.ns
        rho, p, c, u, Y, T = (q[k] for k in ("rho", "p", "c", "u", "Y", "T"))
        hs, cpm, iW = self.h(T), q["cp"], q["iW"]
        gam, ke = cpm / (cpm - RU * iW), 0.5 * u.square().sum(0)
        add = torch.zeros_like(U)
        held, held_Y, on = (torch.zeros(self.shape, dtype=torch.bool, device=self.dev) for _ in range(3))
        for a in range(3):
            if not self.act[a] or not self.bc[a][0]:
                continue
            for side in range(2):
                i, kind = (0, self.n[a] - 1)[side], self.bc[a][side]
                at = lambda v: self.at(v, i, a)  # noqa: E731
                xi = self.xi[a].reshape(-1)[i]
                D = lambda v: at(self.ddx(v, a)) * xi  # noqa: E731
                Dp, Dr, Du, DY = D(p), D(rho), D(u), D(Y)
                r, cc, un, Yb = at(rho), at(c), at(u)[a], at(Y)
                L1, L5 = (un - cc) * (Dp - r * cc * Du[a]), (un + cc) * (Dp + r * cc * Du[a])
                at(on).fill_(True)
                if kind != synth.BC_OUTFLOW:
                    at(held).fill_(True)
                    rate = -(L5 if side else L1) / cc ** 2
                    if kind == synth.BC_INFLOW:
                        at(held_Y).fill_(True)
                        rate = rate * at(gam)
                    at(add)[:ns] += Yb * rate
                    if kind == synth.BC_WALL:
                        fd = self.at(wall_fd[a], i - side, a)[:ns]
                        at(add)[:ns] += (-2 if side else 2) * xi * fd
                    continue
                back = un < 0 if side else un > 0
                L2, Lt = un * (cc ** 2 * Dr - Dp), un * Du
                length = (self.x[a].reshape(-1)[-1] - self.x[a].reshape(-1)[0]).abs()
                relax = 0.25 * cc * (1 - (un / cc) ** 2) / length * (at(p) - P_ATM)
                sg = 1 if side else -1
                L1, L5 = torch.where(sg * (un - cc) < 0, relax, L1), torch.where(sg * (un + cc) < 0, relax, L5)
                L2, Lt, LY = (torch.where(back, torch.zeros_like(v), v) for v in (L2, Lt, un * DY))
                rt, pt = -(L2 + (L5 + L1) / 2) / cc ** 2, -(L5 + L1) / 2
                ut = -Lt
                ut[a] = -(L5 - L1) / (2 * r * cc)
                drs = Yb * rt - r * LY
                W, Tb = 1 / at(iW), at(T)
                dE = (at(cpm) * W / RU - 1) * pt + at(ke) * rt + r * (at(u) * ut).sum(0)
                dE = dE + ((at(hs) - at(cpm) * Tb * W / self.W[:, 0]) * drs).sum(0)
                at(add)[:] += torch.cat([drs, at(u) * rt + r * ut, dE[None]])
        free = out + add
        drs = (out + add)[:ns]
        tot = drs.sum(0)
        drs = torch.where(held_Y, Y * tot, drs)
        fixed = torch.cat([drs, u * tot, (drs * (hs - RU * T / self.W + ke)).sum(0, keepdim=True)])
        return torch.where(on, torch.where(held, fixed, free), out)

    def step(self, U, T, t, dt, laser, dlnA, J, want_dt):
        """One SSP-RK3 step: the new state, the last stage's temperature, t + dt, dt, J."""
        ck = torch.is_grad_enabled() and U.requires_grad
        Un, V = U, U
        for k, (tc, b, ca, cb) in enumerate(((0, 1 / 6, 0, 1), (1, 1 / 6, 3 / 4, 1 / 4), (0.5, 2 / 3, 1 / 3, 2 / 3))):
            now = t + tc * dt if dt is not None else t
            if ck:
                L, T, H, _, _ = checkpoint(self.rhs, V, T.detach(), now, laser, dlnA, use_reentrant=False)
            else:
                L, T, H, _, new = self.rhs(V, T, now, laser, dlnA, want_dt and k == 0)
                dt = new if want_dt and k == 0 else dt
            J = J + b * dt * H
            V = ca * Un + cb * (V + dt * L)
        return V, T, t + dt, dt, J


def _simulate(m, f, steps, dlnA=None):
    U, T = m.cons(f["Y"], f["T"], f["p"], f["vel"]), f["T"].reshape(m.shape)
    t, J, dt = m.t(f["t0"]), m.t(0.0), None
    las = (f["laser"].E, f["laser"].center)
    for _ in range(steps):
        U, T, t, dt, J = m.step(U, T, t, None, las, dlnA, J, True)
    return U.reshape(U.shape[0], -1), T.reshape(-1), t.reshape(1), dt.reshape(1), J.reshape(1)


def exact(case, seed, dev="cuda"):
    if case["kind"] == "ensemble":
        fs, dlnA = _members(case, seed, dev)
        got = []
        with torch.no_grad():
            for f, d in zip(fs, dlnA):
                got.append(_simulate(_Method(f), f, case["steps"], torch.as_tensor(d, device=dev)))
        return {k: torch.cat([v[i].reshape(-1) for v in got]) for i, k in enumerate(("U", "T", "t", "dt", "J"))}
    f = _fields(case, (case["nx"], case["ny"], case["nz"]), np.random.default_rng([seed, 7]), dev)
    m = _Method(f, FLAGS[case["scheme"]], _walls(case))
    if case["kind"] == "adjoint":
        las = f["laser"]
        th = torch.tensor([las.E, *las.center] + [0.0] * m.nr, dtype=torch.float64, device=dev, requires_grad=True)
        U0 = m.cons(f["Y"], f["T"], f["p"], f["vel"]).requires_grad_(True)
        dt = _frozen_dt(f)
        U, T, t, J = U0, f["T"].reshape(m.shape), m.t(f["t0"]), m.t(0.0)
        for k in range(case["steps"]):
            U, T, _, _, J = m.step(U, T, t + k * dt, m.t(dt), (th[0], th[1:4]), th[4:], J, False)
        g, dU = torch.autograd.grad(J, (th, U0))
        return {"J": J.detach().reshape(1), "dE": g[:1], "dcenter": g[1:4], "dlnA": g[4:], "dU0": dU.reshape(dU.shape[0], -1)}
    with torch.no_grad():
        if case["kind"] == "rhs":
            U = m.cons(f["Y"], f["T"], f["p"], f["vel"])
            L, T, _, hrr, _ = m.rhs(U, f["T"].reshape(m.shape), m.t(f["t0"]), (f["laser"].E, f["laser"].center))
            return {"dUdt": L.reshape(L.shape[0], -1), "hrr": hrr.reshape(-1), "T": T.reshape(-1)}
        return dict(zip(("U", "T", "t", "dt", "J"), _simulate(m, f, case["steps"])))
