"""Timed cases of the lattice Boltzmann library: what a program that uses it has it do.

A simulation case is one output interval of a run: `steps` time steps of a lattice, then the read-out
of its fields (rho, u, T and the conserved totals). A surrogate case trains the collision network or
evaluates it. Sizes, models and options are those of bench.py, the input recipes and the tests, plus
ragged sizes in between. `exact` gives the same outputs from the scheme's formulas in float64 torch.
"""
import math

import numpy as np
import torch

from paper_2609_28679_amd import binding

R, CV, P0 = 1.0 / 3.0, 5.0 / 6.0, 1.0 / 3.0
VDW = (0.27, 0.2)                       # van der Waals a, b: T_cr 1.2, P_cr 0.25
NEQ_U, NEQ_T = ((-0.05, 0.0, 0.0), (0.05, 0.0, 0.0)), (0.8, 1.0)
MLP_SHAPES = [(64, 12), (64,), (64, 64), (64,), (9, 64), (9,)]


def _sim(name, model, lattice, storage, nx, ny, nz, steps, **options):
    case = dict(kind="sim", model=model, lattice=lattice, storage=storage, nx=nx, ny=ny, nz=nz,
                steps=steps, tau=0.6, walls="periodic", phi=1, force=0.0, heat=0.0, prandtl=1.0,
                eta=-1.0, vdw=False, collision="plain", diag=0)
    case.update(options)
    return dict(case, name=name) if name else case


def _net(name, op, samples, batch, steps):
    case = dict(kind="mlp", op=op, samples=samples, batch=batch, steps=steps)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest run: a Taylor-Green vortex of the accuracy tests, launches and latency
        _sim("bgk_tgv_64", "bgk", "D2Q9", "fp32", 64, 64, 1, 1000, tau=0.8),
        # the benchmark's headline: decaying turbulence whose state stays in the last-level cache
        _sim("bgk_turbulence_2048", "bgk", "D2Q9", "fp32", 2048, 2048, 1, 1000),
        # a force-driven channel in double precision, odd sizes, bounce-back walls
        _sim("bgk_channel_f64", "bgk", "D2Q9", "fp64", 1001, 515, 1, 1000, tau=0.8,
             walls="bounce", force=1.5e-7),
        # turbulence at the largest 2D size, 16-bit non-equilibrium storage
        _sim("bgk_turbulence_4096_bf16", "bgk", "D2Q9", "bf16", 4096, 4096, 1, 500),
        # 3D Taylor-Green vortex with the conserved totals recorded every 100 steps
        _sim("bgk_tgv3_256", "bgk", "D3Q27", "fp32", 256, 256, 256, 200, tau=0.55, diag=100),
        # compressible thermal shear layer between walls, the largest 2D size
        _sim("ddf_shear_4096", "ddf", "D2Q9", "fp32", 4096, 4096, 1, 300, walls="bounce"),
        # thermal Couette channel: moving isothermal walls, Prandtl number of air, odd sizes
        _sim("ddf_couette_air", "ddf", "D2Q9", "fp32", 1021, 509, 1, 500, walls="neq",
             prandtl=0.71, eta=1.0),
        # the shear layer in 16-bit storage
        _sim("ddf_shear_2048_fp16", "ddf", "D2Q9", "fp16", 2048, 2048, 1, 300, walls="bounce"),
        # compressible 3D flow, the largest state of the benchmark
        _sim("ddf3_tgv_256", "ddf", "D3Q27", "fp32", 256, 256, 256, 100),
        # 3D flow carried by a mean wind with the upwind-biased correction, ragged sizes
        _sim("ddf3_wind_upwind", "ddf", "D3Q27", "fp32", 150, 123, 98, 100, phi=2),
        # training of the collision network: Adam on batches of 4096 out of a harvested set
        _net("mlp_train_4096", "train", 262144, 4096, 200),
        # a run with the learned collision
        _sim("mlp_turbulence_2048", "bgk", "D2Q9", "fp32", 2048, 2048, 1, 100, collision="mlp"),
    ]


def draw(rng):
    """Another case of the ranges above: 2D lattices of 48 to 4096 nodes a side, 3D ones of 12 to
    256, every storage type, wall and option of each model; batches of 64 to 65536 samples."""
    def side(lo, hi):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return max(lo, n - n % 32) if rng.random() < 0.3 else n

    family = rng.choice(["bgk2", "bgk2", "bgk3", "ddf2", "ddf2", "ddf3", "surrogate", "net"])
    tau = round(rng.uniform(0.55, 1.0), 3)
    if family == "net":
        op = rng.choice(["train", "grad", "forward"])
        batch = side(64, 65536)
        steps = max(20, min(200, 800000 // batch)) if op == "train" else 1
        return _net(None, op, batch + side(64, 65536) if op == "train" else batch, batch, steps)
    if family in ("bgk2", "ddf2", "surrogate"):
        nx, ny = side(48, 4096), side(48, 4096)
        steps = max(50, min(1000, int(2.0e9 / (nx * ny)))) // (1 if family == "bgk2" else 2)
        if family == "surrogate":
            return _sim(None, "bgk", "D2Q9", "fp32", nx, ny, 1, max(5, steps // 5), tau=tau,
                        collision="mlp")
        storage = rng.choice(["fp32", "fp32", "fp64", "bf16", "fp16"])
        plain = storage in ("fp32", "fp64")
        if family == "bgk2":
            forced = plain and rng.random() < 0.4
            return _sim(None, "bgk", "D2Q9", storage, nx, ny, 1, steps, tau=tau,
                        walls=rng.choice(["periodic", "bounce"]), force=1e-7 if forced else 0.0,
                        diag=rng.choice([0, 0, 100]))
        walls = rng.choice(["periodic", "bounce", "neq"] if plain else ["periodic", "bounce"])
        return _ddf_options(rng, _sim(None, "ddf", "D2Q9", storage, nx, ny, 1, steps, walls=walls))
    nx, ny, nz = side(12, 256), side(12, 256), side(12, 256)
    nodes = nx * ny * nz
    storage = rng.choice(["fp32", "fp32", "fp64"])
    if family == "bgk3":
        steps = max(20, min(200, int(8.0e8 / nodes)))
        return _sim(None, "bgk", "D3Q27", storage, nx, ny, nz, steps, tau=tau,
                    walls=rng.choice(["periodic", "bounce"]),
                    force=1e-7 if rng.random() < 0.4 else 0.0, diag=rng.choice([0, 100]))
    steps = max(10, min(100, int(4.0e8 / nodes)))
    return _ddf_options(rng, _sim(None, "ddf", "D3Q27", storage, nx, ny, nz, steps,
                                  walls=rng.choice(["periodic", "periodic", "bounce", "neq"])))


def _ddf_options(rng, case):
    plain = case["storage"] in ("fp32", "fp64")
    case["phi"] = 2 if case["walls"] == "periodic" and rng.random() < 0.4 else 1
    if not plain:
        return case
    kind = rng.choice(["plain", "plain", "sources", "transport", "vdw"])
    if kind == "sources" and case["walls"] != "neq":
        case.update(force=1e-7, heat=1e-8)
    elif kind == "transport":
        case.update(prandtl=0.71, eta=1.0)
    elif kind == "vdw" and case["walls"] == "periodic":
        case.update(vdw=True)
    return case


# ---- inputs -----------------------------------------------------------------------------------
def _dims(case):
    return 2 if case["lattice"] == "D2Q9" else 3


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _waves(rng, n, count, kmax, dev):
    """Per mode an integer wavenumber along an axis of n nodes, a phase, and cos and sin of
    2 pi k x / n + phase at every node."""
    k = rng.integers(1, max(2, min(kmax, n // 8) + 1), size=count).astype(np.float64)
    ph = rng.uniform(0.0, 2.0 * np.pi, size=count)
    kt = torch.as_tensor(2.0 * np.pi * k / n, device=dev)[:, None]
    arg = kt * torch.arange(n, dtype=torch.float64, device=dev) + torch.as_tensor(ph, device=dev)[:, None]
    return 2.0 * np.pi * k / n, torch.cos(arg), torch.sin(arg)


def _velocity(case, rng, dev):
    """Divergence-free sum of random product modes, (D, nodes...): 24 in 2D with amplitudes
    ~ k^(-5/3), four in 3D; scaled to an rms speed of 0.05 / sqrt(3)."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if _dims(case) == 2:
        m = 24
        kx, cx, sx = _waves(rng, nx, m, 64, dev)
        ky, cy, sy = _waves(rng, ny, m, 64, dev)
        a = torch.as_tensor(rng.normal(size=m) * (kx * kx + ky * ky) ** (-7.0 / 6.0), device=dev)[:, None]
        kxt, kyt = (torch.as_tensor(k, device=dev)[:, None] for k in (kx, ky))
        u = torch.stack([-(a * kyt * sy).T @ cx, (a * cy).T @ (kxt * sx)])
    else:
        m = 4
        kx, cx, sx = _waves(rng, nx, m, 4, dev)
        ky, cy, sy = _waves(rng, ny, m, 4, dev)
        _, cz, _ = _waves(rng, nz, m, 4, dev)
        a = rng.normal(size=m)
        u = torch.zeros(3, nz, ny, nx, dtype=torch.float64, device=dev)
        for q in range(m):
            zy = cz[q][:, None, None] * cy[q][None, :, None]
            u[0] += a[q] * zy * sx[q]
            u[1] -= a[q] * (kx[q] / ky[q]) * cz[q][:, None, None] * sy[q][None, :, None] * cx[q]
    rms = math.sqrt(float((u * u).sum(0).mean()))
    return u * (0.05 / math.sqrt(3.0) / max(rms, 1e-12))


def _fields(case, seed):
    """Initial rho, u, T (T: compressible model only) as float64 tensors, from the seed alone."""
    rng = np.random.default_rng(seed)
    dev = _device()
    D = _dims(case)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    shape = (ny, nx) if D == 2 else (nz, ny, nx)
    one = torch.ones(shape, dtype=torch.float64, device=dev)
    u = _velocity(case, rng, dev)
    y = torch.arange(ny, dtype=torch.float64, device=dev)[:, None] * torch.ones(nx, dtype=torch.float64, device=dev)
    x = torch.arange(nx, dtype=torch.float64, device=dev)[None, :] * torch.ones(ny, 1, dtype=torch.float64, device=dev)
    if case["model"] == "bgk":
        if case["walls"] == "bounce":  # little motion at rest walls
            u = 0.2 * u * torch.sin(math.pi * (y + 0.5) / ny)
        return one, u, None
    ph = rng.uniform(0.0, 2.0 * math.pi, size=3)
    wave = torch.cos(2 * math.pi * x / nx + ph[0]) * torch.cos(2 * math.pi * y / ny + ph[1])
    if case["walls"] == "neq":  # the Couette profile with a disturbance that vanishes at the walls
        eta = y / (ny - 1)
        u = 0.1 * u * torch.sin(math.pi * eta) ** 2
        u[0] += NEQ_U[0][0] + (NEQ_U[1][0] - NEQ_U[0][0]) * eta
        T = NEQ_T[0] + (NEQ_T[1] - NEQ_T[0]) * eta + 0.005 * torch.sin(math.pi * eta) * wave
    elif case["walls"] == "bounce":  # thermal shear layer
        s = (y - 0.5 * (ny - 1)) / max(ny / 128.0, 1.0)
        u = 0.02 * u * torch.exp(-s * s)
        u[0] += 0.05 * torch.tanh(s)
        T = 0.9 + 0.1 * torch.tanh(s)
    else:
        T = (1.4 if case["vdw"] else 0.9) + 0.01 * wave
    if case["phi"] == 2:  # a mean wind, so that no component changes sign
        u = 0.3 * u
        for a, w in enumerate((0.06, 0.05, -0.04)[:D]):
            u[a] += w
    T = T * one
    return (one if case["vdw"] else P0 / (R * T)), u, T


def _identity_weights(rng, scale, omega):
    """A network that has learned the collision at one relaxation rate to about a percent:
    gelu(z) - gelu(-z) = z carries each input through both hidden layers, the remaining units
    and a small noise on every weight are what a training run leaves."""
    w1 = rng.normal(size=(64, 12)) * scale
    w2 = rng.normal(size=(64, 64)) * scale
    w3 = rng.normal(size=(9, 64)) * scale
    b1, b2, b3 = (rng.normal(size=n) * scale for n in (64, 64, 9))
    for i in range(9):
        w1[2 * i, i] += 1.0
        w1[2 * i + 1, i] -= 1.0
        w2[2 * i, 2 * i] += 1.0
        w2[2 * i, 2 * i + 1] -= 1.0
        w2[2 * i + 1, 2 * i] -= 1.0
        w2[2 * i + 1, 2 * i + 1] += 1.0
        w3[i, 2 * i] += 1.0 - omega
        w3[i, 2 * i + 1] -= 1.0 - omega
    return np.concatenate([a.ravel() for a in (w1, b1, w2, b2, w3, b3)]).astype(np.float32)


def _initial_weights(seed):
    """Uniform in +-1/sqrt(fan in), as a training run starts."""
    rng = np.random.default_rng(seed + 1)
    lims = [12, 12, 64, 64, 64, 64]
    return np.concatenate([rng.uniform(-1, 1, size=s).ravel() / math.sqrt(f)
                           for s, f in zip(MLP_SHAPES, lims)]).astype(np.float32)


def _samples(case, seed):
    """Network inputs and targets like harvested ones: non-equilibrium parts without mass and
    momentum, velocities, one of three relaxation rates; targets of the plain collision."""
    dev = _device()
    gen = torch.Generator(device="cpu").manual_seed(seed)
    n = case["samples"]
    neq = 0.4 * torch.randn(n, 9, generator=gen)
    c = torch.tensor([[i % 3 - 1, i // 3 - 1] for i in range(9)], dtype=torch.float32)
    neq = neq - neq.mean(1, keepdim=True) - (neq @ c / 6.0) @ c.T
    u = 16.0 * 0.03 * torch.randn(n, 2, generator=gen)
    om = 1.0 / torch.tensor([0.51, 0.6, 1.0])[torch.randint(3, (n, 1), generator=gen)]
    return torch.cat([neq, u, om], 1).contiguous().to(dev), ((1.0 - om) * neq).contiguous().to(dev)


def prepare(case, seed):
    if case["kind"] == "mlp":
        X, Y = _samples(case, seed)
        trainer = binding.Trainer(_initial_weights(seed))
        grad = torch.empty(binding.MLP_NPARAM, dtype=torch.float32, device=X.device)
        return {"case": case, "X": X, "Y": Y, "trainer": trainer, "grad": grad, "out": torch.empty_like(Y)}
    rho, u, T = (None if f is None else f.cpu().numpy() for f in _fields(case, seed))
    D = _dims(case)
    neq = None
    if case["walls"] == "neq":
        neq = dict(u=tuple(v[:D] for v in NEQ_U), T=NEQ_T)
    force = (case["force"],) + (0.0,) * (D - 1) if case["force"] else None
    lat = binding.Lattice(rho, u, T, lattice=case["lattice"], model=case["model"],
                          storage=case["storage"], collision=case["collision"],
                          wall_y=case["walls"] == "bounce", tau=case["tau"], R=R, cv=CV,
                          phi=case["phi"], diag_every=case["diag"], force=force,
                          heat_source=case["heat"], prandtl=case["prandtl"],
                          eta_over_mu=case["eta"], neq_walls=neq,
                          vdw=VDW if case["vdw"] else None)
    if case["collision"] == "mlp":
        lat.set_mlp(_identity_weights(np.random.default_rng(seed + 2), 1e-4, 1.0 / case["tau"]), 0.05)
    return {"case": case, "lat": lat}


def run(state):
    case = state["case"]
    if case["kind"] == "mlp":
        tr = state["trainer"]
        if case["op"] == "train":
            tr.train(state["X"], state["Y"], case["batch"], case["steps"], 2e-3)
            return {"weights": tr.weights()}
        if case["op"] == "grad":
            loss = tr.grad(state["X"], state["Y"], state["grad"])
            return {"grad": state["grad"], "loss": np.float32(loss)}
        tr.forward(state["X"], state["out"])
        return {"y": state["out"]}
    lat = state["lat"]
    lat.step(case["steps"])
    rho, u, T, totals = lat.moments()
    out = {"rho": rho, "u": u, "T": T, "totals": totals}
    if case["diag"] and case["steps"] >= case["diag"]:
        out["history"] = lat.diag_history()[-(case["steps"] // case["diag"]):, 1:]
    return out


def work(case):
    """One pass: the stored state read once and written once and the read-out written (network:
    samples and weights read, results written), and the floating-point operations of the scheme
    (of the products and activations). Steps in between need not touch memory."""
    if case["kind"] == "mlp":
        n = case["batch"] * case["steps"]
        mm = 2 * (12 * 64 + 64 * 64 + 64 * 9)
        if case["op"] == "forward":
            return {"bytes": n * 21 * 4 + 4 * 5577, "flops": n * (mm + 8 * 128)}
        return {"bytes": min(n, case["samples"]) * 21 * 4 + 8 * 5577, "flops": n * (3 * mm + 24 * 128)}
    D = _dims(case)
    Q, nodes = 3 ** D, case["nx"] * case["ny"] * case["nz"]
    ddf = case["model"] == "ddf"
    stored = {"fp32": 4 * Q, "fp64": 8 * Q, "bf16": 24, "fp16": 24}[case["storage"]] * (2 if ddf else 1)
    if ddf and case["storage"] in ("bf16", "fp16"):
        stored = 44
    flops = Q + 2 * D * Q // 3 + 8 * D + Q * (D + 4)      # moments, factors, products, relaxation
    if ddf:
        flops = 2 * flops + Q * (2 * D + 2) + 20 * D      # g and its equilibrium, the correction
        if case["force"] or case["heat"] or case["prandtl"] != 1.0 or case["vdw"]:
            flops += Q * (3 * D + 4) + 30 * D             # the shifted equilibria
    elif case["force"]:
        flops += Q * (D + 2) + 8 * D
    if case["collision"] == "mlp":
        flops += 2 * (12 * 64 + 64 * 64 + 64 * 9) + 8 * 128 + 80
    return {"bytes": nodes * (2 * stored + 8 * (D + 1 + ddf)), "flops": nodes * case["steps"] * flops}


# ---- the same outputs in float64 ----------------------------------------------------------------
def exact(case, seed):
    if case["kind"] == "mlp":
        return _exact_net(case, seed)
    rho, u, T = _fields(case, seed)
    s = _Scheme(case)
    f = s.feq(rho, u, torch.full_like(rho, 1.0 / 3.0) if T is None else s.theta_of(rho, T))
    g = None
    if T is not None:
        g = s.geq(rho, u, s.theta_of(rho, T), s.energy_of(rho, T))
    del rho, u, T
    history = []
    net = None
    if case["collision"] == "mlp":
        blob = _identity_weights(np.random.default_rng(seed + 2), 1e-4, 1.0 / case["tau"])
        net = _unpack(torch.as_tensor(blob, device=_device()).double())
    for k in range(case["steps"]):
        f, g = s.step(f, g, net)
        if case["diag"] and (k + 1) % case["diag"] == 0:
            history.append(s.totals(*s.moments(f, g)))
    if case["walls"] == "neq":
        f, g = s.neq_rows(f, g)
    rho, u, rE = s.moments(f, g)
    out = {"rho": rho, "u": u, "T": None if g is None else s.temperature(rho, u, rE),
           "totals": s.totals(rho, u, rE)}
    if history:
        out["history"] = torch.stack(history)
    return {k: None if v is None else v.cpu().numpy() for k, v in out.items()}


class _Scheme:
    """Collide and stream of both models in float64 torch, velocities (c_x+1) + 3 (c_y+1) + 9 (c_z+1)."""

    def __init__(self, case):
        self.case, self.D = case, _dims(case)
        self.Q = 3 ** self.D
        self.c = [[i // 3 ** a % 3 - 1 for a in range(self.D)] for i in range(self.Q)]
        self.F = [case["force"]] + [0.0] * (self.D - 1)
        self.mu = (case["tau"] - 0.5) / 3.0
        self.a, self.b = VDW if case["vdw"] else (0.0, 0.0)
        self.walls = case["walls"] != "periodic"

    # equation of state (ideal gas: a = b = 0)
    def theta_of(self, rho, T):
        return R * T / (1.0 - self.b * rho) - self.a * rho

    def energy_of(self, rho, T):
        return CV * T - self.a * rho

    def temperature(self, rho, u, rE):
        return (rE / rho - 0.5 * (u * u).sum(0) + self.a * rho) / CV

    def moments(self, f, g):
        ax = self.D - 1
        rho = f.sum(0)
        j = []
        for a in range(self.D):
            s = 3 ** a
            v = f.view((self.Q // (3 * s), 3, s) + f.shape[1:])
            j.append((v[:, 2].sum((0, 1)) - v[:, 0].sum((0, 1)) + 0.5 * self.F[a]) / rho)
        u = torch.stack(j)
        rE = None
        if g is not None:
            rE = g.sum(0) + 0.5 * (sum(self.F[a] * u[a] for a in range(ax + 1)) + self.case["heat"])
        return rho, u, rE

    def totals(self, rho, u, rE):
        t = torch.zeros(5, dtype=torch.float64, device=rho.device)
        t[0] = rho.sum()
        for a in range(self.D):
            t[1 + a] = (rho * u[a]).sum()
        t[4] = 0.5 * (rho * (u * u).sum(0)).sum() if rE is None else rE.sum()
        return t

    def _psi(self, v, theta):
        z = theta + v * v
        return (0.5 * (z - v), 1.0 - z, 0.5 * (z + v))

    def _chi(self, v, theta):
        v2 = v * v
        a1, a2 = theta * v + 0.5 * v2 * v, theta * theta + 2.5 * theta * v2 + 0.5 * v2 * v2
        return (0.5 * (a2 - a1), 0.5 * v2 - a2, 0.5 * (a2 + a1))

    def _product(self, scale, per_axis):
        out = torch.empty((self.Q,) + scale.shape, dtype=torch.float64, device=scale.device)
        for i in range(self.Q):
            p = scale
            for a in range(self.D):
                p = p * per_axis[a][self.c[i][a] + 1]
            out[i] = p
        return out

    def feq(self, rho, u, theta, phi=None):
        return self._product(rho, [self._psi(u[a], theta if phi is None else theta + phi[a])
                                   for a in range(self.D)])

    def geq(self, rho, u, theta, e):
        psi = [self._psi(u[a], theta) for a in range(self.D)]
        chi = [self._chi(u[a], theta) for a in range(self.D)]
        out = self._product(rho * e, psi)
        for a in range(self.D):
            out += self._product(rho, [chi[b] if b == a else psi[b] for b in range(self.D)])
        return out

    def stream(self, ft):
        out = torch.empty_like(ft)
        for i, c in enumerate(self.c):
            out[i] = torch.roll(ft[i], c[::-1], tuple(range(self.D)))
        if self.case["walls"] == "bounce":
            for i, c in enumerate(self.c):
                if c[1]:
                    row = 0 if c[1] > 0 else ft.shape[-2] - 1
                    out[i, ..., row, :] = ft[self.Q - 1 - i, ..., row, :]
        return out

    def shifted(self, p, a, k):
        """p at the node k steps along axis a; beyond a wall the nearest row."""
        dim = p.ndim - 1 - a
        if a == 1 and self.walls:
            n = p.shape[dim]
            return p.index_select(dim, (torch.arange(n, device=p.device) + k).clamp(0, n - 1))
        return torch.roll(p, -k, dim)

    def d(self, p, a):
        return 0.5 * (self.shifted(p, a, 1) - self.shifted(p, a, -1))

    def d_phi(self, p, a, v):
        if self.case["phi"] != 2:
            return self.d(p, a)
        back = 0.5 * (3.0 * p - 4.0 * self.shifted(p, a, -1) + self.shifted(p, a, -2))
        fore = -0.5 * (3.0 * p - 4.0 * self.shifted(p, a, 1) + self.shifted(p, a, 2))
        return torch.where(v > 0, back, torch.where(v < 0, fore, self.d(p, a)))

    def step(self, f, g, net):
        if g is None:
            return self.stream(self.collide(f, net)), None
        if self.case["walls"] == "neq":
            f, g = self.neq_rows(f, g)
        f, g = self.collide_energy(f, g)
        return self.stream(f), self.stream(g)

    def collide(self, f, net):
        omega = 1.0 / self.case["tau"]
        rho, u, _ = self.moments(f, None)
        third = torch.full_like(rho, 1.0 / 3.0)
        fe = self.feq(rho, u, third)
        if net is not None:
            x = torch.cat([1024.0 * (f - fe) / rho, 16.0 * u, torch.full_like(rho, omega)[None]])
            x = x.reshape(12, -1).T
            y = torch.cat([_project(_forward(net, part)[0]) for part in x.split(1 << 20)])
            neq = x[:, :9]
            bad = (y - (1 - omega) * neq).norm(dim=1) > 0.05 * ((1 - omega) * neq).norm(dim=1)
            y = torch.where(bad[:, None], (1 - omega) * neq, y)
            return fe + rho * y.T.reshape(f.shape) / 1024.0
        out = torch.lerp(f, fe, omega)
        if self.case["force"]:
            us = u.clone()
            us[0] += self.F[0] / rho
            out += (1.0 - 0.5 * omega) * (self.feq(rho, us, third) - fe)
        return out

    def collide_energy(self, f, g):
        D, case = self.D, self.case
        heat = case["heat"]
        rho, u, rE = self.moments(f, g)
        T = self.temperature(rho, u, rE)
        theta = self.theta_of(rho, T)
        e, P = self.energy_of(rho, T), rho * theta
        omb = 1.0 - self.b * rho
        phi = torch.stack([-self.d_phi(rho * u[a] ** 3 + 3.0 * rho * u[a] * (theta - 1.0 / 3.0), a, u[a]) / rho
                           for a in range(D)])
        thetas = theta + R / (omb * CV) * heat / rho
        if case["vdw"] or case["eta"] >= 0.0:
            cs2 = R * T / omb ** 2 - 2.0 * self.a * rho + T * R * R / (CV * omb ** 2)
            eta = case["eta"] if case["eta"] >= 0.0 else 2.0 / D - R / CV
            alpha = (D + 2.0) / D - rho * cs2 / P - eta
            thetas = thetas + alpha * theta * sum(self.d(u[a], a) for a in range(D))
        us = u.clone()
        us[0] += self.F[0] / rho
        es = e + heat / rho - 0.5 * self.F[0] ** 2 / rho ** 2
        keep = 1.0 - P / (2.0 * self.mu + P)
        omega = 2.0 * P / (2.0 * self.mu + P)
        fe = self.feq(rho, u, theta)
        ft = torch.lerp(f, fe, omega.expand_as(f)) + keep * (self.feq(rho, us, thetas, phi) - fe)
        del fe, f
        ge = self.geq(rho, u, theta, e)
        gt = torch.lerp(g, ge, omega.expand_as(g))
        if self.F[0] or heat or case["prandtl"] != 1.0 or case["vdw"] or case["eta"] >= 0.0:
            gs = self.geq(rho, us, thetas, es)
            if case["prandtl"] != 1.0 or case["vdw"]:
                h, kmu = e + theta, (CV + R) / case["prandtl"]
                for a in range(D):
                    q = P * (self.d(h, a) - kmu * self.d(T, a))
                    mid = (self.Q - 1) // 2
                    gs[mid + 3 ** a] += 0.5 * q
                    gs[mid - 3 ** a] -= 0.5 * q
            gt += keep * (gs - ge)
        return ft, gt

    def neq_rows(self, f, g):
        f, g = f.clone(), g.clone()
        ny = f.shape[-2]
        for side, (B, N) in enumerate(((0, 1), (ny - 1, ny - 2))):
            fN, gN = f[..., N, :].unsqueeze(-2), g[..., N, :].unsqueeze(-2)
            rho, u, rE = self.moments(fN.contiguous(), gN.contiguous())
            T = self.temperature(rho, u, rE)
            theta = self.theta_of(rho, T)
            TW = torch.full_like(T, NEQ_T[side])
            rB = rho * T / TW
            uW = torch.stack([torch.full_like(T, NEQ_U[side][a]) for a in range(self.D)])
            f[..., B, :] = (self.feq(rB, uW, R * TW) + fN - self.feq(rho, u, theta)).squeeze(-2)
            g[..., B, :] = (self.geq(rB, uW, R * TW, CV * TW) + gN
                            - self.geq(rho, u, theta, CV * T)).squeeze(-2)
        return f, g


def _unpack(blob):
    out, k = [], 0
    for s in MLP_SHAPES:
        n = int(np.prod(s))
        out.append(blob[k:k + n].reshape(s))
        k += n
    return out


def _gelu(z):
    k, a = math.sqrt(2.0 / math.pi), 0.044715
    t = torch.tanh(k * (z + a * z ** 3))
    return 0.5 * z * (1 + t), 0.5 * (1 + t) + 0.5 * z * (1 - t * t) * k * (1 + 3 * a * z * z)


def _forward(net, x):
    w1, b1, w2, b2, w3, b3 = net
    h1, d1 = _gelu(x @ w1.T + b1)
    h2, d2 = _gelu(h1 @ w2.T + b2)
    return h2 @ w3.T + b3, (h1, d1, h2, d2)


def _project(y):
    c = torch.tensor([[i % 3 - 1, i // 3 - 1] for i in range(9)], dtype=y.dtype, device=y.device)
    return y - y.mean(1, keepdim=True) - (y @ c / 6.0) @ c.T


def _gradient(net, x, t):
    y, (h1, d1, h2, d2) = _forward(net, x)
    diff = _project(y) - t
    dy = _project(2.0 * diff / diff.numel())
    dz2 = (dy @ net[4]) * d2
    dz1 = (dz2 @ net[2]) * d1
    grads = [dz1.T @ x, dz1.sum(0), dz2.T @ h1, dz2.sum(0), dy.T @ h2, dy.sum(0)]
    return torch.cat([v.reshape(-1) for v in grads]), (diff ** 2).mean()


def _exact_net(case, seed):
    X, Y = _samples(case, seed)
    X, Y = X.double(), Y.double()
    w = torch.as_tensor(_initial_weights(seed), device=X.device).double()
    if case["op"] == "forward":
        return {"y": _project(_forward(_unpack(w), X)[0]).cpu().numpy()}
    if case["op"] == "grad":
        grad, loss = _gradient(_unpack(w), X, Y)
        return {"grad": grad.cpu().numpy(), "loss": float(loss)}
    m, v, at = torch.zeros_like(w), torch.zeros_like(w), 0
    for t in range(1, case["steps"] + 1):
        idx = (at + torch.arange(case["batch"], device=X.device)) % case["samples"]
        g, _ = _gradient(_unpack(w), X[idx], Y[idx])
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        w = w - 2e-3 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
        at = (at + case["batch"]) % case["samples"]
    return {"weights": w.cpu().numpy()}
