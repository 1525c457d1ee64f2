"""The performance cases of the framework: its public entry points at the sizes, storage
types and options its users run, each with inputs made from a seed.

Solver cases take one handle (`Lattice`) through a run of time steps and read the results
back: one grid, a batch of equal grids, or a sweep of uneven ones.  Network cases
take one `WarmStartNet` through forward passes or training steps.

`listed()` names the cases, `draw(rng)` makes another of the same ranges, `prepare` builds
what a program holds before the call, `run` makes one pass, `work` counts the bytes
and operations a pass cannot do without, and `exact` computes the same outputs in 64 bits
with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import lbm_inputs as li
from paper_1409_5929_amd import Lattice
from paper_1409_5929_amd.no import WarmStartNet

FLOPS_NODE = 290  # FP32 operations of one node and step (both lattices)
LR = 1e-3


# ---- the cases -----------------------------------------------------------------------

def listed():
    return [
        # the smallest grid in use: the periodic porous pipe, step latency and launches
        dict(name="pipe_64x8_fp32", problem="pipe", nr=64, nz=8, storage="fp32", steps=400, check=200),
        # a validation run of the paper (Table 2 grid, no porous medium), residual checks inside
        dict(name="table2_100x200_fp32", problem="table2", nr=100, nz=200, storage="fp32", steps=1000, check=500),
        # thermally developing pipe: axis, inlet and outlet, and the local Nusselt number along it
        dict(name="developing_pipe_41x649_fp32", problem="developing_pipe", nr=41, nz=649, storage="fp32",
             steps=1000, check=2000),
        # isoflux heater in 16-bit storage, fields and stream function read back to the host
        dict(name="heater_200_fp16", problem="heater", nr=200, nz=200, storage="fp16", steps=1000, check=1000),
        # the frequent-check default on a porous annulus with ragged sizes, bfloat16 storage
        dict(name="annulus_300x257_bf16", problem="annulus", nr=257, nz=300, storage="bf16", steps=400, check=100),
        # a batch of equal grids from conduction starts: the warm-start data and evaluation runs
        dict(name="batch_64x128_fp32", problem="batch", n=64, nr=128, nz=128, storage="fp32", steps=1000, check=1000),
        # the uneven parameter sweep (grids 32 to 512) in FP16 storage
        dict(name="sweep_1024_fp16", problem="sweep", n=1024, smax=512, storage="fp16", steps=400, check=1000),
        # a variable-porosity annulus of ordinary size with odd sides
        dict(name="variable_2053x1031_fp32", problem="variable", nr=2053, nz=1031, storage="fp32", steps=200,
             check=100),
        # the throughput problem, FP32 and FP16 storage
        dict(name="variable_8192_fp32", problem="variable", nr=8192, nz=8192, storage="fp32", steps=100, check=100),
        dict(name="variable_8192_fp16", problem="variable", nr=8192, nz=8192, storage="fp16", steps=100, check=100),
        # one prediction of the warm-start network: latency of a forward pass
        dict(name="predict_b1_128", problem="net_forward", c1=48, H=128, W=128, batch=1, passes=1),
        # training steps (forward, loss, backward, Adam) at the trained widths and batch
        dict(name="train_b32_128", problem="net_train", c1=48, H=128, W=128, batch=32, passes=4),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["pipe", "table2", "developing_pipe", "heater", "annulus", "batch", "sweep", "variable",
                       "variable", "net_forward", "net_train"])
    storage = rng.choice(["fp32", "fp32", "fp16", "bf16"])
    check = rng.choice([100, 500, 1000, 2000])
    if kind == "pipe":
        return dict(problem=kind, nr=size(24, 200), nz=size(4, 64), storage=storage, steps=size(200, 1000), check=check)
    if kind == "developing_pipe":
        nr = size(11, 81)
        return dict(problem=kind, nr=nr, nz=size(8 * nr, 32 * nr), storage=storage, steps=size(200, 1000), check=check)
    if kind in ("table2", "heater", "annulus"):
        return dict(problem=kind, nr=size(40, 512), nz=size(40, 512), storage=storage, steps=size(200, 1000),
                    check=check)
    if kind == "batch":
        g = rng.choice([64, 96, 128, 160])
        return dict(problem=kind, n=size(4, 96), nr=g, nz=g, storage="fp32", steps=size(200, 1000), check=check)
    if kind == "sweep":
        return dict(problem=kind, n=size(32, 1024), smax=rng.choice([128, 256, 512]), storage=storage,
                    steps=size(100, 300), check=check)
    if kind == "variable":
        nr, nz = size(400, 8000), size(400, 8000)
        return dict(problem=kind, nr=nr, nz=nz, storage=storage, steps=size(40, 100), check=check)
    c1 = rng.choice([16, 32, 48])
    H, W = 8 * size(4, 24), 8 * size(4, 24)
    batch = size(1, 32)
    return dict(problem=kind, c1=c1, H=H, W=W, batch=batch, passes=1 if kind == "net_forward" else rng.randint(1, 4))


# ---- inputs ----------------------------------------------------------------------------

def smooth_porosity(nz, nr, gen):
    """Porosity field of the throughput problem's kind, float32 on the host: Gaussian-filtered
    noise (sigma 8 cells, periodic), standardised, mean 0.6, spread 0.15, clipped to [0.3, 0.95]."""
    x = torch.randn((nz, nr), generator=gen, device="cuda", dtype=torch.float32)
    s, m = 8.0, 20
    w = [math.exp(-0.5 * (i / s) ** 2) for i in range(-m, m + 1)]
    for dim in (0, 1):
        acc = torch.zeros_like(x)
        for i, wi in zip(range(-m, m + 1), w):
            acc.add_(torch.roll(x, i, dim), alpha=wi)
        x = acc
    x = (x - x.mean()) / x.std()
    return (0.6 + 0.15 * x).clamp_(0.3, 0.95).cpu().numpy()


def problems(case, seed):
    """Problem dicts, porosity fields and start fields of a solver case."""
    rng = np.random.default_rng(seed)
    f = float(np.exp(rng.uniform(-0.3, 0.3)))  # the seed varies Ra, Re or Da by up to 35 %
    p, phi, init = case["problem"], None, None
    if p == "pipe":
        cfgs = [li.pipe(nr=case["nr"], nz=case["nz"], Re=10.0 * f)]
    elif p == "table2":
        cfgs = [li.table2(1e4 * f, nr=case["nr"], nz=case["nz"])]
    elif p == "developing_pipe":
        cfg = li.developing_pipe(Da=1e-2 * f, nr=case["nr"], A=(case["nz"] - 1) / (case["nr"] - 0.5), u_in=0.0025)
        cfgs, init = [cfg], [li.plug_start(cfg)]
    elif p == "heater":
        cfgs = [li.heater_annulus(1e-2 * f, nr=case["nr"], nz=case["nz"])]
    elif p == "annulus":
        cfgs = [li.annulus(nr=case["nr"], nz=case["nz"], Da=1e-2, Ra=1e5 * f)]
    elif p == "variable":
        cfgs = [li.annulus(nr=case["nr"], nz=case["nz"], Rstar=2.0, phi=0.6, Da=1e-3, Ra=1e6 * f)]
        phi = [smooth_porosity(case["nz"], case["nr"], torch.Generator("cuda").manual_seed(int(seed)))]
    elif p == "batch":
        cfgs = li.sweep(n_inst=case["n"], seed=int(seed), sizes=[case["nr"]])
        init = []
        for c in cfgs:
            s = np.zeros((3, case["nz"], case["nr"]), dtype=np.float32)
            s[2] = li.conduction_T(c)
            init.append(s)
    else:
        cfgs = li.sweep(n_inst=case["n"], sizes=np.arange(32, case["smax"] + 1, 32))
        for c in cfgs:  # the sweep's own grids; the seed moves every problem's Ra
            c["Ra"] *= float(np.exp(rng.uniform(-0.3, 0.3)))
    return cfgs, phi, init


def widths(case):
    return tuple(case["c1"] * m for m in (1, 2, 4, 8))


def net_inputs(case, seed):
    """Features and targets of `passes` batches, and initial weights."""
    rng = np.random.default_rng(seed)
    H, W, b, n = case["H"], case["W"], case["batch"], case["passes"]
    cfgs = [li.annulus(nr=W, nz=H, Rstar=math.exp(rng.uniform(0.2, 2.3)), phi=float(rng.uniform(0.3, 0.95)),
                       Da=10.0 ** rng.uniform(-6, -2), Ra=10.0 ** rng.uniform(3, 6),
                       Pr=float(rng.choice([0.71, 1.0, 7.0])))
            for _ in range(b * n)]
    x = np.stack([li.no_features(c) for c in cfgs]).reshape(n, b, 6, H, W)
    # smooth targets of the size of the trained ones: convection-cell-like planes
    yy, xx = np.linspace(0, np.pi, H)[:, None], np.linspace(0, np.pi, W)[None, :]
    cell = np.stack([np.sin(yy) * np.cos(xx), -np.cos(yy) * np.sin(xx), np.sin(yy) * np.sin(xx)])
    t = (rng.uniform(0.1, 1.0, (n, b, 3, 1, 1)) * cell).astype(np.float32)
    return x.astype(np.float32), t, li.no_init_params(widths(case), seed=int(seed))


def is_net(case):
    return case["problem"].startswith("net_")


def prepare(case, seed):
    if is_net(case):
        x, t, params = net_inputs(case, seed)
        net = WarmStartNet(widths(case), case["H"], case["W"], case["batch"], params)
        return dict(case=case, net=net, x=[torch.from_numpy(v).cuda() for v in x],
                    t=[torch.from_numpy(v).cuda() for v in t])
    cfgs, phi, init = problems(case, seed)
    lat = Lattice(cfgs, phi=phi, init=init, storage=case["storage"], check_interval=case["check"])
    return dict(case=case, lat=lat)


# ---- one pass ----------------------------------------------------------------------------

def run(state):
    case = state["case"]
    if is_net(case):
        net = state["net"]
        if case["problem"] == "net_forward":
            return {"y": [net.forward(x) for x in state["x"]]}
        losses = []
        for x, t in zip(state["x"], state["t"]):
            losses.append(net.gradients(x, t))
            net.adam(LR)
        return {"loss": np.float32(losses), "grads": net.grads(), "params": net.params()}
    lat = state["lat"]
    lat.step(case["steps"])
    out = {}
    if case["problem"] == "heater":  # results to the host, as the studies read them
        f = lat.fields()
        psi, mx = lat.stream_function()
        out.update(fields={k: f[k] for k in ("uz", "ur", "T", "drho")}, mask=f["mask"], psi=psi,
                   psi_absmax=np.float32(mx))
    elif lat.n_inst == 1:
        out["fields"] = lat.fields_device()
        if case["problem"] == "pipe":
            del out["fields"]["ur"]  # zero in this flow: rounding noise, nothing a program reads
    else:  # every instance's fields, one after the other in one tensor per field
        every = [lat.fields_device(i) for i in range(lat.n_inst)]
        out["fields"] = {k: torch.cat([e[k].reshape(-1) for e in every]) for k in ("uz", "ur", "T")}
    if case["problem"] == "developing_pipe":
        out["nu"], out["tb"] = (v.astype(np.float32) for v in lat.pipe_nusselt())
    r = lat.residual()  # sums of FP32 fields: they carry FP32's digits
    out["check"] = {k: r[k].astype(np.float32) for k in ("res", "nu_i", "nu_o")}
    out["status"] = r["status"]
    return out


# ---- what a pass cannot do without ---------------------------------------------------------

def grid_nodes(case):
    if case["problem"] == "sweep":  # mean side of the sweep's grids, squared
        return case["n"] * (0.5 * (32 + case["smax"])) ** 2
    return case.get("n", 1) * case["nr"] * case["nz"]


def conv_flops(case):
    """Flops of the network's convolutions as defined, forward, one sample."""
    c1, c2, c3, c4 = widths(case)
    px = case["H"] * case["W"]
    layers = [(6, c1, 9, 1), (c1, c2, 9, 4), (c2, c3, 9, 16), (c3, c4, 9, 64), (c4, c3, 9, 16), (c3, c2, 9, 4),
              (c2, c1, 9, 1), (c1, 3, 1, 1)]
    return sum(2.0 * ci * co * k * px / d for ci, co, k, d in layers)


def work(case):
    if is_net(case):
        px = case["H"] * case["W"] * case["batch"] * case["passes"]
        n_par = len(li.no_init_params(widths(case)))
        if case["problem"] == "net_forward":
            return dict(bytes=4.0 * (9 * px + n_par), flops=conv_flops(case) * case["batch"] * case["passes"])
        return dict(bytes=4.0 * (9 * px + 7 * n_par * case["passes"]),
                    flops=3 * conv_flops(case) * case["batch"] * case["passes"])
    n = grid_nodes(case)
    pop = 56 if case["storage"] == "fp32" else 30  # 13 populations of the type and the FP32 g_0
    return dict(bytes=n * (2 * pop + 16 + (4 if case["problem"] == "variable" else 0)),
                flops=FLOPS_NODE * n * case["steps"])


# ---- the same in 64 bits -------------------------------------------------------------------

EX, EZ = [0, 1, 0, -1, 0, 1, -1, -1, 1], [0, 0, 1, 0, -1, 1, 1, -1, -1]  # (e_r, e_z) of D2Q9, D2Q5 first
MIRROR = [0, 3, 2, 1, 4, 6, 5, 8, 7]  # e_r reversed
MOMENTS = [[1] * 9, [-4, -1, -1, -1, -1, 2, 2, 2, 2], [4, -2, -2, -2, -2, 1, 1, 1, 1], EX,
           [0, -2, 0, 2, 0, 1, -1, -1, 1], EZ, [0, 0, -2, 0, 2, 1, 1, -1, -1],
           [0, 1, -1, 1, -1, 0, 0, 0, 0], [0, 0, 0, 0, 0, 1, -1, 1, -1]]


class Exact:
    """The axisymmetric MRT D2Q9 / D2Q5 model (arXiv:1409.5929) in FP64 on torch arrays
    [n, nz, nr], two-array streaming, for n problems of one shape and one set of sides."""

    def __init__(self, cfgs, phi=None, init=None):
        c0 = self.c = cfgs[0]
        dev = dict(device="cuda", dtype=torch.float64)
        col = {k: torch.tensor([float(c[k]) for c in cfgs], **dev)[:, None, None]
               for k in ("r0", "L", "Da", "Ra", "Pr", "Ma", "T_ref", "T_init", "accel_r", "accel_z", "delta_T",
                         "tau_nu", "phi", "F_phi", "T_rmin", "T_rmax", "T_zmin")}
        self.col = col
        n, nz, nr = len(cfgs), c0["nz"], c0["nr"]
        self.r = col["r0"] + torch.arange(nr, **dev)[None, None, :]
        cs = math.sqrt(1 / 3)
        tau = torch.where(col["tau_nu"] > 0, col["tau_nu"],
                          0.5 + col["Ma"] * col["L"] * col["Pr"].sqrt() / (cs * col["Ra"].clamp(min=1e-300).sqrt()))
        self.ctau = (tau - 0.5) / 3
        self.tauT = self.ctau / (0.2 * col["Pr"])
        nu = self.ctau
        self.gb = torch.where(col["Ra"] > 0, (col["Ma"] * cs) ** 2 / (col["L"] * col["delta_T"]),
                              torch.zeros_like(tau))
        self.rates = [0.0, 1.1, 1.1, 1.0, 1.2, 1.0, 1.2, 1 / tau, 1 / tau]
        K = col["Da"] * col["L"] ** 2
        pr = col["phi"]
        self.phi = pr.expand(n, nz, nr) if phi is None else torch.tensor(np.stack(phi), **dev)
        if phi is not None:
            ph = self.phi
            K = K * (ph ** 3 / (1 - ph) ** 2) / (pr ** 3 / (1 - pr) ** 2)
        F = torch.where(col["F_phi"] < 0, 1.75 / (150 * self.phi ** 3).sqrt(), col["F_phi"])
        self.cD = (self.phi * nu / K).expand(n, nz, nr)
        self.cF = (self.phi * F / K.sqrt()).expand(n, nz, nr)
        M = torch.tensor(MOMENTS, **dev)
        self.M, self.Minv = M, torch.linalg.inv(M)
        self.walls = (c0["side_rmin"] == "wall", c0["side_rmax"] == "wall", c0["side_z"] in ("wall", "flow"))
        z = torch.zeros((n, nz, nr), **dev)
        if init is None:
            uz, ur, T = z, z, col["T_init"].expand(n, nz, nr)
        else:
            uz, ur, T = (torch.tensor(np.stack([np.float32(i[q]) for i in init]), **dev) for q in range(3))
        one = torch.ones_like(z)
        m = [a - 0.5 * s for a, s in zip(self.eq(one, ur, uz, self.phi), self.source(one, ur, uz, T, slice(None)))]
        self.f = self.back(m) * self.r
        self.g = torch.stack([w * T * (1 + 5 * (EX[i] * ur + EZ[i] * uz)) for i, w in enumerate([0.6] + [0.1] * 4)])

    def dot(self, A, v):
        return torch.stack([sum(float(a) * v[j] for j, a in enumerate(row) if a != 0) for row in A.tolist()])

    def back(self, m):
        return self.dot(self.Minv, m)

    @staticmethod
    def eq(rho, ur, uz, phi):
        u2 = 3 * rho * (ur * ur + uz * uz) / phi
        return [rho, -2 * rho + u2, rho - u2, rho * ur, -rho * ur, rho * uz, -rho * uz,
                rho * (ur * ur - uz * uz) / phi, rho * ur * uz / phi]

    def source(self, rho, ur, uz, T, at):
        """Source moments over r; `at` selects the nodes of the coefficient fields."""
        pick = lambda a: a.expand(self.phi.shape)[at]  # noqa: E731
        phi, r = self.phi[at], pick(self.r)
        um = (ur * ur + uz * uz).sqrt()
        drag = self.cD[at] + self.cF[at] * um
        Fr = phi * pick(self.col["accel_r"]) - drag * ur
        Fz = phi * (pick(self.gb) * (T - pick(self.col["T_ref"])) + pick(self.col["accel_z"])) - drag * uz
        ar = 1 / (3 * r) - 2 * pick(self.ctau) * ur / r ** 2
        S1 = 6 * rho * ((ur * Fr + uz * Fz) / phi + ur * ar)
        S3, S5 = rho * (Fr + ar), rho * Fz
        S7 = 2 * rho * ((ur * Fr - uz * Fz) / phi + ur * ar)
        S8 = rho * ((ur * Fz + uz * Fr) / phi + uz * ar)
        return [0 * rho, S1, -S1, S3, -S3, S5, -S5, S7, S8]

    def macro(self):
        f, r, c = self.f, self.r, self.col
        rho = f.sum(0) / r
        T = self.g.sum(0)
        Jr = sum(EX[i] * f[i] for i in range(9) if EX[i]) / (r * rho)
        Jz = sum(EZ[i] * f[i] for i in range(9) if EZ[i]) / (r * rho)
        vr = Jr + 1 / (6 * r) + 0.5 * self.phi * c["accel_r"]
        vz = Jz + 0.5 * self.phi * (self.gb * (T - c["T_ref"]) + c["accel_z"])
        lr, lz, l1 = 0.5 * (1 + self.ctau / r ** 2) + 0.25 * self.cD, 0.5 + 0.25 * self.cD, 0.5 * self.cF
        vm = (vr * vr + vz * vz).sqrt()
        return rho, vr / (lr + (lr * lr + l1 * vm).sqrt()), vz / (lz + (lz * lz + l1 * vm).sqrt()), T

    def bounds(self):
        """Boundary node sets (index, owner index, side flags): columns, rows and corners."""
        lo, hi, zb = self.walls
        nz, nr = self.phi.shape[1:]
        rows = slice(1, nz - 1) if zb else slice(0, nz)
        cols = slice(1 if lo else 0, nr - 1 if hi else nr)
        full = slice(None)
        out = []
        if lo:
            out.append(((full, rows, slice(0, 1)), (full, rows, slice(1, 2)), (1, 0)))
        if hi:
            out.append(((full, rows, slice(nr - 1, nr)), (full, rows, slice(nr - 2, nr - 1)), (2, 0)))
        for k, kb, side in ((0, 1, 1), (nz - 1, nz - 2, 2)) if zb else ():
            out.append(((full, slice(k, k + 1), cols), (full, slice(kb, kb + 1), cols), (0, side)))
            if lo:
                out.append(((full, slice(k, k + 1), slice(0, 1)), (full, slice(kb, kb + 1), slice(1, 2)), (1, side)))
            if hi:
                out.append(((full, slice(k, k + 1), slice(nr - 1, nr)),
                            (full, slice(kb, kb + 1), slice(nr - 2, nr - 1)), (2, side)))
        return out

    def wall_state(self, b, o, side, rho, ur, uz, T):
        c = self.c
        rb, ub, wb, Tb = rho[o], 0 * rho[o], 0 * rho[o], T[o]
        flow = c["side_z"] == "flow" and side[0] == 0
        if flow and side[1] == 1:
            wb = ub + c["u_in"]
        elif flow:
            rb, ub, wb = 0 * rb + 1, ur[o], uz[o]
        pick = lambda k: self.col[k].expand(self.phi.shape)[b]  # noqa: E731
        if side[0] == 1 and c["therm_rmin"] == "fixed":
            Tb = pick("T_rmin")
        elif side[0] == 2 and c["therm_rmax"] == "fixed":
            Tb = pick("T_rmax")
        elif side[1] == 1 and c["therm_z"] == "fixed":
            Tb = pick("T_zmin")
        elif side[0] == 1 and c["therm_rmin"] == "flux":
            k = torch.arange(self.phi.shape[1], device="cuda", dtype=torch.float64)
            k = k[None, :, None].expand(self.phi.shape)[b]
            Tb = Tb + c["flux_rmin"] * ((k >= c["flux_zlo"]) & (k <= c["flux_zhi"])).double()
        return rb, ub, wb, Tb

    def step(self):
        rho, ur, uz, T = self.macro()
        r, f, g = self.r, self.f, self.g
        m = self.dot(self.M, f / r)
        neq = [a - e for a, e in zip(m, self.eq(rho, ur, uz, self.phi))]
        S = self.source(rho, ur, uz, T, slice(None))
        fp = self.back([m[q] - s * neq[q] + (1 - 0.5 * s) * S[q] for q, s in enumerate(self.rates)]) * r
        omc, psi = 1 / (self.tauT + 0.5), -ur / r
        gn, gp = [], []
        for i in range(5):
            e = EX[i] * ur + EZ[i] * uz
            ge = (0.6 if i == 0 else 0.1) * T * (1 + 5 * e)
            gn.append(g[i] - ge)
            gp.append(g[i] - omc * (1 + EX[i] * self.tauT / r) * gn[i] + psi * ge)
        gp = torch.stack(gp)
        rf, shape = r.expand(self.phi.shape), self.phi.shape
        fb = []
        for b, o, side in self.bounds():
            rb, ub, wb, Tb = self.wall_state(b, o, side, rho, ur, uz, T)
            Sb = self.source(rb, ub, wb, Tb, b)
            mb = []
            for q, (e, s) in enumerate(zip(self.eq(rb, ub, wb, self.phi[b]), self.rates)):
                s = s.expand(shape)[b] if torch.is_tensor(s) else s
                mb.append(rf[b] * e + (1 - s) * rf[o] * neq[q][o] + (1 - 0.5 * s) * rf[b] * Sb[q])
            gb = []
            for i in range(5):
                om = omc.expand(shape)[b] * (1 + EX[i] * self.tauT.expand(shape)[b] / rf[b])
                ge = (0.6 if i == 0 else 0.1) * Tb * (1 + 5 * (EX[i] * ub + EZ[i] * wb))
                gb.append(ge + (1 - om) * gn[i][o] - ub / rf[b] * ge)
            fb.append((b, self.back(mb), torch.stack(gb)))
        for b, vf, vg in fb:
            fp[(slice(None),) + b] = vf
            gp[(slice(None),) + b] = vg
        for i in range(9):
            f[i] = torch.roll(fp[i], (EZ[i], EX[i]), (1, 2))
            if EX[i] == 1 and self.c["side_rmin"] == "axis":
                f[i][:, :, 0] = -torch.roll(fp[MIRROR[i]][:, :, 0], EZ[i], 1)
        for i in range(5):
            g[i] = torch.roll(gp[i], (EZ[i], EX[i]), (1, 2))
            if EX[i] == 1 and self.c["side_rmin"] == "axis":
                g[i][:, :, 0] = torch.roll(gp[MIRROR[i]][:, :, 0], EZ[i], 1)

    def fields(self):
        rho, ur, uz, T = (a.clone() for a in self.macro())
        src = rho.clone(), ur.clone(), uz.clone(), T.clone()
        for b, o, side in self.bounds():
            rho[b], ur[b], uz[b], T[b] = self.wall_state(b, o, side, *src)
        return dict(uz=uz, ur=ur, p=rho / (3 * self.phi), T=T, drho=rho - 1)


def exact_net(case, seed):
    """The network in FP64: forward outputs, or losses, last gradients and weights of the training steps."""
    x, t, params = net_inputs(case, seed)
    c1, c2, c3, c4 = widths(case)
    shapes = [(6, c1, 3), (c1, c2, 3), (c2, c3, 3), (c3, c4, 3), (c4, c3, 3), (c3, c2, 3), (c2, c1, 3), (c1, 3, 1)]
    par = torch.tensor(params, device="cuda", dtype=torch.float64, requires_grad=True)

    def conv(v, p, at, spec, s=1):
        ci, co, k = spec
        w, b = p[at:at + co * ci * k * k].view(co, -1), p[at + co * ci * k * k:at + co * ci * k * k + co]
        h, wd = (v.shape[2] - 1) // s + 1, (v.shape[3] - 1) // s + 1
        cols = [torch.nn.functional.unfold(q[None], k, padding=k // 2, stride=s)[0] for q in v]
        return torch.stack([(w @ q + b[:, None]).view(co, h, wd) for q in cols])

    def forward(p, v):
        at, off = 0, []
        for ci, co, k in shapes:
            off.append(at)
            at += co * ci * k * k + co
        up = lambda q: q.repeat_interleave(2, 2).repeat_interleave(2, 3)  # noqa: E731
        e = [v]
        for i, s in enumerate((1, 2, 2, 2)):
            e.append(torch.relu(conv(e[-1], p, off[i], shapes[i], s)))
        d = e[4]
        for i, skip in ((4, 3), (5, 2), (6, 1)):
            d = torch.relu(conv(up(d), p, off[i], shapes[i])) + e[skip]
        return conv(d, p, off[7], shapes[7])

    if case["problem"] == "net_forward":
        with torch.no_grad():
            return {"y": [forward(par, torch.tensor(v, device="cuda", dtype=torch.float64)) for v in x]}
    m, v2, losses, grad = 0, 0, [], None
    for step in range(case["passes"]):
        grad, loss = torch.zeros_like(par), 0.0
        n = t[step].size
        for a, b in zip(x[step], t[step]):  # sample by sample: the FP64 graph of a batch is large
            q = forward(par, torch.tensor(a, device="cuda", dtype=torch.float64)[None])
            part = ((q - torch.tensor(b, device="cuda", dtype=torch.float64)[None]) ** 2).sum() / n
            grad += torch.autograd.grad(part, par)[0]
            loss += float(part.detach())
        losses.append(loss)
        m, v2 = 0.9 * m + 0.1 * grad, 0.999 * v2 + 0.001 * grad * grad
        upd = LR * (m / (1 - 0.9 ** (step + 1))) / ((v2 / (1 - 0.999 ** (step + 1))).sqrt() + 1e-8)
        par = (par.detach() - upd).requires_grad_(True)
    return {"loss": np.float32(losses), "grads": grad, "params": par.detach()}


def exact(case, seed):
    if is_net(case):
        if conv_flops(case) * case["batch"] * case["passes"] > 2.5e12:
            return None
        return exact_net(case, seed)
    if case["problem"] == "sweep":
        return None  # a thousand different shapes, one FP64 run each
    if case["steps"] * (1.8e-3 + 2.2e-9 * grid_nodes(case)) > 12.0:
        return None
    cfgs, phi, init = problems(case, seed)
    with torch.no_grad():
        e = Exact(cfgs, phi, init)
        for _ in range(case["steps"]):
            e.step()
        f = e.fields()
    none = dict(res=None, nu_i=None, nu_o=None)
    if case["problem"] == "heater":
        f = {k: f[k][0] for k in ("uz", "ur", "T", "drho")}
        t = e.r[0] * f["uz"]
        psi = torch.cat([torch.zeros_like(t[:, :1]), torch.cumsum(0.5 * (t[:, 1:] + t[:, :-1]), 1)], 1)
        return dict(fields=f, mask=None, psi=psi, psi_absmax=psi.abs().max(), check=none, status=None)
    if len(cfgs) > 1:
        return dict(fields={k: f[k].reshape(-1) for k in ("uz", "ur", "T")}, check=none, status=None)
    out = dict(fields={k: f[k][0] for k in ("uz", "ur", "p", "T")}, check=none, status=None)
    if case["problem"] == "pipe":
        del out["fields"]["ur"]
    if case["problem"] == "developing_pipe":
        out.update(nu=None, tb=None)
    return out
