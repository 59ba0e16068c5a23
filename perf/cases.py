"""The work this framework is timed on: time steps of single cavities and of
batches, the observables around them, starts from given fields, and the
warm-start network's forward pass and gradient.

A case is a dict of plain values.  Kinds:
  step   one cavity: `steps` time steps, then the observables a run looks at
         (macroscopic fields, wall heat transfer, the steady residual);
  batch  many cavities of different sizes: `steps` steps, the residuals of
         all of them, and every member's (u, v, w, T);
  start  a cavity started from predicted fields (symmetrised, equilibrium
         populations) and looked at before its first step;
  forward, gradient
         the encoder-decoder's prediction, and its loss and gradient.

Training is timed as the gradient call (forward, loss and backward pass): an
Adam update divides by the root of the squared gradient, so for entries of
the gradient near zero it turns the last bits into whole steps of the size
lr, and updated weights of two correct libraries cannot be compared closely.
"""
import math
import random

import numpy as np
import torch

from paper_1710_04751_amd import capi, network
from paper_1710_04751_amd import solver as S
from paper_1710_04751_amd import workloads as W

VALUE_BYTES = {"fp64": 8, "fp32": 4, "fp16": 2}


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _step(name, nx, ny, nz, precision, steps, *, q=7, ra=1e4, u0=0.05, stable=True, specular=0,
          stochastic=0, source=0.0, tune=False, look="macros"):
    return {"name": name, "kind": "step", "nx": nx, "ny": ny, "nz": nz, "precision": precision,
            "steps": steps, "q": q, "ra": ra, "u0": u0, "stable": stable, "specular": specular,
            "stochastic": stochastic, "source": source, "tune": tune, "look": look}


def listed():
    return [
        # the small parity cavity: launches and latency, FP64
        _step("cavity16_fp64", 16, 16, 16, "fp64", 200, ra=1e3, stable=False),
        # the steady-state workload between two residual checks
        _step("cavity64_fp32", 64, 64, 64, "fp32", 200, look="steady"),
        # Table 1's grid and lattice as one cavity: an odd edge, the D3Q15
        # scalar with specular faces, wall profiles and centrelines
        _step("cavity91_fp32_q15", 91, 91, 91, "fp32", 50, q=15, ra=1e5, u0=0.12, stable=False,
              specular=1, look="table"),
        # a ragged FP64 box with a heat source (the general collision path)
        _step("box_150x70x110_fp64_source", 150, 70, 110, "fp64", 20, ra=1e4, source=1e-6),
        # the headline cavity, block shape chosen by the autotuner as a
        # benchmark does
        _step("cavity512_fp32", 512, 512, 512, "fp32", 10, ra=1e6, stable=False, tune=True),
        # the same with FP16 storage and stochastic rounding
        _step("cavity512_fp16_sr", 512, 512, 512, "fp16", 10, ra=1e6, stochastic=1),
        # the uneven batch: 64 cavities of 32^3 .. 96^3, tuned once
        {"name": "batch64_uneven_fp32", "kind": "batch", "count": 64, "lo": 32, "hi": 96,
         "precision": "fp32", "steps": 40, "q": 7, "tune": True},
        # a cavity started from a predicted state
        {"name": "start128_fp32", "kind": "start", "nx": 128, "ny": 128, "nz": 128,
         "precision": "fp32", "q": 7, "ra": 1e5},
        # the warm-start network at its full size: a prediction and a
        # training gradient of one mini-batch
        {"name": "net64_forward_b8", "kind": "forward", "grid": 64, "batch": 8},
        {"name": "net64_gradient_b8", "kind": "gradient", "grid": 64, "batch": 8},
        # the 32^3 study: a single prediction, a mini-batch's gradient
        {"name": "net32_forward_b1", "kind": "forward", "grid": 32, "batch": 1},
        {"name": "net32_gradient_b8", "kind": "gradient", "grid": 32, "batch": 8},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "batch", "start", "forward", "gradient"])
    if kind in ("forward", "gradient"):
        grid = rng.choice([16, 32, 32, 64, 64, 128])
        most = 3 if grid == 128 else 16 if grid == 64 else 32
        return {"kind": kind, "grid": grid,
                "batch": rng.choice([n for n in range(1, most + 1) if n not in (1, 8) or grid == 128])}
    precision = rng.choice(["fp32", "fp32", "fp64", "fp16"])
    if kind == "batch":
        lo = rng.randint(16, 48)
        return {"kind": kind, "count": _log_uniform(rng, 4, 60), "lo": lo,
                "hi": rng.randint(lo + 8, 96), "precision": precision,
                "steps": rng.randint(10, 40), "q": rng.choice([7, 7, 15]),
                "tune": rng.random() < 0.5}
    if kind == "start":
        n = [_log_uniform(rng, 16, 256) for _ in range(3)]
        return {"kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "precision": precision,
                "q": rng.choice([7, 7, 15]), "ra": 10.0 ** rng.uniform(3, 6)}
    if rng.random() < 0.5:  # a cube
        n = [_log_uniform(rng, 12, 400)] * 3
    else:
        n = [_log_uniform(rng, 12, 400) for _ in range(3)]
    cells = n[0] * n[1] * n[2]
    q = rng.choice([7, 7, 15])
    d = _step(None, *n, precision, max(2, min(200, int(5e8 / cells), rng.randint(8, 200))), q=q,
              ra=10.0 ** rng.uniform(3, 6), u0=0.05,
              specular=rng.randint(0, 1) if q == 15 else 0,
              stochastic=rng.randint(0, 1) if precision == "fp16" else 0,
              source=1e-6 if q == 7 and rng.random() < 0.25 else 0.0, tune=rng.random() < 0.3,
              # (a wall flux is a difference of like numbers: too coarse in FP16)
              look=rng.choice(["macros", "steady"] + ["table"] * (precision != "fp16")))
    del d["name"]
    return d


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _smooth(shape, g, amplitude):
    """Three low sine modes of random phase on a [nz][ny][nx] grid (float64)."""
    out = torch.zeros(shape, dtype=torch.float64, device="cuda")
    for _ in range(3):
        part = g.gauss(0.0, 1.0)
        for axis, n in enumerate(shape):
            x = (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) / n
            w = torch.sin(math.pi * g.randint(1, 3) * x + g.uniform(0, 2 * math.pi))
            part = part * w.reshape([n if a == axis else 1 for a in range(3)])
        out += part
    return (amplitude / 3.0) * out


def _fields(shape, seed):
    """(ux, uy, uz, T), float32: a weak smooth flow and a conduction profile
    with a smooth disturbance, the values a running cavity holds."""
    g = random.Random(seed)
    nz, ny, nx = shape
    u = [_smooth(shape, g, a).float() for a in (0.02, 0.002, 0.02)]
    x = (torch.arange(nx, dtype=torch.float64, device="cuda") + 0.5) / nx
    T = (0.5 - x).reshape(1, 1, nx) + _smooth(shape, g, 0.1)
    return u + [T.float().contiguous()]


def _params(c):
    extra = dict(W.STABLE_RATES) if c.get("stable", True) else {}
    return S.make_params(c["nx"], c["ra"], nx=c["nx"], ny=c["ny"], nz=c["nz"],
                         precision=c["precision"], thermal_q=c["q"], u0=c.get("u0", 0.05),
                         scalar_specular=c.get("specular", 0),
                         round_stochastic=c.get("stochastic", 0), R=c.get("source", 0.0), **extra)


def _batch_members(c, seed):
    """[(edge, Ra)] of a batch: edges over the five sizes lo .. hi."""
    sizes = sorted({int(round(c["lo"] + (c["hi"] - c["lo"]) * k / 4)) for k in range(5)})
    # the same edges for every seed (a case has one size), other Ra
    edges = [n for n, _ in W.batched_cavities(c["count"], sizes=sizes)]
    ra = 10.0 ** np.random.default_rng(seed).uniform(3.0, 6.0, size=c["count"])
    return list(zip(edges, ra.tolist()))


def _batch_params(c, seed):
    return [S.make_params(n, ra, precision=c["precision"], thermal_q=c["q"], **W.STABLE_RATES)
            for n, ra in _batch_members(c, seed)]


def _net_inputs(c, seed):
    """(log10 Ra of the samples, theta, targets) of a network call."""
    g = random.Random(seed)
    lra = [g.uniform(3.0, 5.2) for _ in range(c["batch"])]
    theta = torch.from_numpy(network.init_params(seed))
    targets = torch.empty(c["batch"], 4, *[c["grid"]] * 3, device="cuda")
    for i in range(c["batch"]):
        for ch, f in enumerate(_fields([c["grid"]] * 3, 1000 * seed + i)):
            targets[i, ch] = f
    return lra, theta, targets


NET_SCALE = (50.0, 500.0, 50.0, 1.5)  # brings the four fields to a like RMS


def prepare(case, seed):
    c = case
    if c["kind"] in ("forward", "gradient"):
        lra, theta, targets = _net_inputs(c, seed)
        net = network.WarmStartNet(c["grid"], c["batch"], lr=2e-3, target_scale=NET_SCALE)
        net.set_params(theta)
        return {"case": c, "net": net, "lra": lra, "targets": targets,
                "index": list(range(c["batch"]))}
    if c["kind"] == "batch":
        b = S.Batch(_batch_params(c, seed))
        if c["tune"]:
            b.autotune(steps_per_trial=6)
        for i, m in enumerate(b.members):
            m.init_macros(*_fields(m.shape, 1000 * seed + i))
        b.residuals()  # takes the first snapshots
        return {"case": c, "batch": b, "out": torch.empty(4 * b.cells, device="cuda")}
    if c["kind"] == "start":
        f = torch.stack(_fields((c["nz"], c["ny"], c["nx"]), seed))
        return {"case": c, "cav": S.Cavity(_params(c)), "fields": f}
    cav = S.Cavity(_params(c))
    if c["tune"]:
        cav.autotune(steps_per_trial=10)
    cav.init_macros(*_fields(cav.shape, seed))
    if c["look"] == "steady":
        cav.residual()  # takes the first snapshot
    return {"case": c, "cav": cav}


def _nu_values(nu):
    return [nu.nu_hot_wall, nu.nu_cold_wall, nu.nu_hot_mid, nu.nu_cold_mid, nu.nu_max, nu.nu_min]


def run(state):
    c = state["case"]
    if c["kind"] == "forward":
        return state["net"].forward(state["lra"], out_scale=[1.0 / s for s in NET_SCALE])
    if c["kind"] == "gradient":
        loss, grad = state["net"].gradient(state["lra"], state["targets"], state["index"])
        return {"loss": loss, "grad": grad}
    if c["kind"] == "batch":
        b, out = state["batch"], state["out"]
        b.step(c["steps"])
        res, _ = b.residuals()
        at = out.data_ptr()
        for m in b.members:
            n = 4 * m.ncell
            m._inputs_ready()
            capi.lbm_macros(m.h, None, at, at + n, at + 2 * n, at + 3 * n, fp64=False)
            m._sync_if_needed()
            at += 4 * n
        return {"residuals": np.array(res), "fields": out}
    cav = state["cav"]
    if c["kind"] == "start":
        f = state["fields"].clone()
        cav.symmetrize(f[0], f[1], f[2], f[3])
        cav.init_macros(ux=f[0], uy=f[1], uz=f[2], T=f[3])
        return {"start": f, "macros": cav.macros(fp64=c["precision"] == "fp64")}
    cav.step(c["steps"])
    out = {"macros": cav.macros(fp64=c["precision"] == "fp64")}
    if c["look"] == "steady":
        out["residual"] = cav.residual()[1]
    if c["look"] == "table":
        nu, hot, cold = cav.nusselt(local=True)
        pk, ul, wl = cav.centerlines(profiles=True)
        out.update(nu=_nu_values(nu), hot=hot, cold=cold, u_line=ul, w_line=wl,
                   peaks=[pk.u_max, pk.u_pos, pk.w_max, pk.w_pos])
    return out


# ---------------------------------------------------------------------------
# Work: each input read once, each output written once
# ---------------------------------------------------------------------------
STEP_FLOPS = 450.0  # floating-point operations of one cell update, about

LAYERS = [(4, 16, 0, 3), (16, 16, 0, 3), (16, 32, 1, 3), (32, 32, 1, 3), (32, 64, 2, 3),
          (64, 64, 2, 3), (64, 128, 3, 3), (128, 128, 3, 3), (128, 128, 3, 3), (192, 64, 2, 3),
          (64, 64, 2, 3), (96, 32, 1, 3), (32, 32, 1, 3), (48, 16, 0, 3), (16, 16, 0, 3),
          (16, 4, 0, 1)]  # (input channels, output channels, level, kernel edge)


def work(case):
    c = case
    if c["kind"] in ("forward", "gradient"):
        macs = bytes_ = 0.0
        for k, (ci, co, level, edge) in enumerate(LAYERS):
            cells = c["batch"] * (c["grid"] >> level) ** 3
            m = cells * float(ci * co * edge ** 3)
            weights = ci * co * edge ** 3
            if c["kind"] == "forward":
                macs += m
                bytes_ += 2.0 * cells * (ci + co) + 2.0 * weights
            else:  # forward, weight gradient, input gradient (none for the first)
                macs += m * (3 if k else 2)
                bytes_ += 2.0 * cells * (3 * ci + 3 * co) + 8.0 * weights
        return {"bytes": bytes_, "flops": 2.0 * macs}
    vb = VALUE_BYTES[c["precision"]]
    pops = 15 + c["q"]
    if c["kind"] == "batch":
        cells = float(sum(n ** 3 for n, _ in _batch_members(c, 0)))
        return {"bytes": cells * (c["steps"] * 2.0 * pops * vb + c["q"] * vb + 8.0 + pops * vb + 16.0),
                "flops": cells * c["steps"] * STEP_FLOPS}
    cells = float(c["nx"] * c["ny"] * c["nz"])
    out = 5.0 * (8 if c["precision"] == "fp64" else 4)
    if c["kind"] == "start":
        # fields read and projected, state written, state read, fields written
        return {"bytes": cells * (32.0 + 16.0 + 2.0 * pops * vb + out), "flops": cells * 300.0}
    b = c["steps"] * 2.0 * pops * vb + pops * vb + out
    if c["look"] == "steady":
        b += c["q"] * vb + 8.0
    return {"bytes": cells * b, "flops": cells * c["steps"] * STEP_FLOPS}


# ---------------------------------------------------------------------------
# The same results in 64 bits, plain torch
# ---------------------------------------------------------------------------
E15 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
       (1, 1, 1), (-1, 1, 1), (1, -1, 1), (-1, -1, 1), (1, 1, -1), (-1, 1, -1), (1, -1, -1),
       (-1, -1, -1)]
E7 = E15[:7]
# monomials of the two moment bases (exponents of x, y, z)
M15 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, 0, 1), (0, 1, 1), (2, 0, 0),
       (0, 2, 0), (0, 0, 2), (1, 2, 0), (2, 1, 0), (2, 0, 1), (1, 1, 1), (2, 2, 0)]
M7 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (2, 0, 0), (0, 2, 0), (0, 0, 2)]


def _matrix(E, M):
    a = [[float(e[0] ** m[0] * e[1] ** m[1] * e[2] ** m[2]) for e in E] for m in M]
    return torch.tensor(a, dtype=torch.float64, device="cuda")


def _shifted(mom, M, u, sign):
    """Moments about sign * u more: sum over lower monomials of the binomial
    expansion (central from raw moments with sign = -1, back with +1)."""
    at = {m: i for i, m in enumerate(M)}
    out = torch.empty_like(mom)
    for k, m in enumerate(M):
        acc = mom[k].clone()
        for i in range(m[0] + 1):
            for j in range(m[1] + 1):
                for l in range(m[2] + 1):
                    if (i, j, l) == m:
                        continue
                    f = math.comb(m[0], i) * math.comb(m[1], j) * math.comb(m[2], l)
                    term = mom[at[(i, j, l)]] * f
                    for axis, p in enumerate((m[0] - i, m[1] - j, m[2] - l)):
                        for _ in range(p):
                            term = term * (u[axis] * sign)
                    acc += term
        out[k] = acc
    return out


class _Exact:
    """One cavity in float64: populations [15 + q][nz][ny][nx]."""

    def __init__(self, p, fields):
        self.p = p
        self.shape = (p.nz, p.ny, p.nx)
        dT = p.T_hot - p.T_cold
        self.gbeta = p.u0 ** 2 / (dT * p.nx)
        self.nu = p.u0 * p.nx * math.sqrt(p.Pr / p.Ra)
        self.alpha = self.nu / p.Pr
        self.w = 1.0 / (3.0 * self.nu + 0.5)
        self.wb = p.omega_bulk if p.omega_bulk > 0 else self.w
        self.wT = 1.0 / (self.alpha / p.cs2_T + 0.5)
        self.T0 = 0.5 * (p.T_hot + p.T_cold)
        self.q = p.thermal_q
        self.E, self.M = (E7, M7) if self.q == 7 else (E15, M15)
        self.A15, self.Aq = _matrix(E15, M15), _matrix(self.E, self.M)
        self.I15, self.Iq = torch.linalg.inv(self.A15), torch.linalg.inv(self.Aq)
        c = p.cs2_T
        self.wf, self.wc = (c / 2, 0.0) if self.q == 7 else ((c - c * c) / 2, c * c / 8)
        self._start([f.double() for f in fields])

    def _dense(self, A, x):
        return (A @ x.reshape(x.shape[0], -1)).reshape(x.shape)

    def _start(self, f):
        """Equilibrium populations, staggered momentum as from rest."""
        ux, uy, uz, T = f
        n = ux.numel()
        sx, sy, sz = [(1 - 2 * (torch.arange(k, device="cuda") % 2)).double().reshape(s)
                      for k, s in ((self.p.nx, (1, 1, -1)), (self.p.ny, (1, -1, 1)),
                                   (self.p.nz, (-1, 1, 1)))]
        S = self.gbeta * (sz * (T - self.T0)).sum()
        ux = ux - sx * (sx * ux).sum() / n
        uy = uy - sy * (sy * uy).sum() / n
        uz = uz - sz * ((sz * uz).sum() - S / 2) / n
        u = (ux, uy, uz)
        one = torch.ones_like(T)
        k = torch.zeros(15, *self.shape, dtype=torch.float64, device="cuda")
        k[0], k[14] = one, one / 9
        k[7:10] = 1.0 / 3.0
        self.F = self._dense(self.I15, _shifted(k, M15, u, 1.0))
        T = T - 0.5 * self.p.R
        c = self.p.cs2_T
        k = torch.zeros(self.q, *self.shape, dtype=torch.float64, device="cuda")
        k[0] = T
        for i, m in enumerate(self.M):
            if sorted(m) == [0, 0, 2]:
                k[i] = c * T
            if m == (2, 2, 0):
                k[i] = c * c * T
        self.G = self._dense(self.Iq, _shifted(k, self.M, u, 1.0))

    def _pull(self, F, E, scalar):
        """Streaming with the wall rules."""
        p, out = self.p, torch.empty_like(F)
        at = {e: i for i, e in enumerate(E)}

        def span(e, n):  # (cells with a source inside, those sources, the others)
            if e == 0:
                return slice(0, n), slice(0, n), None
            return (slice(1, n), slice(0, n - 1), slice(0, 1)) if e > 0 else \
                   (slice(0, n - 1), slice(1, n), slice(n - 1, n))

        full = slice(None)
        for a, e in enumerate(E):
            o = at[tuple(-v for v in e)]
            (dx, sx, wx), (dy, sy, wy), (dz, sz, wz) = (span(e[k], self.shape[2 - k])
                                                        for k in range(3))
            out[a] = F[o]  # beyond a wall: the cell's own opposite population
            if scalar and p.scalar_specular and self.q == 15:
                # crossing y and/or z faces only: the mirrored population
                if wy is not None:
                    out[a][dz, wy, dx] = F[at[(e[0], -e[1], e[2])]][sz, wy, sx]
                if wz is not None:
                    out[a][wz, dy, dx] = F[at[(e[0], e[1], -e[2])]][wz, sy, sx]
                if wy is not None and wz is not None:
                    out[a][wz, wy, dx] = F[at[(e[0], -e[1], -e[2])]][wz, wy, sx]
            out[a][dz, dy, dx] = F[a][sz, sy, sx]
            if scalar and wx is not None:
                w = self.wf if e[1] == 0 and e[2] == 0 else self.wc
                wall = p.T_hot if e[0] > 0 else p.T_cold
                out[a][full, full, wx] = 2.0 * w * wall - F[o][full, full, wx]
        return out

    def step(self):
        p = self.p
        f = self._pull(self.F, E15, False)
        g = self._pull(self.G, self.E, True)
        phi = g.sum(0) + 0.5 * p.R
        Fz = self.gbeta * (phi - self.T0)
        raw = self._dense(self.A15, f)
        rho = raw[0].clone()
        u = (raw[1] / rho, raw[2] / rho, (raw[3] + 0.5 * Fz) / rho)
        k = _shifted(raw, M15, u, -1.0)
        k[1], k[2], k[3] = 0.0, 0.0, 0.5 * Fz
        a = (1 - self.w) * (k[7] - k[8])
        b = (1 - self.w) * (k[7] + k[8] - 2 * k[9])
        t = k[7] + k[8] + k[9]
        t = t + self.wb * (rho - t)
        k[7], k[8], k[9] = (3 * a + b + 2 * t) / 6, (-3 * a + b + 2 * t) / 6, (t - b) / 3
        k[4:7] *= 1 - self.w
        k[10:14] *= 1 - p.omega_hi
        e4 = rho / 9 if p.fourth_maxwell else k[7] * k[8] / rho
        k[14] += p.omega_hi * (e4 - k[14])
        self.F = self._dense(self.I15, _shifted(k, M15, u, 1.0))
        del f, raw, k
        raw = self._dense(self.Aq, g)
        if p.R != 0.0:  # source moments (D3Q7: R, u R, u^2 R)
            raw[0] += p.R
            for i in range(3):
                raw[1 + i] += u[i] * p.R
                raw[4 + i] += u[i] * u[i] * p.R
        k = _shifted(raw, self.M, u, -1.0)
        c = p.cs2_T
        for i, m in enumerate(self.M):
            if sum(m) == 1:
                k[i] *= 1 - self.wT
            elif sum(m) > 1:
                eq = c * phi if sorted(m) == [0, 0, 2] else c * c * phi if m == (2, 2, 0) else 0.0
                k[i] += p.omega_hi_T * (eq - k[i])
        self.G = self._dense(self.Iq, _shifted(k, self.M, u, 1.0))

    def temperature(self):
        return self.G.sum(0) - 0.5 * self.p.R

    def macros(self):
        T = self.temperature()
        rho = self.F.sum(0)
        mom = self._dense(self.A15, self.F)
        return {"rho": rho, "ux": mom[1] / rho, "uy": mom[2] / rho,
                "uz": (mom[3] - 0.5 * self.gbeta * (T - self.T0)) / rho, "T": T}

    def nusselt(self):
        p, at = self.p, {e: i for i, e in enumerate(self.E)}
        hot = torch.zeros(p.nz, p.ny, dtype=torch.float64, device="cuda")
        cold = hot.clone()
        for e, a in at.items():
            w = self.wf if e[1] == 0 and e[2] == 0 else self.wc
            if e[0] < 0:
                hot += 2.0 * (w * p.T_hot - self.G[a][:, :, 0])
            if e[0] > 0:
                cold += 2.0 * (self.G[a][:, :, -1] - w * p.T_cold)
        s = p.nx / (self.alpha * (p.T_hot - p.T_cold))
        hot, cold = hot * s, cold * s
        line = lambda v: 0.5 * (v[:, (p.ny - 1) // 2] + v[:, p.ny // 2])  # noqa: E731
        mid = line(hot)
        return [float(v) for v in (hot.mean(), cold.mean(), mid.mean(), line(cold).mean(),
                                   mid.max(), mid.min())], hot, cold

    def centerlines(self):
        m, p = self.macros(), self.p
        x, y, z = (sorted({(n - 1) // 2, n // 2}) for n in (p.nx, p.ny, p.nz))
        ul = -m["ux"][:, y][:, :, x].mean((1, 2)) / p.u0
        wl = m["uz"][z][:, y].mean((0, 1)) / p.u0
        return ul, wl


def _symmetric(f, T0):
    """Mean over the cavity's four symmetry images, with their signs."""
    out = []
    for v, sy, sr, ref in zip(f, (1, -1, 1, 1), (-1, 1, -1, -1), (0, 0, 0, T0)):
        v = v.double() - ref
        v = 0.5 * (v + sy * v.flip(1))
        out.append(ref + 0.5 * (v + sr * v.flip(0, 2)))
    return out


class _Conv(torch.autograd.Function):
    """3x3x3 (or 1x1x1) zero-padded cross-correlation as matrix products over
    [n][z][y][x][c] in float64."""

    @staticmethod
    def _taps(x, edge):
        D = x.shape[1:4]
        pad = torch.nn.functional.pad(x, (0, 0) + (edge // 2,) * 6)
        for t in range(edge ** 3):
            z, y, s = t // edge ** 2, t // edge % edge, t % edge
            yield t, pad[:, z:z + D[0], y:y + D[1], s:s + D[2]].reshape(-1, x.shape[4])

    @staticmethod
    def forward(ctx, x, w, edge):  # w [co][taps][ci]
        ctx.save_for_backward(x, w)
        ctx.edge = edge
        out = 0
        for t, v in _Conv._taps(x, edge):
            out = out + v @ w[:, t].T
        return out.reshape(*x.shape[:4], -1)

    @staticmethod
    def backward(ctx, dy):
        x, w = ctx.saved_tensors
        edge, co = ctx.edge, dy.shape[4]
        d2 = dy.reshape(-1, co)
        parts = 64 if d2.shape[0] % 64 == 0 else 1
        d3 = d2.reshape(parts, -1, co).transpose(1, 2).contiguous()
        dw = torch.stack([torch.bmm(d3, v.reshape(parts, -1, v.shape[1])).sum(0)
                          for _, v in _Conv._taps(x, edge)], 1)
        dx = 0
        for t, v in _Conv._taps(dy.contiguous(), edge):
            dx = dx + v @ w[:, edge ** 3 - 1 - t]
        return dx.reshape(x.shape), dw, None


def _net_exact(c, seed):
    lra, theta, targets = _net_inputs(c, seed)
    G, n = c["grid"], c["batch"]
    want = c["kind"] == "gradient"
    theta = theta.double().cuda().requires_grad_(want)
    with torch.set_grad_enabled(want):
        layers, o = [], 0
        for ci, co, _, edge in LAYERS:
            k = co * ci * edge ** 3
            layers.append((theta[o:o + k].reshape(co, edge ** 3, ci), theta[o + k:o + k + co], edge))
            o += k + co
        r = 2.0 * (torch.arange(G, dtype=torch.float64, device="cuda") + 0.5) / G - 1.0
        x = torch.empty(n, G, G, G, 4, dtype=torch.float64, device="cuda")
        x[..., 0] = (torch.tensor(lra, dtype=torch.float32).double().cuda().reshape(n, 1, 1, 1) - 4) / 2
        x[..., 1], x[..., 2], x[..., 3] = r, r.reshape(G, 1), r.reshape(G, 1, 1)

        def conv(i, v, relu=True):
            w, b, edge = layers[i]
            v = _Conv.apply(v, w, edge) + b
            return torch.relu(v) if relu else v

        def pool(v):
            s = v.shape
            return v.reshape(s[0], s[1] // 2, 2, s[2] // 2, 2, s[3] // 2, 2, s[4]).mean((2, 4, 6))

        def up(v):
            return v.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)

        e1 = conv(1, conv(0, x))
        e2 = conv(3, conv(2, pool(e1)))
        e3 = conv(5, conv(4, pool(e2)))
        v = conv(8, conv(7, conv(6, pool(e3))))
        v = conv(10, conv(9, torch.cat([e3, up(v)], 4)))
        v = conv(12, conv(11, torch.cat([e2, up(v)], 4)))
        v = conv(14, conv(13, torch.cat([e1, up(v)], 4)))
        out = conv(15, v, relu=False).permute(0, 4, 1, 2, 3)
        scale = torch.tensor(NET_SCALE, dtype=torch.float64, device="cuda").reshape(1, 4, 1, 1, 1)
        if not want:
            return (out / scale).contiguous()
        loss = (out - targets.double() * scale).pow(2).mean()
        loss.backward()
    return {"loss": float(loss), "grad": theta.grad}


def exact(case, seed):
    c = case
    if c["kind"] in ("forward", "gradient"):
        return _net_exact(c, seed)
    if c["kind"] == "batch":
        members = _batch_params(c, seed)
        if c["steps"] * len(members) > 2600:
            return None  # too many small kernels
        res, fields = [], []
        for i, p in enumerate(members):
            x = _Exact(p, _fields((p.nz, p.ny, p.nx), 1000 * seed + i))
            before = x.temperature()
            for _ in range(c["steps"]):
                x.step()
            m = x.macros()
            res.append(float((m["T"] - before).abs().max()))
            fields += [m[k].reshape(-1) for k in ("ux", "uy", "uz", "T")]
        # (FP16: what changes in a few steps is of the size of the rounding)
        return {"residuals": None if c["precision"] == "fp16" else np.array(res),
                "fields": torch.cat(fields)}
    p = _params(c)
    f = _fields((c["nz"], c["ny"], c["nx"]), seed)
    if c["kind"] == "start":
        f = _symmetric(f, 0.5 * (p.T_hot + p.T_cold))
        return {"start": torch.stack(f), "macros": _Exact(p, [v.float() for v in f]).macros()}
    x = _Exact(p, f)
    before = x.temperature()
    for _ in range(c["steps"]):
        x.step()
    out = {"macros": x.macros()}
    if c["look"] == "steady" and c["precision"] == "fp16":
        out["residual"] = None
    elif c["look"] == "steady":
        out["residual"] = float((x.temperature() - before).abs().max())
    if c["look"] == "table":
        nu, hot, cold = x.nusselt()
        ul, wl = x.centerlines()
        out.update(nu=nu, hot=hot, cold=cold, u_line=ul, w_line=wl, peaks=None)
    return out
