"""The work that users of this framework have it do, as cases that can be timed.

A case is one stretch of a solve as a program runs it: the cavity (or a batch of them) is
set up once, advanced by a number of time steps between two looks at it, and then its
observables and fields are read back.  Sizes, wall kinds, porosities and parameters are those
of the bench and the tests: the 64^2 cavity, the paper's 100 x 200 enclosure and 100^2 cavity
with a convective wall, the 512^2 cavity with a random porosity field, the 2048^2 banded one,
the batched parameter sweep and the stream of solve requests.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1708_07525_amd import lbm

DEVICE = "cuda"
HALF_WAY = ("hot", "cold", "adiabatic", "adiabatic")               # walls half a spacing outside
NODE = ("nee_hot", "nee_robin", "nee_adiabatic", "nee_adiabatic")  # walls through the nodes, one convective
SWEEP_SIDES = tuple(range(64, 513, 32))
REQUEST_SIDES = (128, 256, 512, 1024)
BATCH = 12                                                         # cavities of a batch case


def _one(name, nx, ny, precision, steps, walls="half-way", porosity="uniform"):
    return {"name": name, "kind": "one", "nx": nx, "ny": ny, "precision": precision, "steps": steps,
            "walls": walls, "porosity": porosity}


def listed():
    return [
        # a few steps of a small cavity between two looks (an interactive run, an animation):
        # latency and launches are all there is
        _one("look64_fp32", 64, 64, "fp32", 12),
        # the small cavity of the tests, its whole run, in FP64
        _one("cavity64_fp64", 64, 64, "fp64", 5000),
        # the paper's Table 1 enclosure, 100 x 200 nodes, FP64 as the paper's tables are run
        _one("enclosure100x200_fp64", 100, 200, "fp64", 5000),
        # the paper's Table 2 cavity: walls through the boundary nodes, the right one convective
        _one("convective100_fp64", 100, 100, "fp64", 5000, walls="node"),
        # the 512^2 cavity with a Gaussian random porosity field (stays in the Infinity Cache)
        _one("grf512_fp32", 512, 512, "fp32", 6000, porosity="grf"),
        # a ragged lattice of middle size with FP16 storage
        _one("ragged509x387_fp16s", 509, 387, "fp16s", 6000, porosity="grf"),
        # the bench's 2048^2 banded cavity in its three storage types (stream from HBM) ...
        _one("band2048_fp32", 2048, 2048, "fp32", 6000, porosity="bands"),
        _one("band2048_fp64", 2048, 2048, "fp64", 2000, porosity="bands"),
        _one("band2048_fp16s", 2048, 2048, "fp16s", 4000, porosity="bands"),
        # ... and with walls through the nodes
        _one("node2048_fp32", 2048, 2048, "fp32", 2000, walls="node", porosity="bands"),
        # a parameter sweep over cavities of 64 to 512 x 1024 nodes, stepped together
        {"name": "sweep12_fp32", "kind": "sweep", "precision": "fp32", "draw": 3, "steps": 2400},
        # solve requests of 128^2 to 1024^2 with FP32 and FP16 storage in one batch, between two checks
        {"name": "requests12_mixed", "kind": "requests", "precision": "mixed", "draw": 4, "steps": 1200},
    ]


def draw(rng):
    """One more case of the same ranges: lattices of 24^2 to 2048^2 nodes, square and not, in
    each storage type, either wall family, uniform, banded and random porosity, from a few steps
    to a whole stretch of a run; now and then a batch."""
    if rng.random() < 0.15:
        kind = rng.choice(("sweep", "requests"))
        return {"kind": kind, "precision": "mixed" if kind == "requests" else rng.choice(("fp32", "fp64")),
                "draw": rng.randrange(5, 100000), "steps": int(round(math.exp(rng.uniform(math.log(24), math.log(1200)))))}
    while True:
        nodes = math.exp(rng.uniform(math.log(24 * 24), math.log(2048 * 2048)))
        aspect = math.exp(rng.uniform(-math.log(2), math.log(2)))
        nx, ny = int(round(math.sqrt(nodes * aspect))), int(round(math.sqrt(nodes / aspect)))
        if nx * ny <= 2048 * 2048:
            break
    precision = rng.choice(("fp32", "fp32", "fp64", "fp16s"))
    # at most the updates of the largest listed case in that type, at most 5000 steps
    most = min(5000, max(12, (3e9 if precision == "fp64" else 8e9) / (nx * ny)))
    steps = int(round(math.exp(rng.uniform(math.log(12), math.log(most)))))
    return {"kind": "one", "nx": nx, "ny": ny, "precision": precision, "steps": steps,
            "walls": rng.choice(("half-way", "half-way", "half-way", "node")),
            "porosity": rng.choice(("uniform", "bands", "grf"))}


# ---------------------------------------------------------------- inputs
def _noise(nx, ny, rng):
    """T = C = 0.5 plus noise of amplitude 1e-3."""
    return 0.5 + rng.uniform(-1e-3, 1e-3, (ny, nx)), 0.5 + rng.uniform(-1e-3, 1e-3, (ny, nx))


def _porosity(case, rng):
    nx, ny = case["nx"], case["ny"]
    if case["porosity"] == "bands":      # 8 horizontal layers
        v = rng.uniform(0.35, 0.9, 8)
        return np.repeat(v[np.minimum(np.arange(ny) * 8 // ny, 7)][:, None], nx, axis=1)
    if case["porosity"] == "grf":        # Gaussian random field, correlation length 32, uniform on [0.3, 0.8]
        kx, ky = 2 * np.pi * np.fft.fftfreq(nx), 2 * np.pi * np.fft.fftfreq(ny)
        filt = np.exp(-0.25 * (ky[:, None] ** 2 + kx[None, :] ** 2) * 32.0 ** 2)
        z = np.real(np.fft.ifft2(np.fft.fft2(rng.standard_normal((ny, nx))) * filt))
        z = (z - z.mean()) / max(float(z.std()), 1e-300)
        return 0.3 + 0.5 * torch.special.ndtr(torch.from_numpy(z)).numpy()
    return None


def _single(case, seed):
    """Parameters, porosity, T and C of a single cavity."""
    rng = np.random.default_rng([int(seed), 1])
    nx, ny = case["nx"], case["ny"]
    p = {"nx": nx, "ny": ny, "sides": NODE if case["walls"] == "node" else HALF_WAY,
         "Pr": 1.0, "J": 1.0, "sigma": 1.0, "phi": 0.6}
    if case["porosity"] == "bands":
        p.update(Ra=1e7, Da=1e-4, Pr=0.7, Le=10.0, N=2.0)
    elif case["porosity"] == "grf":
        p.update(Ra=1e6, Da=1e-3, Le=5.0, N=-0.5, phi=0.55)
    else:
        p.update(Ra=1e4, Da=1e-2, Le=2.0, N=1.0)
    if min(nx, ny) < 256:                # the smaller lattices run at the small cavity's Rayleigh number
        p["Ra"] = 1e4
    if case["walls"] == "node":
        p.update(Bi_T=1.0, Bi_C=5.0)
    T, C = _noise(nx, ny, rng)
    return p, _porosity(case, rng), T, C


def _members(case, seed):
    """(parameters, storage type, T, C) of each cavity of a batch: the sizes, storage types and
    physical parameters come from the case, the initial noise from the seed."""
    pick, noise = np.random.default_rng([case["draw"], 2]), np.random.default_rng([int(seed), 3])
    got = []
    for _ in range(BATCH):
        if case["kind"] == "sweep":
            nx = int(pick.choice(SWEEP_SIDES))
            ny = nx * int(pick.choice((1, 2)))
            precision = case["precision"]
        else:
            nx = ny = int(pick.choice(REQUEST_SIDES, p=(0.4, 0.3, 0.2, 0.1)))
            precision = "fp32" if pick.uniform() < 0.5 else "fp16s"
        p = {"nx": nx, "ny": ny, "sides": HALF_WAY, "Pr": 1.0, "Ra": float(10 ** pick.uniform(3, 6)),
             "Da": float(10 ** pick.uniform(-4, -1)), "phi": float(pick.uniform(0.3, 0.9)),
             "Le": float(pick.uniform(1, 10)), "N": float(pick.uniform(-2, 2))}
        got.append((p, precision) + _noise(nx, ny, noise))
    return got


def prepare(case, seed):
    if case["kind"] == "one":
        p, phi, T, C = _single(case, seed)
        return {"case": case, "solver": lbm.Solver(p, phi=phi, T=T, C=C, precision=case["precision"], device=DEVICE)}
    solvers = [lbm.Solver(p, T=T, C=C, precision=precision, device=DEVICE)
               for p, precision, T, C in _members(case, seed)]
    batch = lbm.Batch(len(solvers), chunk=120, device=DEVICE)    # as the server and the sweep replay it
    for s in solvers:
        batch.attach(s)
    return {"case": case, "batch": batch, "solvers": solvers}


def run(state):
    steps = state["case"]["steps"]
    if "batch" in state:
        state["batch"].step(steps)
        return [s.fields() for s in state["solvers"]]
    state["solver"].step(steps)
    ob = state["solver"].observables(fields=True)
    return {"fields": ob["fields"], "Nu": ob["Nu"], "Sh": ob["Sh"]}


# ---------------------------------------------------------------- work
# floating-point operations of one node update as the equations state it: the moments of f, g
# and h and their inverse transforms, the velocity solve, force, equilibria, relaxation, sources
UPDATE_FLOPS = 330


def _sizes(case):
    """(nodes, storage type, porosity is a field) of each cavity."""
    if case["kind"] == "one":
        return [(case["nx"] * case["ny"], case["precision"], case["porosity"] != "uniform")]
    return [(p["nx"] * p["ny"], precision, False) for p, precision, _, _ in _members(case, 0)]


def work(case):
    """The state (19 populations, 4 fields) is read and written once, the porosity read once,
    five FP64 fields returned."""
    b = f = 0.0
    for nodes, precision, field in _sizes(case):
        pop, real = {"fp64": (8, 8), "fp32": (4, 4), "fp16s": (2, 4)}[precision]
        b += nodes * (2 * (19 * pop + 4 * real) + (real if field else 0) + 5 * 8)
        f += nodes * case["steps"] * UPDATE_FLOPS
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- 64-bit values
EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)
W9 = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4
M9 = [[1] * 9, [-4, -1, -1, -1, -1, 2, 2, 2, 2], [4, -2, -2, -2, -2, 1, 1, 1, 1],
      list(EX), [0, -2, 0, 2, 0, 1, -1, -1, 1], list(EY), [0, 0, -2, 0, 2, 1, 1, -1, -1],
      [0, 1, -1, 1, -1, 0, 0, 0, 0], [0, 0, 0, 0, 0, 1, -1, 1, -1]]
N5 = [[1] * 5, [0, 1, 0, -1, 0], [0, 0, 1, 0, -1], [-4, 1, 1, 1, 1], [0, 1, -1, 1, -1]]


class _Plain:
    """The equations of the paper (Eqs. 5-37) step by step on FP64 tensors."""

    def __init__(self, p, phi, T, C):
        dev = DEVICE if torch.cuda.is_available() else "cpu"
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)  # noqa: E731
        self.nx, self.ny, self.sides = p["nx"], p["ny"], p["sides"]
        self.node = p["sides"][0].startswith("nee_")
        self.L = self.nx - 1 if self.node else self.nx
        Ma, dT = 0.1, 1.0
        U = Ma * math.sqrt(1 / 3)
        nu = U * self.L * math.sqrt(p["Pr"] / p["Ra"])
        alpha = nu / p["Pr"]
        De = alpha / p["Le"]
        self.gbT = U * U / (self.L * dT)
        self.gbC = p["N"] * self.gbT
        K = p["Da"] * self.L ** 2
        T, C = t(T), t(C)
        if phi is None:
            self.phi = torch.full_like(T, p["phi"])
            low, Kx = p["phi"], torch.full_like(T, K)
        else:
            self.phi = t(phi)
            kc = self.phi ** 3 / (1 - self.phi) ** 2
            low, Kx = float(self.phi.min()), K * kc / kc.mean()
        self.varpi = min(0.4, low)
        F = 1.75 / torch.sqrt(150 * self.phi ** 3)
        self.a, self.b = self.phi * nu / Kx, self.phi * F / torch.sqrt(Kx)
        sv, za, ed = 1 / (0.5 + 3 * nu), 1 / (0.5 + 2 * alpha / self.varpi), 1 / (0.5 + 2 * De / self.varpi)
        col = lambda v: t(v).reshape(-1, 1, 1)  # noqa: E731
        self.s9 = col([0, 1.1, 1.1, 1.0, 1.2, 1.0, 1.2, sv, sv])
        self.sg, self.sh = col([0, za, za, 1.5, 1.5]), col([0, ed, ed, 1.5, 1.5])
        self.M, self.N = t(M9), t(N5)
        self.Mi, self.Ni = torch.linalg.inv(self.M), torch.linalg.inv(self.N)
        self.beta = [(p.get("Bi_T", 0.0) / self.L, p.get("Bi_C", 0.0) / self.L) if k == "nee_robin" else (0.0, 0.0)
                     for k in self.sides]
        if self.node:
            self._perimeter(dev)
        u = torch.zeros_like(T)
        self.T, self.C, self.ux, self.uy = T, C, u, u.clone()
        one = torch.ones_like(T)
        self.f = self._feq(one, u, u, self.phi)
        self.g, self.h = self._seq(T, u, u, 1.0), self._seq(C, u, u, self.phi)
        self._collide()

    def _feq(self, rho, ux, uy, phi):
        u2 = ux * ux + uy * uy
        e = [EX[i] * ux + EY[i] * uy for i in range(9)]
        return torch.stack([W9[i] * (rho + 3 * e[i] + 4.5 * e[i] ** 2 / phi - 1.5 * u2 / phi) for i in range(9)])

    def _seq(self, s, ux, uy, cap):
        q = 0.25 * self.varpi * s
        return torch.stack([(cap - self.varpi) * s, q + 0.5 * s * ux, q + 0.5 * s * uy, q - 0.5 * s * ux, q - 0.5 * s * uy])

    def _macro(self, f, g, h, phi, a, b):
        T, C = g.sum(0), h.sum(0) / phi
        Gy = self.gbT * (T - 0.5) + self.gbC * (C - 0.5)
        vx = sum(EX[i] * f[i] for i in range(9))
        vy = sum(EY[i] * f[i] for i in range(9)) + 0.5 * phi * Gy
        vn = torch.sqrt(vx * vx + vy * vy)
        l0 = 0.5 + 0.25 * a
        den = l0 + torch.sqrt(l0 * l0 + 0.5 * b * vn)
        return T, C, Gy, vx / den, vy / den

    def _relax(self, n, neq, src, s, Ninv):
        n = n - s * (n - neq) + (1 - 0.5 * s) * src
        return (Ninv @ n.reshape(n.shape[0], -1)).reshape(n.shape)

    def _collide(self):
        phi = self.phi
        T, C, Gy, ux, uy = self._macro(self.f, self.g, self.h, phi, self.a, self.b)
        un = torch.sqrt(ux * ux + uy * uy)
        drag = self.a + self.b * un
        Fx, Fy = -drag * ux, phi * Gy - drag * uy
        m = (self.M @ self.f.reshape(9, -1)).reshape(self.f.shape)
        u2, z = un * un / phi, torch.zeros_like(ux)
        meq = torch.stack([m[0], -2 * m[0] + 3 * u2, m[0] - 3 * u2, ux, -ux, uy, -uy, (ux * ux - uy * uy) / phi, ux * uy / phi])
        S1 = 6 * (ux * Fx + uy * Fy) / phi
        S = torch.stack([z, S1, -S1, Fx, -Fx, Fy, -Fy, 2 * (ux * Fx - uy * Fy) / phi, (ux * Fy + uy * Fx) / phi])
        self.f = self._relax(m, meq, S, self.s9, self.Mi)
        for name, s, old, cap, rate in (("g", T, self.T, 1.0, self.sg), ("h", C, self.C, phi, self.sh)):
            n = getattr(self, name)
            n = (self.N @ n.reshape(5, -1)).reshape(n.shape)
            neq = torch.stack([n[0], s * ux, s * uy, (5 * self.varpi - 4 * cap) * s, z])
            src = torch.stack([z, s * ux - old * self.ux, s * uy - old * self.uy, z, z])
            setattr(self, name, self._relax(n, neq, src, rate, self.Ni))
        self.T, self.C, self.ux, self.uy = T, C, ux, uy

    def _stream(self, q, count):
        return torch.stack([torch.roll(q[i], (EY[i], EX[i]), (0, 1)) for i in range(count)])

    def step(self):
        f, g, h = self.f, self.g, self.h
        F, G, H = self._stream(f, 9), self._stream(g, 5), self._stream(h, 5)
        if not self.node:
            edge = ((slice(None), 0), (slice(None), -1), (0, slice(None)), (-1, slice(None)))
            into = (lambda i: EX[i] > 0, lambda i: EX[i] < 0, lambda i: EY[i] > 0, lambda i: EY[i] < 0)
            wall = {"hot": 0.5 * self.varpi, "cold": 0.0}
            for s, kind in enumerate(self.sides):
                for i in range(1, 9):
                    if into[s](i):
                        F[i][edge[s]] = f[OPP[i]][edge[s]]
                        if i < 5:
                            for Q, q in ((G, g), (H, h)):
                                v = q[OPP[i]][edge[s]]
                                Q[i][edge[s]] = v if kind == "adiabatic" else wall[kind] - v
        else:
            self._extrapolate(F, G, H)
        self.f, self.g, self.h = F, G, H
        self._collide()

    def _perimeter(self, dev):
        """Index lists of the boundary nodes and of the two nodes inward of each; the scalar rule."""
        nx, ny = self.nx, self.ny
        pts = [(x, y) for y in range(ny) for x in ((range(nx) if y in (0, ny - 1) else (0, nx - 1)))]
        rows = []
        for x, y in pts:
            dx, dy = (x == 0) - (x == nx - 1), (y == 0) - (y == ny - 1)
            kx = (0 if x == 0 else 1) if dx else None
            ky = (2 if y == 0 else 3) if dy else None
            side = None
            for want in (("nee_hot", "nee_cold"), ("nee_robin",)):
                for k in (kx, ky):
                    if side is None and k is not None and self.sides[k] in want:
                        side = k
            fixed = side is not None and self.sides[side] != "nee_robin"
            value = 1.0 if fixed and self.sides[side] == "nee_hot" else 0.0
            bT, bC = self.beta[side] if side is not None and not fixed else (0.0, 0.0)
            rows.append((y * nx + x, (y + dy) * nx + x + dx, (y + 2 * dy) * nx + x + 2 * dx, float(fixed), value, bT, bC))
        r = np.array(rows)
        self.at, self.one_in, self.two_in = (torch.as_tensor(r[:, k].astype(np.int64), device=dev) for k in range(3))
        self.fixed, self.value, self.bT, self.bC = (torch.as_tensor(r[:, k], device=dev) for k in range(3, 7))

    def _extrapolate(self, F, G, H):
        """Eqs. (33)-(37), (39) on the just streamed populations: the perimeter from the nodes inward."""
        take = lambda q, at: q.reshape(q.shape[0], -1)[:, at]  # noqa: E731
        flat = lambda q, at: q.reshape(-1)[at]  # noqa: E731
        ff, gf, hf = (take(q, self.one_in) for q in (F, G, H))
        g2, h2 = (take(q, self.two_in) for q in (G, H))
        phif, phib = flat(self.phi, self.one_in), flat(self.phi, self.at)
        Tf, Cf, _, ux, uy = self._macro(ff, gf, hf, phif, flat(self.a, self.one_in), flat(self.b, self.one_in))
        T2, C2 = g2.sum(0), h2.sum(0) / flat(self.phi, self.two_in)
        Tb = torch.where(self.fixed > 0, self.value, (4 * Tf - T2) / (3 + 2 * self.bT))   # ambient T = C = 0
        Cb = torch.where(self.fixed > 0, self.value, (4 * Cf - C2) / (3 + 2 * self.bC))
        z, rho = torch.zeros_like(ux), ff.sum(0)
        F.reshape(9, -1)[:, self.at] = self._feq(rho, z, z, phib) + ff - self._feq(rho, ux, uy, phif)
        G.reshape(5, -1)[:, self.at] = self._seq(Tb, z, z, 1.0) + gf - self._seq(Tf, ux, uy, 1.0)
        H.reshape(5, -1)[:, self.at] = self._seq(Cb, z, z, phib) + hf - self._seq(Cf, ux, uy, phif)

    def fields(self):
        return {"rho": self.f.sum(0), "ux": self.ux, "uy": self.uy, "T": self.T, "C": self.C}

    def wall_numbers(self, q):
        """Mean wall gradient of Eq. (38) at each side, 0 at a zero-flux side."""
        out = []
        lines = ([q[:, k] for k in (0, 1, 2)], [q[:, -1 - k] for k in (0, 1, 2)], [q[k] for k in (0, 1, 2)], [q[-1 - k] for k in (0, 1, 2)])
        for kind, (a, b, c) in zip(self.sides, lines):
            if "adiabatic" in kind:
                out.append(0.0)
                continue
            if self.node:
                d = (-3 * a + 4 * b - c) / 2
                mean = (d.sum() - 0.5 * (d[0] + d[-1])) / (d.numel() - 1)
            else:
                mean = ((-8 * (1.0 if kind == "hot" else 0.0) + 9 * a - b) / 3).mean()
            out.append((-1.0 if "hot" in kind else 1.0) * self.L * float(mean))
        return out


def exact(case, seed):
    """The same stretch from the equations in FP64 (fields and wall numbers after one pass);
    None where that takes long: batches, large lattices and long runs."""
    if case["kind"] != "one":
        return None
    # about 120 small tensor operations a step, or the bytes of some 500 FP64 planes
    seconds = case["steps"] * max(2.2e-3, case["nx"] * case["ny"] * 4000 / 3e12)
    if seconds > 15:
        return None
    p, phi, T, C = _single(case, seed)
    s = _Plain(p, phi, T, C)
    for _ in range(case["steps"]):
        s.step()
    return {"fields": {k: v.cpu().numpy() for k, v in s.fields().items()},
            "Nu": s.wall_numbers(s.T), "Sh": s.wall_numbers(s.C)}
