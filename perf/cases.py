"""Performance cases of the solver: what a simulation program has it do, through the public
classes of ``paper_2108_06476_amd.dgx``.

``listed()`` holds the named cases, ``draw(rng)`` gives further ones of the same ranges,
``prepare``/``run`` make and pass one through the library, ``work`` counts what a pass cannot
do without, and ``exact`` computes the same results with plain float64 torch operations.

A case is a dict with
  kind      "euler" (Cartesian, 2D or 3D), "curved" (the warped box with the manufactured
            solution's source), "mhd" (Alfven wave) or "batch" (an ensemble of runs)
  op        "step": advance the state in place by nsteps Runge-Kutta steps, CFL time step;
            "rhs": one right-hand side
and the solver's configuration.
"""
import math

import numpy as np
import torch

from paper_2108_06476_amd import dgx, inputs

CFL = 0.5


def listed():
    return [
        # the smallest meshes, where a step is a chain of short launches: the 2D density wave
        # and the 4^3 warped mesh of the paper's own timing study
        dict(name="wave2d_16", kind="euler", op="step", nsteps=10, dim=2, polydeg=3, kx=16, ky=16,
             kz=1, init="wave", volume="ec", surface="llf", precision="fp64"),
        dict(name="curved_4", kind="curved", op="step", nsteps=10, polydeg=3, k=4),
        # the headline workload: Taylor-Green vortex on 32^3 elements, time stepping, and the
        # right-hand side alone as an outside integrator calls it
        dict(name="tgv_32", kind="euler", op="step", nsteps=4, dim=3, polydeg=3, kx=32, ky=32,
             kz=32, init="tgv", volume="ec", surface="llf", precision="fp64"),
        dict(name="tgv_32_rhs", kind="euler", op="rhs", nsteps=0, dim=3, polydeg=3, kx=32, ky=32,
             kz=32, init="tgv", volume="ec", surface="llf", precision="fp64"),
        # the largest: beyond the last-level cache, float32 volume fluxes
        dict(name="tgv_64_mixed", kind="euler", op="step", nsteps=2, dim=3, polydeg=3, kx=64, ky=64,
             kz=64, init="tgv", volume="ec", surface="llf", precision="mixed"),
        # high degree, and an odd-sized box of another degree with the other interface flux
        dict(name="tgv_n7_24", kind="euler", op="step", nsteps=2, dim=3, polydeg=7, kx=24, ky=24,
             kz=24, init="tgv", volume="ec", surface="llf", precision="fp64"),
        dict(name="tgv_n5_ragged", kind="euler", op="step", nsteps=2, dim=3, polydeg=5, kx=19,
             ky=23, kz=13, init="tgv", volume="ec", surface="hll", precision="fp64"),
        # the blast wave with shock capturing
        dict(name="sedov_32", kind="euler", op="step", nsteps=4, dim=3, polydeg=3, kx=32, ky=32,
             kz=32, init="sedov", volume="shockcap_hg", surface="llf", precision="fp64"),
        # many independent runs of different sizes and degrees advanced together
        dict(name="ensemble_32", kind="batch", op="step", nsteps=2, nruns=32, draw=2109),
        # the warped mesh and ideal MHD (weak form; entropy-conservative) at production size
        dict(name="curved_32", kind="curved", op="step", nsteps=2, polydeg=3, k=32),
        dict(name="alfven_32", kind="mhd", op="step", nsteps=4, polydeg=3, k=32, volume="weak",
             surface="hll"),
        dict(name="alfven_ec_20", kind="mhd", op="step", nsteps=4, polydeg=3, k=20, volume="ec",
             surface="ec"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["euler", "euler", "euler", "euler2d", "curved", "mhd", "batch"])
    op = "step" if rng.random() < 0.8 else "rhs"
    nsteps = rng.randint(2, 6) if op == "step" else 0
    if kind == "batch":
        return dict(kind="batch", op="step", nsteps=2, nruns=_logint(rng, 4, 24),
                    draw=rng.randrange(1 << 20))
    if kind == "euler2d":
        n = rng.choice([1, 2, 3, 3, 4, 5, 6, 7])
        return dict(kind="euler", op=op, nsteps=nsteps, dim=2, polydeg=n, kx=_logint(rng, 8, 200),
                    ky=_logint(rng, 8, 200), kz=1, init="wave",
                    volume=rng.choice(["ec", "ec", "weak"]), surface=rng.choice(["llf", "hll"]),
                    precision="fp64")
    if kind == "euler":
        n = rng.choice([1, 2, 3, 3, 3, 4, 5, 6, 7])
        nodes = math.exp(rng.uniform(math.log(2e4), math.log(8e6)))
        k = max(4.0, (nodes / (n + 1) ** 3) ** (1.0 / 3.0))
        kx, ky, kz = (max(3, int(round(k * rng.uniform(0.75, 1.3)))) for _ in range(3))
        how = rng.choice(["ec", "ec", "ec", "weak", "shockcap_hg", "mixed"])
        return dict(kind="euler", op=op, nsteps=nsteps, dim=3, polydeg=n, kx=kx, ky=ky, kz=kz,
                    init="sedov" if how == "shockcap_hg" else "tgv",
                    volume="ec" if how == "mixed" else how, surface=rng.choice(["llf", "llf", "hll"]),
                    precision="mixed" if how == "mixed" else "fp64")
    n = rng.choice([2, 3, 3, 3, 4, 5, 6, 7])
    nodes = math.exp(rng.uniform(math.log(4e3), math.log(2e6)))
    k = max(4, int(round((nodes / (n + 1) ** 3) ** (1.0 / 3.0))))
    if kind == "curved":
        return dict(kind="curved", op=op, nsteps=nsteps, polydeg=n, k=k)
    volume = rng.choice(["weak", "ec"])
    return dict(kind="mhd", op=op, nsteps=nsteps, polydeg=n, k=k, volume=volume,
                surface="hll" if volume == "weak" else rng.choice(["ec", "llf"]))


# ---------------------------------------------------------------------- the library's side
def _box(case):
    half = {"tgv": math.pi, "sedov": 1.0, "wave": 2.0}[case["init"]]
    dim = case["dim"]
    return dict(dim=dim, polydeg=case["polydeg"], cells=(case["kx"], case["ky"], case["kz"]),
                xmin=(-half,) * dim, xmax=(half,) * dim, gamma=inputs.GAMMA,
                volume=case["volume"], surface=case["surface"], precision=case["precision"])


def _par(seed):
    """Parameters of the initial state, from the seed: times, Mach numbers, energies."""
    rng = np.random.default_rng(seed)
    return dict(t=float(rng.uniform(0.0, 1.0)), mach=float(rng.uniform(0.09, 0.11)),
                E0=float(rng.uniform(0.9, 1.1)), seed=int(seed))


def _state(case, xyz, seed):
    """The initial state at node positions xyz (a torch tensor) and its time."""
    p = _par(seed)
    if case["kind"] == "curved":
        return inputs.mms(xyz, t=p["t"]), p["t"]
    if case["kind"] == "mhd":
        return inputs.alfven(xyz, t=p["t"]), p["t"]
    if case["init"] == "wave":   # the density wave at a time of its own
        rho = 2.0 + 0.1 * torch.sin(math.pi * (xyz[0] + xyz[1] - 2.0 * p["t"]))
        return inputs.prim_to_cons(rho, [1.0, 1.0], 10.0), 0.0
    if case["init"] == "sedov":
        r2 = xyz[0] ** 2 + xyz[1] ** 2 + xyz[2] ** 2
        sg = 0.25
        pr = 1.0e-5 + 0.4 * p["E0"] * torch.exp(-r2 / (2 * sg ** 2)) / ((2 * math.pi) ** 1.5 * sg ** 3)
        return inputs.prim_to_cons(torch.ones_like(r2), [0.0, 0.0, 0.0], pr), 0.0
    return inputs.tgv(xyz, mach=p["mach"], perturb_seed=p["seed"]), 0.0


def _runs(case, seed):
    """The ensemble's runs: sizes and degrees by the case, Mach numbers and shifts by the seed."""
    runs = inputs.ensemble(case["nruns"], seed=case["draw"])
    for r, other in zip(runs, inputs.ensemble(case["nruns"], seed=seed)):
        r["mach"], r["shift"] = other["mach"], other["shift"]
    return runs


def prepare(case, seed):
    if case["kind"] == "batch":
        runs = _runs(case, seed)
        configs = [inputs.ensemble_config(r) for r in runs]
        solver = dgx.Batch(configs)
        xyz, us = {}, []
        for r, c in zip(runs, configs):
            key = (r["K"], r["N"])
            if key not in xyz:
                xyz[key] = dgx.Solver(**c).node_coords()
            us.append(inputs.ensemble_state(r, xyz[key]).contiguous())
        t = torch.zeros(case["nruns"], dtype=torch.float64, device="cuda")
        return dict(case=case, solver=solver, u=us, t=t)
    if case["kind"] == "curved":
        solver = dgx.CurvSolver(case["polydeg"], case["k"])
    elif case["kind"] == "mhd":
        solver = dgx.MhdSolver(case["polydeg"], case["k"], surface=case["surface"],
                               volume=case["volume"])
    else:
        solver = dgx.Solver(**_box(case))
    u, time = _state(case, solver.node_coords(), seed)
    u = u.contiguous()
    t = torch.full((1,), time, dtype=torch.float64, device="cuda")
    du = torch.empty_like(u) if case["op"] == "rhs" else None
    u0 = u.clone() if case["kind"] == "mhd" and case["op"] == "step" else None
    return dict(case=case, solver=solver, u=u, t=t, du=du, time=time, u0=u0)


def run(state):
    case, solver, u = state["case"], state["solver"], state["u"]
    if case["op"] == "rhs":
        return solver.rhs(u, state["du"], t=state["time"])
    if state.get("u0") is not None:
        # without divergence control the Alfven wave does not stay smooth for thousands of
        # steps: a pass starts from the stored state, as a convergence study's does
        u.copy_(state["u0"])
    solver.step(u, case["nsteps"], cfl=CFL, t=state["t"])
    return {"u": u, "t": state["t"]}


def work(case):
    """Bytes and operations of a pass.  A Runge-Kutta stage reads and writes the state; its
    register is written by stages 1-4 and read by 2-5: 18 arrays in five stages.  A
    right-hand side reads the state and writes the result.  The warped mesh reads its metric
    terms, Jacobian and positions besides (13 values a node)."""
    if case["kind"] == "batch":
        each = [dict(kind="euler", op="step", nsteps=case["nsteps"], dim=3, polydeg=r["N"],
                     kx=r["K"], ky=r["K"], kz=r["K"], volume="ec") for r in _runs(case, 1)]
        got = [work(c) for c in each]
        return {k: sum(g[k] for g in got) for k in ("bytes", "flops")}
    dim = case.get("dim", 3)
    n = case["polydeg"] + 1
    cells = case["k"] ** 3 if "k" in case else case["kx"] * case["ky"] * case["kz"]
    nodes = cells * n ** dim
    nv = 8 if case["kind"] == "mhd" else dim + 2
    stages = 5 * case["nsteps"] if case["op"] == "step" else 1
    arrays = 3.6 if case["op"] == "step" else 2.0
    per_node = 8 * nv * arrays + (8 * 13 if case["kind"] == "curved" else 0)
    pairs = 0.5 * dim * case["polydeg"]          # two-point fluxes per node
    faces = 2.0 * dim / n                        # face fluxes per node (each side its own)
    if case.get("volume") == "weak":
        flops = dim * (2 * nv * n + 4 * nv) + faces * 8 * nv
    else:
        flops = pairs * (60 + 4 * nv) + faces * 8 * nv
    return {"bytes": float(nodes) * per_node * stages,
            "flops": float(nodes) * (flops + 30 + 4 * nv) * stages}


# --------------------------------------------------- the same results in plain float64 torch
def _legendre(N, x):
    """P_0..P_N at x."""
    P = [np.ones_like(x), x]
    for m in range(1, N):
        P.append(((2 * m + 1) * x * P[m] - m * P[m - 1]) / (m + 1))
    return P


def _lgl(N):
    """Legendre-Gauss-Lobatto nodes, weights, differentiation matrix and the inverse
    Vandermonde matrix of the orthonormal Legendre polynomials, formed in extended precision."""
    x = -np.cos(np.pi * np.arange(N + 1, dtype=np.longdouble) / N)
    for _ in range(60):   # Newton on (1 - x^2) P_N'(x), whose derivative is -N (N + 1) P_N
        P = _legendre(N, x)
        x = x - (x * P[N] - P[N - 1]) / ((N + 1) * P[N])
    x = 0.5 * (x - x[::-1])
    P = _legendre(N, x)
    w = 2 / (N * (N + 1) * P[N] ** 2)
    dx = x[:, None] - x[None, :] + np.eye(N + 1, dtype=np.longdouble)
    D = P[N][:, None] / P[N][None, :] / dx
    D[np.diag_indices(N + 1)] = 0
    D[np.diag_indices(N + 1)] = -D.sum(axis=1)
    V = np.array([P[m] * np.sqrt(np.longdouble(m) + 0.5) for m in range(N + 1)]).T
    f = np.array([1 / np.sum(w * V[:, m] ** 2) for m in range(N + 1)])   # discrete norms
    Vinv = (V * w[:, None] * f[None, :]).T
    return tuple(a.astype(np.float64) for a in (x, w, D, Vinv))


def _ln_mean(a, b):
    z = (b - a) / (b + a)
    z2 = z * z
    q = torch.where(z2 < 1e-3, 1 + z2 * (1 / 3 + z2 * (1 / 5 + z2 * (1 / 7 + z2 * (1 / 9 + z2 / 11)))),
                    torch.atanh(z) / torch.where(z2 < 1e-3, torch.ones_like(z), z))
    return 0.5 * (a + b) / q


class _Exact:
    """The semidiscretisation in float64 torch operations.  States are viewed as
    [variable][z cell][y cell][x cell][k][j][i]; direction d has node axis -1-d and cell
    axis -4-d."""

    def __init__(self, kind, dim, polydeg, cells, lo, hi, gamma, volume, surface, device):
        self.kind, self.dim, self.N, self.n = kind, dim, polydeg, polydeg + 1
        self.cells, self.gamma, self.volume, self.surface = cells, gamma, volume, surface
        self.dev = device
        x, w, D, self.Vinv = _lgl(polydeg)
        self.x, self.w, self.D = x, w, D
        self.h = [(hi[d] - lo[d]) / cells[d] for d in range(dim)]
        B = np.zeros((self.n, self.n))
        B[0, 0], B[-1, -1] = -1.0, 1.0
        self.S = 2 * D - B / w[:, None]
        self.nv = 8 if kind == "mhd" else dim + 2
        nn = [self.n] * dim + [1] * (3 - dim)
        self.full = (cells[2], cells[1], cells[0], nn[2], nn[1], nn[0])
        pos = []
        for d in range(dim):
            e = torch.arange(cells[d], dtype=torch.float64, device=device)
            xt = torch.tensor(x, dtype=torch.float64, device=device)
            shape = [1] * 6
            shape[2 - d], shape[5 - d] = cells[d], self.n
            p = lo[d] + self.h[d] * (e[:, None] + 0.5 * (1.0 + xt[None, :]))
            pos.append(p.reshape(shape).expand(self.full))
        self.xyz = torch.stack(pos)
        if kind == "curved":
            self._warp()

    def _along(self, M, f, d):
        """M applied along node direction d."""
        M = torch.as_tensor(M, dtype=torch.float64, device=self.dev)
        return torch.tensordot(f, M, dims=([f.dim() - 1 - d], [1])).movedim(-1, f.dim() - 1 - d)

    def _warp(self):
        xi, eta, ze = self.xyz
        pi, a = math.pi, 0.15
        y = eta + a * torch.cos(1.5 * pi * xi) * torch.cos(0.5 * pi * eta) * torch.cos(0.5 * pi * ze)
        x = xi + a * torch.cos(0.5 * pi * xi) * torch.cos(2 * pi * y) * torch.cos(0.5 * pi * ze)
        z = ze + a * torch.cos(0.5 * pi * x) * torch.cos(pi * y) * torch.cos(0.5 * pi * ze)
        X = torch.stack([x, y, z])
        self.xyz = X
        dX = torch.stack([self._along(self.D, X, j) for j in range(3)])     # [j][component]
        cr = torch.cross(dX[1], dX[2], dim=0)
        self.J = (dX[0] * cr).sum(0)
        self.Ja = torch.empty((3, 3) + self.full, dtype=torch.float64, device=self.dev)
        for c in range(3):
            m, l = (c + 1) % 3, (c + 2) % 3
            V = [X[l] * dX[j, m] for j in range(3)]
            for i in range(3):
                j, k = (i + 1) % 3, (i + 2) % 3
                self.Ja[i, c] = -(self._along(self.D, V[k], j) - self._along(self.D, V[j], k))

    def prim(self, u):
        rho = u[0]
        nvel = 3 if self.kind == "mhd" else self.dim
        v = u[1:1 + nvel] / rho
        p = u[1 + nvel] - 0.5 * rho * (v * v).sum(0)
        q = dict(u=u, rho=rho, v=v)
        if self.kind == "mhd":
            q["B"] = u[5:8]
            p = p - 0.5 * (q["B"] ** 2).sum(0)
        q["p"] = (self.gamma - 1) * p
        return q

    @staticmethod
    def at(q, idx, axis):
        """The node data at index idx of an axis (a list of indices keeps the axis)."""
        return {k: a.select(axis, idx) for k, a in q.items()}

    def speed(self, q, d, a=None):
        """(normal velocity, sound speed) along d, or through the vector a."""
        c2 = self.gamma * q["p"] / q["rho"]
        if self.kind == "mhd":
            b2 = (q["B"] ** 2).sum(0) / q["rho"]
            s = c2 + b2
            disc = (s * s - 4 * c2 * q["B"][d] ** 2 / q["rho"]).clamp_min(0.0)
            return q["v"][d], torch.sqrt(0.5 * (s + torch.sqrt(disc)))
        if a is not None:
            return (q["v"] * a).sum(0), torch.sqrt(c2 * (a * a).sum(0))
        return q["v"][d], torch.sqrt(c2)

    def flux(self, q, d, a=None):
        u, v, p = q["u"], q["v"], q["p"]
        if self.kind == "mhd":
            B = q["B"]
            pt, vB = p + 0.5 * (B * B).sum(0), (v * B).sum(0)
            m = u[1 + d] * v - B[d] * B
            m[d] += pt
            return torch.cat([u[1 + d][None], m, (v[d] * (u[4] + pt) - B[d] * vB)[None], v[d] * B - B[d] * v])
        if a is not None:
            va = (v * a).sum(0)
            return torch.cat([(u[0] * va)[None], u[1:4] * va + p * a, (va * (u[4] + p))[None]])
        m = u[1 + d] * v
        m[d] += p
        return torch.cat([u[1 + d][None], m, (v[d] * (u[-1] + p))[None]])

    def ec(self, L, R, d, a=None):
        """The entropy-conservative two-point flux."""
        g1 = self.gamma - 1
        rl = _ln_mean(L["rho"], R["rho"])
        bl = _ln_mean(L["rho"] / L["p"], R["rho"] / R["p"])
        va = 0.5 * (L["v"] + R["v"])
        if self.kind == "mhd":
            Ba = 0.5 * (L["B"] + R["B"])
            betaL, betaR = 0.5 * L["rho"] / L["p"], 0.5 * R["rho"] / R["p"]
            ba = 0.5 * (betaL + betaR)
            B2 = 0.5 * ((L["B"] ** 2).sum(0) + (R["B"] ** 2).sum(0))
            v2 = 0.5 * ((L["v"] ** 2).sum(0) + (R["v"] ** 2).sum(0))
            vB = 0.5 * ((L["v"] * L["B"]).sum(0) + (R["v"] * R["B"]).sum(0))
            bv = 0.5 * (betaL * L["v"][d] + betaR * R["v"][d])
            fr = rl * va[d]
            m = fr * va - Ba[d] * Ba
            m[d] += 0.25 * (L["rho"] + R["rho"]) / ba + 0.5 * B2
            fB = bv / ba * Ba - Ba[d] * va
            e = fr * (1 / (g1 * bl) - 0.5 * v2) + (va * m).sum(0) + (Ba * fB).sum(0) \
                + Ba[d] * vB - 0.5 * B2 * va[d]
            return torch.cat([fr[None], m, e[None], fB])
        an = (lambda w: w[d]) if a is None else (lambda w: (w * a).sum(0))
        fr = rl * an(va)
        m = fr * va
        pa = 0.5 * (L["p"] + R["p"])
        if a is None:
            m[d] += pa
        else:
            m = m + pa * a
        e = fr * (1 / (g1 * bl) + 0.5 * (L["v"] * R["v"]).sum(0)) \
            + 0.5 * (L["p"] * an(R["v"]) + R["p"] * an(L["v"]))
        return torch.cat([fr[None], m, e[None]])

    def face(self, L, R, d, a=None, how=None):
        how = how or self.surface
        if how == "ec":
            return self.ec(L, R, d, a)
        fL, fR = self.flux(L, d, a), self.flux(R, d, a)
        vL, cL = self.speed(L, d, a)
        vR, cR = self.speed(R, d, a)
        if how == "llf":
            lam = torch.maximum(vL.abs() + cL, vR.abs() + cR)
            return 0.5 * (fL + fR) - 0.5 * lam * (R["u"] - L["u"])
        sL, sR = torch.minimum(vL - cL, vR - cR), torch.maximum(vL + cL, vR + cR)
        mid = (sR * fL - sL * fR + sL * sR * (R["u"] - L["u"])) / (sR - sL)
        return torch.where(sL >= 0, fL, torch.where(sR <= 0, fR, mid))

    def phi(self, q):
        """Powell's factor (0, B, v.B, v)."""
        z = torch.zeros_like(q["rho"])
        return torch.cat([z[None], q["B"], (q["v"] * q["B"]).sum(0)[None], q["v"]])

    def alpha(self, q):
        """Blending factor per cell, [z][y][x]."""
        f = q["rho"] * q["p"]
        for d in range(self.dim):
            f = self._along(self.Vinv, f, d)
        f = f * f
        n = self.n
        cut = [(slice(None),) * 3 + (slice(0, m) if self.dim == 3 else slice(None), slice(0, m), slice(0, m))
               for m in (n, n - 1, n - 2)]
        t0, t1, t2 = (f[c].sum(dim=(3, 4, 5)) if m > 0 else torch.zeros(self.full[:3], dtype=f.dtype, device=f.device)
                      for c, m in zip(cut, (n, n - 1, n - 2)))
        one = torch.ones_like(t0)
        r1 = torch.where(t0 != 0, (t0 - t1) / torch.where(t0 != 0, t0, one), 0 * one)
        r2 = torch.where(t1 != 0, (t1 - t2) / torch.where(t1 != 0, t1, one), 0 * one)
        thr = 0.5 * 10 ** (-1.8 * n ** 0.25)
        sharp = math.log((1 - 1e-4) / 1e-4) / thr
        al = torch.sigmoid(sharp * (torch.maximum(r1, r2) - thr))
        al = torch.where(al < 1e-3, 0 * al, torch.where(al > 1 - 1e-3, one, al)).clamp_max(0.5)
        out = al
        for ax in range(3 - self.dim, 3):
            for s in (1, -1):
                out = torch.maximum(out, 0.5 * torch.roll(al, s, ax))
        return out

    def rhs(self, u, t=0.0):
        q = self.prim(u)
        R = torch.zeros_like(u)
        V = torch.zeros_like(u)
        F = torch.zeros_like(u)
        n, N = self.n, self.N
        shock = self.volume == "shockcap_hg"
        for d in range(self.dim):
            scale = 1.0 if self.kind == "curved" else 2.0 / self.h[d]
            ax, cell = -1 - d, -4 - d
            a = self.Ja[d] if self.kind == "curved" else None
            nodes = [self.at(q, i, ax) for i in range(n)]
            met = [a.select(ax, i) if a is not None else None for i in range(n)]
            if self.volume == "weak":
                V += scale * self._along(self.D.T * self.w[None, :] / self.w[:, None], self.flux(q, d), d)
            else:
                Vd = [V.select(ax, i) for i in range(n)]
                for i in range(n):
                    for m in range(i + 1, n):
                        f = self.ec(nodes[i], nodes[m], d, None if a is None else 0.5 * (met[i] + met[m]))
                        Vd[i] -= scale * self.S[i, m] * f
                        Vd[m] -= scale * self.S[m, i] * f
                if self.kind == "mhd":   # Powell's term: phi_i sum_m S_im {{B_d}}
                    Bd, ph = q["B"][d], self.phi(q)
                    off = self.S - np.diag(np.diag(self.S))
                    row = torch.as_tensor(off.sum(1), dtype=u.dtype, device=u.device)
                    shape = [1] * Bd.dim()
                    shape[ax] = n
                    V -= scale * ph * 0.5 * (self._along(off, Bd, d) + row.reshape(shape) * Bd)
            if shock:
                for i in range(N):
                    f = self.face(nodes[i], nodes[i + 1], d, how="llf")
                    F.select(ax, i).sub_(scale / self.w[i] * f)
                    F.select(ax, i + 1).add_(scale / self.w[i + 1] * f)
            # interfaces: F* of every cell's plus face from (own last, next cell's first) node
            cax = cell + 1   # the node axis is selected away
            L, nxt = nodes[N], {k: torch.roll(x, -1, cax) for k, x in nodes[0].items()}
            f = self.face(L, nxt, d, met[N])
            R.select(ax, N).sub_(scale / self.w[N] * f)
            R.select(ax, 0).add_(scale / self.w[0] * torch.roll(f, 1, cax))
            if self.kind == "mhd" and self.volume == "ec":
                Bm = 0.5 * (L["B"][d] + nxt["B"][d])
                R.select(ax, N).sub_(scale / self.w[N] * self.phi(L) * Bm)
                R.select(ax, 0).add_(scale / self.w[0] * self.phi(nodes[0]) * torch.roll(Bm, 1, cax))
        if shock:
            al = self.alpha(q)[..., None, None, None]
            V = (1 - al) * V + al * F
        R += V
        if self.kind == "curved":
            R = R / self.J
            th = math.pi * self.xyz.sum(0) - 2 * math.pi * t
            rho, hc = 2 + 0.1 * torch.sin(th), 0.1 * torch.cos(th)
            k, om, g1 = math.pi, 2 * math.pi, self.gamma - 1
            dp = g1 * (2 * rho - 1.5) * k * hc
            s0 = (3 * k - om) * hc
            R += torch.stack([s0, s0 + dp, s0 + dp, s0 + dp,
                              -2 * rho * om * hc + 3 * k * (2 * rho + g1 * (2 * rho - 1.5)) * hc])
        return R

    def dt(self, u):
        q = self.prim(u)
        lam = 0.0
        for d in range(self.dim):
            if self.kind == "curved":
                v, c = self.speed(q, d, self.Ja[d])
                lam = lam + ((v.abs() + c) / self.J).amax(dim=(3, 4, 5))
            else:
                v, c = self.speed(q, d)
                lam = lam + (2.0 / self.h[d]) * (v.abs() + c).amax(dim=(3, 4, 5))
        return CFL * 2.0 / (self.n * float(lam.max()))

    A = (0.0, -567301805773 / 1357537059087, -2404267990393 / 2016746695238,
         -3550918686646 / 2091501179385, -1275806237668 / 842570457699)
    B = (1432997174477 / 9575080441755, 5161836677717 / 13612068292357,
         1720146321549 / 2090206949498, 3134564353537 / 4481467310338,
         2277821191437 / 14882151754819)
    C = (0.0, 1432997174477 / 9575080441755, 2526269341429 / 6820363183890,
         2006345519317 / 3224310063776, 2802321613138 / 2924317926251)

    def step(self, u, nsteps, t):
        u = u.clone()
        for _ in range(nsteps):
            dt = self.dt(u)
            k = torch.zeros_like(u)
            for A, B, c in zip(self.A, self.B, self.C):
                k = A * k + dt * self.rhs(u, t + c * dt)
                u = u + B * k
            t += dt
        return u, t


def _exact_of(case, device):
    if case["kind"] == "euler":
        b = _box(case)
        pad = (3 - case["dim"]) * (0.0,)
        return _Exact("euler", case["dim"], case["polydeg"], b["cells"], b["xmin"] + pad, b["xmax"] + pad,
                      inputs.GAMMA, case["volume"], case["surface"], device)
    k = (case["k"],) * 3
    lo, hi = (-1.0,) * 3, (1.0,) * 3
    if case["kind"] == "curved":
        return _Exact("curved", 3, case["polydeg"], k, lo, hi, inputs.GAMMA, "ec", "llf", device)
    return _Exact("mhd", 3, case["polydeg"], k, lo, hi, 5.0 / 3.0, case["volume"], case["surface"], device)


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] == "batch":
        us, ts = [], []
        for r in _runs(case, seed):
            c = inputs.ensemble_config(r)
            ex = _Exact("euler", 3, r["N"], c["cells"], c["xmin"], c["xmax"], inputs.GAMMA, "ec", "llf", device)
            u0 = inputs.ensemble_state(r, ex.xyz)
            u, t = ex.step(u0, case["nsteps"], 0.0)
            us.append(u.reshape(5, r["K"] ** 3, -1))
            ts.append(t)
        return {"u": us, "t": torch.tensor(ts, dtype=torch.float64, device=device)}
    ex = _exact_of(case, device)
    u0, t0 = _state(case, ex.xyz, seed)
    cells = ex.full[0] * ex.full[1] * ex.full[2]
    if case["op"] == "rhs":
        return ex.rhs(u0, t0).reshape(ex.nv, cells, -1)
    u, t = ex.step(u0, case["nsteps"], t0)
    return {"u": u.reshape(ex.nv, cells, -1), "t": torch.tensor([t], dtype=torch.float64, device=device)}
