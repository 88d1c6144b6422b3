"""What a user of the solver has it do, as measurable cases.

Every case goes through the public classes of `paper_2512_09904_amd.sph`
(`Solver`, `Pool`) the way a program does: particles are handed over once
(`prepare`), and one pass advances the solve, reads the reports and the
fields, or serves a batch of requests, relaxes a body, or reads the contact
factor.  `exact` repeats a pass in plain torch, FP64, from the equations.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2512_09904_amd import cases as geo
from paper_2512_09904_amd import sph


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a monitored small solve: a few steps, then its reports and fields;
        # launch latency and the read-back decide
        dict(name="tank 12k", path="step", shape="tank", dp=2e-3, omega=150.0, precision="mixed", steps=4),
        # the smallest request of the parameter sweep, a stretch of its steps
        # between two outputs
        dict(name="sweep 50k", path="step", shape="serving", n=50_000, omega=300.0, immersion=0.04, nu=1e-4,
             precision="mixed", steps=40),
        # the benchmark's gearbox proxy at 1.5 mm, from hand-over to fields (it
        # is usable for its first few hundred steps, so a pass starts it anew)
        dict(name="gearbox 1.5mm", path="pool", shape="gearbox", dp=1.5e-3, omega=300.0, immersion=0.03, nu=1e-4, count=1,
             precision="mixed", steps=80),
        # the largest request of the sweep
        dict(name="sweep 2M", path="step", shape="serving", n=2_000_000, omega=300.0, immersion=0.05, nu=1e-4,
             precision="mixed", steps=16),
        # the precision study's tank in its two other arithmetics
        dict(name="tank 196k fp64", path="step", shape="tank", dp=0.788e-3, omega=450.0, precision="fp64", steps=16),
        dict(name="tank 196k fp32", path="step", shape="tank", dp=0.788e-3, omega=450.0, precision="fp32", steps=24),
        # dissipation heating and two oils: the options of the heat equation
        dict(name="sweep 300k heated", path="step", shape="serving", n=300_000, omega=450.0, immersion=0.03, nu=2e-4,
             precision="mixed", steps=24, viscous_heating=1, materials=2),
        # a batch of sweep requests from admission to release
        dict(name="pool of 4", path="pool", shape="serving", n=60_000, count=4, omega=250.0, immersion=0.04, nu=1e-4,
             precision="mixed", steps=60),
        # wetting of the gears and the housing, read between steps
        dict(name="contact 1.5mm", path="contact", shape="gearbox", dp=1.5e-3, omega=300.0, immersion=0.03, nu=1e-4,
             precision="mixed"),
        # particle generation inside a body: the gear of the proxy, and a small ball
        dict(name="relax gear 177k", path="relax", kind="gear", dp=1.5e-3, size=0.084, precision="mixed", iterations=10),
        dict(name="relax ball 14k", path="relax", kind="sphere", dp=2e-3, size=0.030, precision="fp64", iterations=4),
    ]


def draw(rng):
    def log(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    path = rng.choice(["step"] * 6 + ["pool", "contact", "relax"])
    prec = rng.choice(["mixed", "mixed", "mixed", "fp64", "fp32"])
    if path == "relax":
        kind = rng.choice(["sphere", "box", "cylinder", "gear"])
        n = log(8e3, 1.7e5)
        size = 0.084 if kind == "gear" else rng.uniform(0.02, 0.06)
        # volumes of the bodies made by relax_shape
        vol = {"sphere": 4.19 * size ** 3, "box": 3.84 * size ** 3, "cylinder": 3.77 * size ** 3, "gear": 6.0e-4}[kind]
        return dict(path="relax", kind=kind, dp=(vol / n) ** (1 / 3), size=size,
                    precision="fp64" if prec == "fp64" else "mixed", iterations=rng.randint(2, 8))
    c = dict(path=path, precision=prec, omega=rng.uniform(150.0, 600.0), immersion=rng.uniform(0.02, 0.06),
             nu=log(0.5e-4, 3e-4))
    if path == "pool" and rng.random() < 0.7:
        return dict(c, shape="serving", n=int(log(5e4, 1.5e5)), count=rng.randint(2, 5), steps=rng.randint(20, 60))
    shape = "gearbox" if path == "pool" else rng.choice(["tank", "serving", "serving", "gearbox"][: 3 + (path == "contact")])
    if shape == "tank":
        c.update(shape=shape, dp=log(0.7e-3, 2.4e-3))
        n = 12240 * (2e-3 / c["dp"]) ** 3
    elif shape == "gearbox":
        c.update(shape=shape, dp=log(1.5e-3, 4e-3), omega=rng.uniform(150.0, 300.0), immersion=rng.uniform(0.03, 0.05))
    else:
        n = int(log(5e4, 1.4e6 if prec == "mixed" else 5e5))
        c.update(shape=shape, n=n)
    if path == "contact":
        return c
    if path == "pool":
        return dict(c, count=1, steps=rng.randint(20, 80))
    c["steps"] = max(2, min(rng.randint(4, 40), int(1.6e7 / n)))
    if shape == "serving":
        c["h_over_dp"] = rng.choice([1.3, 1.3, 1.3, 1.0])
        if rng.random() < 0.3:
            c["viscous_heating"] = 1
        if rng.random() < 0.3:
            c["materials"] = 2
        if rng.random() < 0.15:
            c["wall_visc"] = 1
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=4)
def _geometry(shape, dp, n, omega, immersion, nu):
    if shape == "tank":
        return geo.tank_c1(seed=0, dp=dp, omega=omega)
    if shape == "gearbox":
        return geo.gearbox(seed=0, dp=dp, omega_big=omega, immersion=immersion, nu=nu)
    return geo.serving_tank(n, omega, immersion, nu, seed=0)


def _solve(case, seed):
    """A started tank or gearbox: the lattice with a seeded jitter, a slow swirl
    with some noise, a temperature that varies over the box."""
    base = _geometry(case["shape"], case.get("dp"), case.get("n"), case["omega"], case.get("immersion"), case.get("nu"))
    c = base.copy()
    p = c.params
    dp, umax = p["dp"], c.meta["umax"]
    c.xf = base.xf - geo.jitter(0, base.nf, dp) + geo.jitter(seed + 1, base.nf, dp)
    L = np.asarray(c.meta["box"])
    rng = np.random.default_rng(seed)
    u = (c.xf / L - 0.5) * (2.0 * math.pi)
    c.vf = (0.01 * umax) * rng.uniform(-1.0, 1.0, c.xf.shape)
    c.vf[:, 0] += 0.03 * umax * np.sin(u[:, 2]) * np.cos(u[:, 0] / 2)
    c.vf[:, 2] -= 0.03 * umax * np.cos(u[:, 2] / 2) * np.sin(u[:, 0]) * 0.5
    c.Tf = base.Tf + 4.0 * np.sin(u[:, 0] + 0.3 * (seed % 17)) * np.cos(u[:, 1]) + rng.uniform(-0.5, 0.5, c.nf)
    hod = case.get("h_over_dp", 1.3)
    if hod != 1.3:
        m = 2.0 * hod * dp + 3 * dp
        p.update(h_over_dp=hod, grid_lo=(-m,) * 3, grid_hi=tuple(float(x) + m for x in L))
    if case.get("materials"):
        p["materials"] = [(0.13, 2000.0), (0.45, 1300.0)]
        c.material = (c.xf[:, 0] > 0.5 * L[0]).astype(np.int32)
    p["viscous_heating"] = case.get("viscous_heating", 0)
    p["wall_visc"] = case.get("wall_visc", 0)
    return c


def _requests(case, seed):
    out = []
    for k in range(case["count"]):
        one = dict(shape=case["shape"], omega=case["omega"] + 40.0 * k, immersion=case["immersion"], nu=case["nu"])
        one.update({"n": int(case["n"] * (1.0 + 0.6 * k))} if case["shape"] == "serving" else {"dp": case["dp"]})
        out.append(_solve(one, seed * 16 + k))
    return out


def _shape(case):
    s = case["size"]
    size = {"sphere": (s,), "box": (s, 0.6 * s, 0.8 * s), "cylinder": (s, 0.6 * s), "gear": (s, s - 0.009, 0.015)}[case["kind"]]
    return dict(kind=case["kind"], center=(0.19, 0.075, 0.1), size=size, teeth=40, phase=0.5)


@functools.lru_cache(maxsize=4)
def _body_sites(kind, dp, size):
    shape = _shape(dict(kind=kind, size=size))
    return geo.relax_case(shape, dp, 1.1 * size, jitter_amp=0.0)


def _body(case, seed):
    base = _body_sites(case["kind"], case["dp"], case["size"])
    c = base.copy()
    shift = geo.jitter(seed + 1, c.nf, case["dp"], 0.25)
    inside = geo.shape_inside(_shape(case))(c.xf + shift)
    c.xf = np.where(inside[:, None], c.xf + shift, c.xf)
    return c


def prepare(case, seed):
    path = case["path"]
    if path == "pool":
        reqs = _requests(case, seed)
        need = sum(sph.Pool.bytes_required(c, case["precision"]) for c in reqs)
        return dict(path=path, reqs=reqs, pool=sph.Pool(need, max_slots=len(reqs), precision=case["precision"]),
                    steps=case["steps"])
    if path == "relax":
        return dict(path=path, solver=sph.Solver(_body(case, seed), precision=case["precision"]), shape=_shape(case),
                    iterations=case["iterations"])
    c = _solve(case, seed)
    return dict(path=path, solver=sph.Solver(c, precision=case["precision"]), case=c, precision=case["precision"],
                steps=case.get("steps", 0))


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
REPORT = ("t", "dt_ad", "dt", "vmax", "mass", "kinetic", "thermal", "heat_step", "heat_total", "mass_proxy", "diss_step",
          "diss_total")
COUNTS = ("step", "n_ac", "substeps")
BODY = ("force", "torque", "torque_axis", "power", "heat_rate", "torque_axis_int", "energy_int", "heat_int")


def _answer(r, f):
    out = {k: f[k] for k in ("x", "v", "rho", "T")}
    out["counts"] = [r[k] for k in COUNTS]
    out["report"] = {k: r[k] for k in REPORT}
    out["bodies"] = {k: np.array([b[k] for b in r["bodies"]]) for k in BODY}
    return out


def run(state):
    path = state["path"]
    if path == "pool":
        pool = state["pool"]
        slots = [pool.admit(c, state["steps"]) for c in state["reqs"]]
        pool.step(state["steps"])
        out = []
        for s in slots:
            done, r = pool.poll(s)
            while not done:
                done, r = pool.poll(s)
            f = pool.get_fluid(s)
            pool.release(s)
            b = np.concatenate([np.concatenate([np.ravel(x[k]) for k in BODY]) for x in r["bodies"]])
            out.append({"x": f["x"], "v": f["v"], "rho": f["rho"], "T": f["T"], "t": r["t"], "kinetic": r["kinetic"],
                        "thermal": r["thermal"], "heat_total": r["heat_total"], "bodies": b,
                        "counts": np.array([r[k] for k in COUNTS])})
        return out
    s = state["solver"]
    if path == "contact":
        zeta, mean = s.contact_factor()
        return {"zeta": zeta, "mean": mean}
    if path == "relax":
        r = s.relax(state["shape"], state["iterations"])
        return {"x": s.get_fluid()["x"], "amax_first": r["amax_first"], "amax_last": r["amax_last"],
                "dt_last": r["dt_last"], "bounded_last": r["bounded_last"]}
    s.step(state["steps"])
    try:
        r = s.reduce()
    except sph.SphError as e:
        # now and then, after hundreds of steps, a splash carries a particle
        # through the walls: the program starts that solve again
        if e.code != sph.SPH_ERR_DOMAIN:
            raise
        s.close()
        s = state["solver"] = sph.Solver(state["case"], precision=state["precision"])
        s.step(state["steps"])
        r = s.reduce()
    return _answer(r, s.get_fluid())


def _counts(case):
    """Fluid and solid particles of a case (approximate for the solids)."""
    if case["path"] == "pool" and case["shape"] == "serving":
        n = sum(int(case["n"] * (1.0 + 0.6 * k)) for k in range(case["count"]))
        return n, 1.1 * case["count"] * (n / case["count"]) ** (2 / 3) * 18
    shape = case["shape"]
    if shape == "tank":
        k = 2e-3 / case["dp"]
        return 12240 * k ** 3, 23456 * k ** 2
    if shape == "gearbox":
        k = 1.5e-3 / case["dp"]
        return 888440 * k ** 3, 478448 * k ** 2
    return case["n"], 20 * case["n"] ** (2 / 3)


def work(case):
    """One pass.  Bytes: the state a sweep needs and what it changes, each once
    per sweep (positions, velocity and density, temperature; walls once per
    step), and the fields read back.  Operations: the pair interactions of the
    sweeps of a step at two acoustic sub-steps."""
    prec = 8 if case["precision"] == "fp64" else 4
    if case["path"] == "relax":
        s = case["size"]
        vol = {"sphere": 4.19 * s ** 3, "box": 3.84 * s ** 3, "cylinder": 3.77 * s ** 3, "gear": 6.0e-4}[case["kind"]]
        n = vol / case["dp"] ** 3
        # near the surface the kernel-gradient integral takes about 2000 cells
        return {"bytes": n * (case["iterations"] * 120.0 + 24), "flops": n * case["iterations"] * (76 * 20 + 0.3 * 2000 * 15)}
    nf, ns = _counts(case)
    pairs = 4.19 * (2 * case.get("h_over_dp", 1.3)) ** 3
    if case["path"] == "contact":
        return {"bytes": nf * (32 + 4 * prec) + ns * (64 + 8), "flops": ns * pairs * 0.5 * 20}
    step = nf * (2 * (32 + 4 * prec) + 8 + 4 * prec * 4 + 2 * 8 * prec * 2) + ns * (64 + 12 * prec)
    return {"bytes": case["steps"] * step + nf * 64.0, "flops": case["steps"] * nf * pairs * (15 + 30 + 2 * (35 + 25))}


# ---------------------------------------------------------------------------
# the same in plain torch, FP64
# ---------------------------------------------------------------------------
def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _t(a):
    return torch.as_tensor(np.asarray(a, dtype=np.float64), device=_dev())


def _rows(xi, xj, h, lo, dims, same):
    """For each point of xi its neighbours in xj within 2h: indices [n, K]
    (padded with 0), differences xi - xj, |.| and the mask of real entries."""
    cs = 2.0 * h
    cut2 = cs * cs
    dev = xi.device

    def cells(x):
        return torch.minimum(((x - lo) / cs).floor().long().clamp(min=0), dims - 1)

    ci, cj = cells(xi), cells(xj)
    lin = (cj[:, 2] * dims[1] + cj[:, 1]) * dims[0] + cj[:, 0]
    lin, order = torch.sort(lin)
    total = int(dims.prod())
    start = torch.searchsorted(lin, torch.arange(total + 1, device=dev))
    I, J = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            y, z = ci[:, 1] + dy, ci[:, 2] + dz
            ok = (y >= 0) & (z >= 0) & (y < dims[1]) & (z < dims[2])
            row = (z.clamp(0) * dims[1] + y.clamp(0)) * dims[0]
            row = torch.where(ok, row, torch.zeros_like(row))
            a = start[row + (ci[:, 0] - 1).clamp(min=0)]
            b = start[row + torch.minimum(ci[:, 0] + 1, dims[0] - 1) + 1]
            cnt = torch.where(ok, b - a, torch.zeros_like(a))
            i = torch.repeat_interleave(torch.arange(len(xi), device=dev), cnt)
            off = torch.arange(len(i), device=dev) - torch.repeat_interleave(cnt.cumsum(0) - cnt, cnt)
            j = order[a[i] + off]
            d = xi[i] - xj[j]
            keep = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2] < cut2
            if same:
                keep &= i != j
            I.append(i[keep])
            J.append(j[keep])
    I, J = torch.cat(I), torch.cat(J)
    I, o = torch.sort(I)
    J = J[o]
    cnt = torch.bincount(I, minlength=len(xi))
    K = max(1, int(cnt.max()) if len(xi) else 1)
    nb = torch.zeros((len(xi), K), dtype=torch.long, device=dev)
    mask = torch.zeros((len(xi), K), dtype=torch.bool, device=dev)
    pos = torch.arange(len(I), device=dev) - (cnt.cumsum(0) - cnt)[I]
    nb[I, pos] = J
    mask[I, pos] = True
    d = torch.where(mask[..., None], xi[:, None, :] - xj[nb], torch.zeros((), dtype=torch.float64, device=dev))
    return nb, d, d.square().sum(-1).sqrt(), mask


def _W(r, h, mask):
    q = r / h
    k = 21.0 / (16.0 * math.pi * h ** 3)
    return torch.where(mask, k * (1 - 0.5 * q) ** 4 * (1 + 2 * q), torch.zeros_like(r))


def _F(r, h, mask):
    k = -5.0 * 21.0 / (16.0 * math.pi * h ** 5)
    return torch.where(mask, k * (1 - 0.5 * r / h) ** 3, torch.zeros_like(r))


def _outer(a, b):
    """sum over the neighbours of the outer products [n, 3, 3]"""
    return torch.stack([(a * b[..., k:k + 1]).sum(1) for k in range(3)], -1)


def _lattice(hod, half):
    R = int(math.ceil(2 * hod)) + 1
    g = np.arange(-R, R + 1)
    a, b, c = np.meshgrid(g, g, g, indexing="ij")
    q = np.sqrt(a * a + b * b + c * c) / hod
    w = 21.0 / (16.0 * math.pi * hod ** 3) * (1 - 0.5 * q) ** 4 * (1 + 2 * q) * (q < 2)
    return float(w[a > 0].sum() if half else w.sum())


class _Exact:
    """The scheme of the paper's Section 2 in FP64 torch."""

    def __init__(self, c):
        p = self.p = c.params
        self.c = c
        self.h = p["h_over_dp"] * p["dp"]
        self.lo = _t(p["grid_lo"])
        self.dims = torch.ceil((_t(p["grid_hi"]) - self.lo) / (2 * self.h)).long()
        self.x, self.v, self.rho, self.T = _t(c.xf), _t(c.vf), _t(c.rhof), _t(c.Tf)
        self.drho = torch.zeros_like(self.rho)
        self.m, self.V = p["rho0"] * p["dp"] ** 3, p["dp"] ** 3
        mats = p.get("materials") or [(p["k_f"], p["cp_f"])]
        ix = torch.as_tensor(c.material if c.material is not None else np.zeros(c.nf), device=_dev()).long()
        self.k, self.cp = _t([m[0] for m in mats])[ix], _t([m[1] for m in mats])[ix]
        self.dt_T = min(0.5 * p["rho0"] * cp * self.h ** 2 / k for k, cp in mats)
        self.body = torch.as_tensor(c.body, device=_dev()).long()
        self.ctr, self.om = _t([b.center for b in c.bodies]), _t([b.omega for b in c.bodies])
        ax = _t([b.axis for b in c.bodies])
        self.ax = ax / ax.norm(dim=1, keepdim=True)
        self.bT, self.bk = _t([b.T for b in c.bodies]), _t([b.k for b in c.bodies])
        u = _t(c.xs0) - self.ctr[self.body]
        a = self.ax[self.body]
        r = (u - (u * a).sum(-1, keepdim=True) * a).norm(dim=1)
        self.tip = float((self.om[self.body].abs() * r).max()) if c.ns else 0.0
        self.t, self.n, self.sub = 0.0, 0, 0
        self.tot = dict(heat=0.0, diss=0.0, body=torch.zeros((len(c.bodies), 3), dtype=torch.float64, device=_dev()))
        self.S0 = _lattice(p["h_over_dp"], False)

    def geometry(self):
        c, h = self.c, self.h
        a, th = self.ax[self.body], (self.om * self.t)[self.body][:, None]

        def turn(u):
            return u * th.cos() + torch.linalg.cross(a, u) * th.sin() + a * (a * u).sum(-1, keepdim=True) * (1 - th.cos())

        self.lev = turn(_t(c.xs0) - self.ctr[self.body])
        self.xs = self.ctr[self.body] + self.lev
        self.nw = turn(_t(c.ns0))
        self.vw = torch.linalg.cross(self.om[self.body][:, None] * a, self.lev)
        self.ff = _rows(self.x, self.x, h, self.lo, self.dims, True)
        self.fs = _rows(self.x, self.xs, h, self.lo, self.dims, False)
        sw = 21.0 / (16.0 * math.pi * h ** 3)
        sw = sw + _W(self.ff[2], h, self.ff[3]).sum(1) + _W(self.fs[2], h, self.fs[3]).sum(1)
        re = self.p["rho0"] * self.V * sw / self.S0
        self.rho = torch.maximum(self.rho, re) if self.p["free_surface"] else re

    def body_sum(self, nb, f):
        """Sums over wall pairs f [n, K, q] by the body of the pair's solid particle."""
        out = torch.zeros((len(self.om), f.shape[-1]), dtype=torch.float64, device=f.device)
        b = self.body[nb]
        for k in range(len(self.om)):
            out[k] = (f * (b == k)[..., None]).sum((0, 1))
        return out

    def step(self):
        p, h, m, V, c0, rho0 = self.p, self.h, self.m, self.V, self.p["c0"], self.p["rho0"]
        self.geometry()
        vm = max(float(self.v.norm(dim=1).max()), self.tip)
        visc = h * h / p["nu"]
        tad = min(p["cfl_ad"] * min(h / vm if vm > 0 else visc, visc), self.dt_T)
        tac = p["cfl_ac"] * h / (c0 + vm)
        nac = max(1, math.ceil(tad / tac))
        if nac > p["nac_max"]:
            nac, tad = p["nac_max"], p["nac_max"] * tac
        dt = tad / nac
        g = _t(p["gravity"])
        nb, d, r, mk = self.ff
        F = _F(r, h, mk)
        wb, dw, rw, wk = self.fs
        Fw = _F(rw, h, wk)
        eta = rho0 * p["nu"]
        # dummy velocity of the walls (eq. 18)
        vd = self.vw
        if not p.get("wall_visc") and len(self.xs):
            sb, _, sr, sk = _rows(self.xs, self.x, h, self.lo, self.dims, False)
            w = _W(sr, h, sk)
            ws = w.sum(1)
            mean = (w[..., None] * self.v[sb]).sum(1) / torch.where(ws > 0, ws, torch.ones_like(ws))[:, None]
            vd = torch.where((ws > 0)[:, None], 2 * self.vw - mean, self.vw)
        rho, T = self.rho, self.T
        Vj = m / rho[nb]
        c2 = (2 * eta / rho)[:, None]
        dv = self.v[:, None, :] - self.v[nb]
        av = ((c2 * Vj * F)[..., None] * dv).sum(1)
        Kij = 4 * self.k[:, None] * self.k[nb] / (self.k[:, None] + self.k[nb])
        hs = (Vj * Kij * (T[:, None] - T[nb]) * F).sum(1)
        G = _outer(-dv * (Vj * F)[..., None], d) if p["viscous_heating"] else None
        del dv, Kij
        fw = (c2 * V * Fw)[..., None] * (self.v[:, None, :] - vd[wb])
        av = av + fw.sum(1)
        bw = self.body[wb]
        Kiw = 4 * self.k[:, None] * self.bk[bw] / (self.k[:, None] + self.bk[bw])
        term = V * Kiw * (T[:, None] - self.bT[bw]) * Fw
        hs = hs + term.sum(1)
        rc = 1 / (rho * self.cp)
        lev = self.lev[wb]
        gx = -m * fw
        vis = self.body_sum(wb, torch.cat([gx, torch.linalg.cross(lev, gx), (m * self.cp * rc)[:, None, None] * term[..., None]], -1))
        ds = 0.0
        if G is not None:
            G = G + _outer((V * Fw)[..., None] * (self.vw[wb] - self.v[:, None, :]), dw)
            S = 0.5 * (G + G.transpose(1, 2))
            phi = 2 * eta * S.square().sum((1, 2))
            hs = hs + phi
            ds = tad * float((m / rho * phi).sum())
        dT = rc * hs
        pr = torch.zeros((len(self.om), 6), dtype=torch.float64, device=d.device)
        x, v = self.x, self.v
        inv = torch.where(r > 0, 1 / r, torch.zeros_like(r))
        for _ in range(nac):
            rho = rho + 0.5 * dt * self.drho
            x = x + 0.5 * dt * v
            P = c0 * c0 * (rho - rho0)
            rj = rho[nb]
            dU = -((v[:, None, :] - v[nb]) * d).sum(-1) * inv
            beta = torch.clamp(3 * torch.clamp(dU, min=0), max=c0)
            ps = 0.5 * (P[:, None] + P[nb]) + rho[:, None] * rj * beta * dU / (rho[:, None] + rj)
            a = ((-2 / rho[:, None] * (m / rj) * ps * F)[..., None] * d).sum(1)
            PR = P[:, None] - rho[:, None] * (dw * g).sum(-1)
            rR = rho0 + PR / (c0 * c0)
            pw = (rho[:, None] * PR + rR * P[:, None]) / (rho[:, None] + rR)
            f = (-2 / rho[:, None] * V * pw * Fw)[..., None] * dw
            a = a + f.sum(1)
            pr += self.body_sum(wb, torch.cat([-m * f, torch.linalg.cross(lev, -m * f)], -1))
            v = v + dt * (a + av + g)
            x = x + 0.5 * dt * v
            s = 0.5 * ((v[:, None, :] - v[nb]) * d).sum(-1) + (P[:, None] - P[nb]) * r / (c0 * (rho[:, None] + rj))
            s = ((m / rj) * s * F).sum(1)
            n = self.nw[wb]
            UL, uw = -(n * v[:, None, :]).sum(-1), -(n * self.vw[wb]).sum(-1)
            Us = uw + (P[:, None] - PR) / (c0 * (rho[:, None] + rR))
            s = s + (V * (Us - UL) * (n * dw).sum(-1) * Fw).sum(1)
            self.drho = 2 * rho * s
            rho = rho + 0.5 * dt * self.drho
        self.x, self.v, self.rho, self.T = x, v, rho, T + tad * dT
        self.t += tad
        self.n += 1
        self.sub += nac
        force, torque = vis[:, 0:3] + pr[:, 0:3] / nac, vis[:, 3:6] + pr[:, 3:6] / nac
        ta = (self.ax * torque).sum(1)
        now = torch.stack([ta, -self.om * ta, vis[:, 6]], 1)
        self.tot["body"] += tad * now
        hst = tad * float(vis[:, 6].sum())
        self.tot["heat"] += hst
        self.tot["diss"] += ds
        v2 = v.square().sum(1)
        self.rep = dict(t=self.t, dt_ad=tad, dt=dt, vmax=float(v2.max().sqrt()), mass=m * len(x),
                        kinetic=float(0.5 * m * v2.sum()), thermal=float((m * self.cp * self.T).sum()), heat_step=hst,
                        heat_total=self.tot["heat"], mass_proxy=float(rho.sum() * V), diss_step=ds, diss_total=self.tot["diss"])
        ints = self.tot["body"]
        self.bod = dict(force=force, torque=torque, torque_axis=ta, power=now[:, 1], heat_rate=now[:, 2],
                        torque_axis_int=ints[:, 0].clone(), energy_int=ints[:, 1].clone(), heat_int=ints[:, 2].clone())

    def answer(self):
        out = {k: getattr(self, k).cpu().numpy() for k in ("x", "v", "rho", "T")}
        out["counts"] = [self.n, math.nan if not self.n else round(self.rep["dt_ad"] / self.rep["dt"]), self.sub]
        out["report"] = dict(self.rep)
        out["bodies"] = {k: self.bod[k].cpu().numpy() for k in BODY}
        return out


def _phi(shape, x):
    """Signed distance of the relaxation bodies, negative inside."""
    d = x - _t(shape["center"])
    s, kind = shape["size"], shape["kind"]
    if kind == "sphere":
        return d.norm(dim=-1) - s[0]
    if kind == "box":
        q = d.abs() - _t(s)
        return q.clamp(min=0).norm(dim=-1) + q.amax(-1).clamp(max=0)
    r = (d[..., 0].square() + d[..., 2].square()).sqrt()
    if kind == "cylinder":
        d2, half = r - s[0], s[1]
    else:
        tip, root, half = s
        z = shape["teeth"]
        k = torch.floor(2 * (z / (2 * math.pi) * torch.atan2(d[..., 2], d[..., 0]) + 0.25 + shape["phase"]))
        even = torch.remainder(k, 2) == 0
        Rn = torch.where(even, torch.full_like(r, root), torch.full_like(r, tip))
        best = (r - torch.where(even, torch.full_like(r, tip), torch.full_like(r, root))).abs()
        for j in (-1, 0, 1, 2):
            th = 2 * math.pi * (0.5 * (k + j) - 0.25 - shape["phase"]) / z
            ex, ez = th.cos(), th.sin()
            t = (d[..., 0] * ex + d[..., 2] * ez).clamp(root, tip)
            best = torch.minimum(best, ((d[..., 0] - t * ex).square() + (d[..., 2] - t * ez).square()).sqrt())
            best = torch.minimum(best, ((d[..., 0] - Rn * ex).square() + (d[..., 2] - Rn * ez).square()).sqrt())
        d2 = torch.where((r <= root) | ((r <= tip) & even), -best, best)
    dy = d[..., 1].abs() - half
    return (d2.clamp(min=0).square() + dy.clamp(min=0).square()).sqrt() + torch.maximum(d2, dy).clamp(max=0)


def _exact_relax(case, seed):
    c, shape = _body(case, seed), _shape(case)
    p = c.params
    dp, h = p["dp"], p["h_over_dp"] * p["dp"]
    V, m, de = dp ** 3, p["rho0"] * dp ** 3, 0.25 * h
    x = _t(c.xf)
    lo = _t(p["grid_lo"])
    dims = torch.ceil((_t(p["grid_hi"]) - lo) / (2 * h)).long()
    g = (torch.arange(-8, 8, device=_dev(), dtype=torch.float64) + 0.5) * de
    off = torch.stack(torch.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    off = off[off.norm(dim=1) < 2 * h]
    rr = off.norm(dim=1)
    w = _F(rr, h, rr < 2 * h)[:, None] * -off * de ** 3
    for it in range(case["iterations"]):
        nb, d, r, mk = _rows(x, x, h, lo, dims, True)
        s = V * (_F(r, h, mk)[..., None] * d).sum(1)
        near = torch.nonzero(_phi(shape, x) > -2 * h - de)[:, 0]
        for k in range(0, len(near), 16384):
            i = near[k:k + 16384]
            f = (0.5 + _phi(shape, x[i][:, None, :] + off) / de).clamp(0, 1)
            s[i] += (f[..., None] * w).sum(1)
        a = -(2 / m) * V * s
        amax = float(a.norm(dim=1).max())
        dt = 0.25 * math.sqrt(h / amax)
        first = amax if it == 0 else first
        x = x + 0.5 * a * dt * dt
        phi = _phi(shape, x)
        i = torch.nonzero(phi > -0.5 * dp)[:, 0]
        e = torch.eye(3, dtype=torch.float64, device=x.device) * (1e-6 * h)
        n = torch.stack([_phi(shape, x[i] + e[q]) - _phi(shape, x[i] - e[q]) for q in range(3)], -1)
        x[i] -= (phi[i] + 0.5 * dp)[:, None] * n / n.norm(dim=1, keepdim=True)
    return {"x": x.cpu().numpy(), "amax_first": first, "amax_last": amax, "dt_last": dt, "bounded_last": int(len(i))}


def exact(case, seed):
    path = case["path"]
    if path == "relax":
        return _exact_relax(case, seed)
    if path == "pool":
        return None   # hundreds of steps in FP64 take longer than 20 s
    e = _Exact(_solve(case, seed))
    if path == "contact":
        e.geometry()
        nb, _, r, mk = _rows(e.xs, e.x, e.h, e.lo, e.dims, False)
        z = ((e.m / e.rho[nb]) * _W(r, e.h, mk)).sum(1) / _lattice(e.p["h_over_dp"], True)
        mean = [float(z[e.body == b].mean()) if bool((e.body == b).any()) else 0.0 for b in range(len(e.om))]
        return {"zeta": z.cpu().numpy(), "mean": np.array(mean)}
    if _counts(case)[0] * case["steps"] > 9e6:
        return None   # over 20 s
    for _ in range(case["steps"]):
        e.step()
    return e.answer()
