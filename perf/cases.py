"""The work that a program using this framework has it do, as cases that can be timed and compared.

Four kinds of call, each through the public entry points of paper_2108_08919_amd:
  box          time steps of one periodic box, then the box's state as a program records it
  ensemble     time steps of several boxes of uneven size advanced together, then every state
  learned      macro steps corrected by the network, then the box's state
  train        minibatch training of the network, then its weights
  diagnostics  the reductions, spectrum, defects, vorticity correlation, pathlines and mixing
               of one stored state

Inputs come from numpy and torch alone: particles on a lattice or displaced from it, a few
smooth velocity modes, random or nearly aligned directors. exact() computes the same outputs
in 64 bits with torch, written from the paper's equations.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

DT = 1e-3          # time step of every box
FIELDS32 = ("ux", "uy", "qxx", "qxy", "rho", "ax", "ay", "qyy", "qzz")


# ------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest box a program steps (64 x 64, nearly aligned start), a few steps between
        # two looks at it: launches and latency
        _box("box64", 64, 10, start="lattice", angles="small", zeta=0.01),
        # an odd side: ragged tiles at two edges; the second-order corrector, a disordered state
        _box("box137_midpoint", 137, 40, integrator=1),
        # the conservative pair forces of momentum studies, odd side, contractile activity
        _box("box211_conservative", 211, 40, form=1, zeta=-0.02),
        # the 3 x 3 order tensor in an in-plane flow
        _box("box256_quasi2d", 256, 40, q3d=1, B=0.3, lam=0.9),
        # the full elastic stress
        _box("box300_elastic", 300, 40, elastic=1),
        # a single run at scale: 512 x 512 from an isotropic start on the lattice
        _box("box512", 512, 100, start="lattice"),
        # the compact kernel on a million particles, with the tile its documentation advises
        _box("box1024_wendland", 1024, 100, kernel=1, tile=8),
        # the large box that throughput is quoted on, 250 steps between two records
        _box("box2048", 2048, 250, start="lattice"),
        # 32 replicas of sides 128 to 384 in one launch, replayed from a captured graph:
        # a parameter sweep
        dict(name="ensemble32", kind="ensemble", replicas=32, lo=128, hi=384, draw=0, steps=100, graph=10),
        # macro steps of four time steps corrected by the network, on a 512 x 512 box
        dict(name="learned512", kind="learned", side=512, mult=4, macro=25),
        # an epoch of the corrector's training at its own batch size
        dict(name="train256k", kind="train", samples=262144, batch=4096, epochs=2),
        # what a sweep looks at between its steps, on a grid of the box's own spacing
        dict(name="diagnostics512", kind="diagnostics", side=512, grid=512),
    ]


def _box(name, side, steps, start="jitter", angles="isotropic", zeta=0.02, **kw):
    c = dict(kind="box", side=side, steps=steps, start=start, angles=angles, zeta=zeta, K=0.02, lam=0.7, B=0.0,
             kernel=0, integrator=0, form=0, elastic=0, q3d=0, tile=4, lpp=1)
    if name:
        c["name"] = name
    c.update(kw)
    return c


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["box"] * 6 + ["ensemble", "learned", "train", "diagnostics"])
    if kind == "box":
        side = _log_int(rng, 60, 1700)
        most = max(10, min(250, int(2.5e8 / side ** 2)))
        variant = rng.choice([{}, {}, dict(integrator=1), dict(form=1), dict(elastic=1), dict(q3d=1, B=0.3),
                              dict(kernel=1), dict(kernel=1, tile=8)])
        return _box(None, side, _log_int(rng, 5, most), start=rng.choice(["lattice", "jitter"]),
                    zeta=rng.choice([-1, 1]) * round(math.exp(rng.uniform(math.log(0.005), math.log(0.04))), 4),
                    K=round(math.exp(rng.uniform(math.log(0.01), math.log(0.08))), 4), **variant)
    if kind == "ensemble":
        lo = rng.randrange(60, 160)
        return dict(kind="ensemble", replicas=rng.randrange(2, 33), lo=lo, hi=lo + rng.randrange(1, 180),
                    draw=rng.randrange(1000), steps=rng.randrange(10, 100), graph=rng.choice([0, 10]))
    if kind == "learned":
        return dict(kind="learned", side=_log_int(rng, 96, 1024), mult=rng.choice([4, 4, 16]), macro=rng.randrange(5, 25))
    if kind == "train":
        return dict(kind="train", samples=_log_int(rng, 20000, 500000), batch=rng.choice([1024, 2048, 4096, 8192]),
                    epochs=1)
    grid = rng.choice([64, 128, 256, 512, 1024])
    return dict(kind="diagnostics", side=grid, grid=grid, variant=rng.randrange(1, 100))


# ------------------------------------------------------------------ inputs

def _fields(side, seed, start="jitter", angles="isotropic", amp_u=2e-3, q3d=0):
    """One box's fields in 64 bits, particle id = row * side + column of the lattice."""
    rng = np.random.default_rng(seed)
    c = np.arange(side) + 0.5
    x, y = (v.ravel().copy() for v in np.meshgrid(c, c, indexing="xy"))
    n = x.size
    if start == "jitter":
        x = np.mod(x + rng.uniform(-0.2, 0.2, n), side)
        y = np.mod(y + rng.uniform(-0.2, 0.2, n), side)
    ux, uy = np.zeros(n), np.zeros(n)
    for _ in range(4):
        kx, ky = rng.integers(-3, 4, size=2)
        ph, a = rng.uniform(0, 2 * math.pi, size=2), rng.normal(size=2) * amp_u
        arg = 2 * math.pi * (kx * x + ky * y) / side
        ux += a[0] * np.sin(arg + ph[0])
        uy += a[1] * np.sin(arg + ph[1])
    th = rng.uniform(-0.1, 0.1, n) if angles == "small" else rng.uniform(0.0, math.pi, n)
    rho = 1.0 + (1e-4 * rng.normal(size=n) if start == "jitter" else 0.0)
    f = dict(x=x, y=y, ux=ux, uy=uy, rho=rho * np.ones(n), ax=np.zeros(n), ay=np.zeros(n))
    if q3d:
        cs, sn = np.cos(th), np.sin(th)
        f.update(qxx=1.5 * (cs * cs - 1 / 3), qxy=1.5 * cs * sn, qyy=1.5 * (sn * sn - 1 / 3))
    else:
        f.update(qxx=np.cos(2 * th), qxy=np.sin(2 * th))
    return f


def _params(side, zeta=0.02, K=0.02, lam=0.7, B=0.0, kernel=0, integrator=0, form=0, elastic=0, q3d=0):
    return SimpleNamespace(L=float(side), dx=1.0, h=1.3, rho0=1.0, eta=1.0, Gamma=0.34, lam=lam, A=0.0, B=B, C=0.5,
                           K=K, zeta=zeta, dt=DT, gamma_eos=7.0, beta=1.0, c0_factor=10.0, skin=0.1, form=form,
                           elastic=elastic, apd=1, kernel=kernel, integrator=integrator, q3d=q3d)


PHYS = ("zeta", "K", "lam", "B", "kernel", "integrator", "form", "elastic", "q3d")


def _replicas(case):
    rng = np.random.default_rng(case["draw"])
    zetas, Ks = (0.005, 0.01, 0.02, 0.04), (0.01, 0.02, 0.04, 0.08)
    return [(int(rng.integers(case["lo"], case["hi"] + 1)), zetas[(r // 8) % 4], Ks[(r // 2) % 4])
            for r in range(case["replicas"])]


def _network(seed):
    """Weights (W1, b1, W2, b2, W3, b3, flat) and normalisation of a corrector of realistic size:
    z-scored inputs, corrections of a few 1e-6."""
    rng = np.random.default_rng(seed + 77)
    w = np.concatenate([rng.normal(size=12 * 64) / math.sqrt(12), 0.1 * rng.normal(size=64),
                        rng.normal(size=64 * 64) / 8, 0.1 * rng.normal(size=64),
                        rng.normal(size=64 * 5) / 8, 0.1 * rng.normal(size=5)]).astype(np.float32)
    norm = np.concatenate([np.zeros(12), [0.7, 0.7, 1e-3, 1e-3, 1e-3, 1e-3, 0.4, 0.4, 1e-4, 1.0, 1e-4, 1e-4],
                           np.zeros(5), [2e-6, 2e-6, 2e-6, 1e-7, 1e-7]]).astype(np.float32)
    return w, norm


def _samples(case, seed):
    """Training inputs and targets with the spread of the solver's own samples."""
    g = torch.Generator(device="cpu").manual_seed(int(seed))
    z = torch.randn((case["samples"], 12), generator=g)
    mix = torch.randn((12, 5), generator=g) / 4
    t = torch.tanh(z @ mix) + 0.1 * torch.randn((case["samples"], 5), generator=g)
    scale = torch.tensor([0.7, 0.7, 1e-3, 1e-3, 1e-3, 1e-3, 0.4, 0.4, 1e-4, 0.01, 1e-4, 1e-4])
    return z * scale, t * torch.tensor([2e-6, 2e-6, 2e-6, 1e-7, 1e-7])


def prepare(case, seed):
    import paper_2108_08919_amd as P
    if case["kind"] == "train":
        m = P.Mlp()
        X, T = (v.cuda() for v in _samples(case, seed))
        m.fit_norm(X, T)
        m.set_weights(_network(seed)[0])
        return SimpleNamespace(case=case, mlp=m, X=X, T=T)
    if case["kind"] == "ensemble":
        reps = _replicas(case)
        sim = P.Sim([_params(s, z, k) for s, z, k in reps], [s * s for s, _, _ in reps])
        for r, (s, _, _) in enumerate(reps):
            sim.set_state(r, _fields(s, 1000 * seed + r, start="lattice"))
        if case["graph"]:
            sim.set_option(P.NEM_OPT_GRAPH, case["graph"])
        return SimpleNamespace(case=case, sim=sim)
    side = case["side"]
    if case["kind"] == "box":
        sim = P.Sim([_params(side, **{k: case[k] for k in PHYS})], [side * side])
        sim.set_option(P.NEM_OPT_TILE, case["tile"])
        sim.set_option(P.NEM_OPT_LPP, case["lpp"])
        sim.set_state(0, _fields(side, seed, case["start"], case["angles"], q3d=case["q3d"]))
        return SimpleNamespace(case=case, sim=sim)
    sim = P.Sim([_params(side)], [side * side])
    sim.set_state(0, _fields(side, seed))
    st = SimpleNamespace(case=case, sim=sim)
    if case["kind"] == "learned":
        st.mlp = P.Mlp()
        w, norm = _network(seed)
        st.mlp.set_weights(w)
        st.mlp.set_norm(norm)
    else:
        st.ids = np.random.default_rng(seed).choice(side * side, min(4096, side * side), replace=False).astype(np.int32)
        q = np.arange(side) >= side // 2
        st.colour = (2 * q[:, None] + q[None, :]).astype(np.uint8).ravel()
    return st


# --------------------------------------------------------------------- run

def _record(f):
    """A state as a program keeps it: positions in 64 bits, the fields in the 32 that the solver holds."""
    return {k: v.astype(np.float32) if k in FIELDS32 else v for k, v in f.items()}


def run(state):
    case = state.case
    if case["kind"] == "box":
        state.sim.step(case["steps"])
        return _record(state.sim.get_state(0))
    if case["kind"] == "ensemble":
        state.sim.step(case["steps"])
        f = [_record(state.sim.get_state(r)) for r in range(case["replicas"])]
        return {k: np.concatenate([g[k] for g in f]) for k in f[0]}
    if case["kind"] == "learned":
        fallbacks, worst = state.sim.step_learned(state.mlp, case["macro"], case["mult"])
        return dict(_record(state.sim.get_state(0)), fallbacks=fallbacks, worst=np.float32(worst))
    if case["kind"] == "train":
        loss = state.mlp.train(state.X, state.T, case["epochs"], case["batch"], 2e-3)
        return dict(weights=state.mlp.get_weights(), loss=np.float32(loss))
    sim, M = state.sim, case["grid"]
    out = dict(diag=sim.diagnostics(0))
    out["spectrum"], out["slope"] = sim.spectrum(0, M)
    out["defects"] = sim.defects(0, M)
    out["cx"], out["cy"], out["lx"], out["ly"] = sim.vorticity_correlation(0, M)
    out["track"] = sim.track(state.ids)
    out["mixing"] = sim.mixing(state.colour, 4, max(2, M // 8))
    return out


def work(case):
    """Per particle and step: offsets (high and low), u, Q, rho - rho0, the acceleration and the
    pair passes' intermediate fields, 208 bytes; 8352 FLOP over 44 neighbours (quintic), about
    3900 over 20 (Wendland). The network: 2 (12 64 + 64 64 + 64 5) per sample and pass."""
    mlp = 2 * (12 * 64 + 64 * 64 + 64 * 5)
    if case["kind"] == "box":
        n = case["side"] ** 2
        return dict(bytes=n * (208 * case["steps"] + 72), flops=n * case["steps"] * (3900 if case["kernel"] else 8352))
    if case["kind"] == "ensemble":
        n = sum(s * s for s, _, _ in _replicas(case))
        return dict(bytes=n * (208 * case["steps"] + 72), flops=n * case["steps"] * 8352)
    if case["kind"] == "learned":
        n = case["side"] ** 2
        return dict(bytes=n * ((208 + 136) * case["macro"] + 72), flops=n * case["macro"] * (8352 + mlp))
    if case["kind"] == "train":
        n = case["epochs"] * (case["samples"] // case["batch"]) * case["batch"]
        return dict(bytes=n * 68, flops=3 * mlp * n)
    n, M = case["side"] ** 2, case["grid"]
    fft = 5 * M * M * 2 * math.log2(M)
    return dict(bytes=n * 6 * 40 + M * M * 3 * 80, flops=n * 5000 + 3 * M * M * 44 * 30 + 3 * fft)


# --------------------------------------------- the same in 64 bits, by torch

def _table(side, reach, dev):
    """Table (n, K) of the lattice ids within `reach` of each particle's own site."""
    w = int(math.ceil(reach)) + 1
    a = torch.arange(side, device=dev)
    cols = []
    for dj in range(-w, w + 1):
        for di in range(-w, w + 1):
            if (di or dj) and math.hypot(di, dj) < reach:
                cols.append((((a + dj) % side)[:, None] * side + ((a + di) % side)[None, :]).reshape(-1))
    return torch.stack(cols, 1)


class _Box64:
    """The time step of one box in 64 bits."""

    def __init__(self, p, f, dev):
        self.p, self.side = p, int(p.L)
        self.f = {k: torch.tensor(np.asarray(v), dtype=torch.float64, device=dev) for k, v in f.items()}
        self.R = (2.0 if p.kernel else 3.0) * p.h
        # displaced by up to 0.2 per direction at the start, and a little more on the way
        self.idx = _table(self.side, self.R + 0.75, dev)
        self.n = self.side ** 2
        self.chunk = max(1, (1 << 23) // self.idx.shape[1])

    def chunks(self):
        for b in range(0, self.n, self.chunk):
            yield slice(b, min(self.n, b + self.chunk))

    def pairs(self, s, x, y, xi=None, yi=None):
        """j, r vector, r, W and F = W'/r of the pairs of rows s (zero where not neighbours)."""
        p, j = self.p, self.idx[s]
        rx = (x[s] if xi is None else xi[s])[:, None] - x[j]
        ry = (y[s] if yi is None else yi[s])[:, None] - y[j]
        rx = rx - p.L * torch.round(rx / p.L)
        ry = ry - p.L * torch.round(ry / p.L)
        r = torch.sqrt(rx * rx + ry * ry)
        m = ((r > 0) & (r < self.R)).to(torch.float64)
        r = torch.where(m > 0, r, torch.ones_like(r))
        q = r / p.h
        if p.kernel:
            a = 7.0 / (4.0 * math.pi * p.h ** 2)
            t = (1 - 0.5 * q).clamp(min=0)
            W, F = a * t ** 4 * (1 + 2 * q), -5 * a / p.h ** 2 * t ** 3
            self.W0 = a
        else:
            a = 7.0 / (478.0 * math.pi * p.h ** 2)
            t3, t2, t1 = (3 - q).clamp(min=0), (2 - q).clamp(min=0), (1 - q).clamp(min=0)
            W = a * (t3 ** 5 - 6 * t2 ** 5 + 15 * t1 ** 5)
            F = -5 * a / p.h * (t3 ** 4 - 6 * t2 ** 4 + 15 * t1 ** 4) / r
            self.W0 = 66 * a
        return j, rx, ry, r, m * W, m * F, m

    def gradients(self, s, x, y, V, fields):
        """B and the corrected gradients of `fields`, with the pair weights."""
        j, rx, ry, r, W, F, m = self.pairs(s, x, y)
        c = V[j] * F
        axx, axy, ayy = -(c * rx * rx).sum(1), -(c * rx * ry).sum(1), -(c * ry * ry).sum(1)
        det = axx * ayy - axy * axy
        B = (ayy / det, -axy / det, axx / det)
        g = []
        for v in fields:
            d = (v[j] - v[s][:, None]) * c
            gx, gy = (d * rx).sum(1), (d * ry).sum(1)
            g.append((gx * B[0] + gy * B[1], gx * B[1] + gy * B[2]))
        return j, rx, ry, r, W, F, m, c, B, g

    def laplacian(self, v, s, j, rx, ry, r, c, B):
        d = -(v[j] - v[s][:, None]) * c / r ** 2
        return 2 * (B[0] * (d * rx * rx).sum(1) + 2 * B[1] * (d * rx * ry).sum(1) + B[2] * (d * ry * ry).sum(1))

    def volumes(self, x, y):
        V = torch.empty_like(x)
        for s in self.chunks():
            W = self.pairs(s, x, y)[4].sum(1)
            V[s] = 1 / (self.W0 + W)
        return V

    def step(self, dt):
        p, f = self.p, self.f
        un, vn = f["ux"], f["uy"]
        u, v = un + 0.5 * dt * f["ax"], vn + 0.5 * dt * f["ay"]
        x, y = f["x"] + 0.5 * dt * u, f["y"] + 0.5 * dt * v
        V = self.volumes(x, y)
        qa, qb = f["qxx"], f["qxy"]
        qc = f["qyy"] if p.q3d else -qa
        new = {k: torch.empty_like(qa) for k in ("qa", "qb", "qc", "k", "px", "py", "Bxx", "Bxy", "Byy", "Pa", "Pb")}
        feat = torch.empty((self.n, 12), dtype=torch.float64, device=x.device)
        for s in self.chunks():
            fields = [u, v, qa, qb] + ([qc] if p.q3d else [])
            j, rx, ry, r, W, F, m, c, B, g = self.gradients(s, x, y, V, fields)
            (G11, G12), (G21, G22), (dax, day), (dbx, dby) = g[:4]
            a, b = qa[s], qb[s]
            div, e12, w12 = G11 + G22, 0.5 * (G12 + G21), 0.5 * (G12 - G21)
            la, lb = (self.laplacian(q, s, j, rx, ry, r, c, B) for q in (qa, qb))
            dux, duy = u[j] - u[s][:, None], v[j] - v[s][:, None]
            rho = f["rho"][s]
            new["k"][s] = -rho * div
            if p.q3d:
                cc, z = qc[s], -a - qc[s]
                lc = self.laplacian(qc, s, j, rx, ry, r, c, B)
                t2 = a * a + 2 * b * b + cc * cc + z * z
                bulk = p.A + p.C * t2
                Ha = -bulk * a + p.B * (a * a + b * b - t2 / 3) + p.K * la
                Hb = -bulk * b + p.B * b * (a + cc) + p.K * lb
                Hc = -bulk * cc + p.B * (b * b + cc * cc - t2 / 3) + p.K * lc
                Hz = -bulk * z + p.B * (z * z - t2 / 3) - p.K * (la + lc)
                xx, yy, zz = a + 1 / 3, cc + 1 / 3, z + 1 / 3
                l2 = 2 * p.lam * (a * G11 + 2 * b * e12 + cc * G22)
                Sxx = 2 * p.lam * (G11 * xx + e12 * b) + 2 * w12 * b - l2 * xx
                Sxy = p.lam * (e12 * (xx + yy) + b * div) + w12 * (yy - xx) - l2 * b
                Syy = 2 * p.lam * (e12 * b + G22 * yy) - 2 * w12 * b - l2 * yy
                tr = (Sxx + Syy - l2 * zz + p.Gamma * (Ha + Hc + Hz)) / 3
                new["qa"][s] = a + dt * (Sxx + p.Gamma * Ha - tr)
                new["qb"][s] = b + dt * (Sxy + p.Gamma * Hb)
                new["qc"][s] = cc + dt * (Syy + p.Gamma * Hc - tr)
                divx, divy = dax + dby, dbx + g[4][1]
            else:
                bulk = p.A + 2 * p.C * (a * a + b * b)
                Ha, Hb = -bulk * a + p.K * la, -bulk * b + p.K * lb
                QG = a * (G11 - G22) + 2 * b * e12
                Sa = p.lam * (a * div + 0.5 * (G11 - G22)) + 2 * w12 * b - 2 * p.lam * a * QG
                Sb = p.lam * (b * div + e12) - 2 * w12 * a - 2 * p.lam * b * QG
                new["qa"][s], new["qb"][s] = a + dt * (Sa + p.Gamma * Ha), b + dt * (Sb + p.Gamma * Hb)
                divx, divy = dax + dby, dbx - day
            sv = -(dux * rx + duy * ry) / r ** 2
            if p.form:
                new["k"][s] = -((dux * rx + duy * ry) * F).sum(1)
                w = 8 * p.eta * sv / (rho[:, None] * f["rho"][j]) * F
                ca = (a / rho ** 2)[:, None] + qa[j] / f["rho"][j] ** 2
                cb = (b / rho ** 2)[:, None] + qb[j] / f["rho"][j] ** 2
                new["px"][s] = (w * rx).sum(1) - p.zeta * ((ca * rx + cb * ry) * F).sum(1)
                new["py"][s] = (w * ry).sum(1) - p.zeta * ((cb * rx - ca * ry) * F).sum(1)
            else:
                vx, vy = (sv * c * rx).sum(1), (sv * c * ry).sum(1)
                new["px"][s] = 8 * p.eta * (vx * B[0] + vy * B[1]) - p.zeta * divx
                new["py"][s] = 8 * p.eta * (vx * B[1] + vy * B[2]) - p.zeta * divy
            if p.elastic:
                QH = 2 * (a * Ha + b * Hb)
                new["Pa"][s], new["Pb"][s] = p.lam * (2 * QH * a - Ha), p.lam * (2 * QH * b - Hb)
            new["Bxx"][s], new["Bxy"][s], new["Byy"][s] = B
            feat[s, :10] = torch.stack([a, b, G11, G12, G21, G22, Ha, Hb, rho - 1.0, torch.full_like(a, p.zeta)], 1)
        rhoh = f["rho"] + 0.5 * dt * new["k"]
        c0 = p.c0_factor * float(torch.sqrt((u * u + v * v).max()))
        rhat, uv = torch.empty_like(x), torch.empty_like(x)
        for s in self.chunks():
            j, rx, ry, r, W, F, m = self.pairs(s, x, y)
            shep = V[s] * (self.W0 * (rhoh[s] - 1.0) + (W * (rhoh[j] - 1.0)).sum(1)) + 1.0
            rhat[s] = rhoh[s] - p.beta * (rhoh[s] - shep)
            uv[s] = V[s] * torch.hypot(((u[s][:, None] - u[j]) * W).sum(1), ((v[s][:, None] - v[j]) * W).sum(1))
        P = c0 ** 2 / p.gamma_eos * torch.expm1(p.gamma_eos * torch.log(rhat)) / rhat ** 2
        out = {k: torch.empty_like(x) for k in ("x", "y", "ux", "uy", "ax", "ay")}
        for s in self.chunks():
            j, rx, ry, r, W, F, m = self.pairs(s, x, y)
            B = new["Bxx"][s], new["Bxy"][s], new["Byy"][s]
            c = F if p.form else V[j] * F
            w = (P[s][:, None] + P[j]) * c
            gx, gy = (w * rx).sum(1), (w * ry).sum(1)
            if p.form:
                ax, ay = new["px"][s] - gx, new["py"][s] - gy
            else:
                ax = -rhat[s] * (gx * B[0] + gy * B[1]) + new["px"][s] / rhat[s]
                ay = -rhat[s] * (gx * B[1] + gy * B[2]) + new["py"][s] / rhat[s]
            if p.elastic:
                d = [(new[k][j] - new[k][s][:, None]) * c for k in ("Pa", "Pb")]
                e = [((q * rx).sum(1), (q * ry).sum(1)) for q in d]
                e = [(gx_ * B[0] + gy_ * B[1], gx_ * B[1] + gy_ * B[2]) for gx_, gy_ in e]
                ax, ay = ax + (e[0][0] + e[1][1]) / rhat[s], ay + (e[1][0] - e[0][1]) / rhat[s]
            if p.integrator:
                out["ux"][s], out["uy"][s] = un[s] + dt * ax, vn[s] + dt * ay
                mx, my = u[s], v[s]
            else:
                out["ux"][s], out["uy"][s] = u[s] + 0.5 * dt * ax, v[s] + 0.5 * dt * ay
                mx, my = out["ux"][s], out["uy"][s]
            w = ((m * r).sum(1) / m.sum(1)) ** 2 * uv[s] * dt
            out["x"][s] = x[s] + 0.5 * dt * mx + w * (m * rx / r ** 3).sum(1)
            out["y"][s] = y[s] + 0.5 * dt * my + w * (m * ry / r ** 3).sum(1)
            out["ax"][s], out["ay"][s] = ax, ay
        feat[:, 10], feat[:, 11] = out["ax"] - f["ax"], out["ay"] - f["ay"]
        out.update(qxx=new["qa"], qxy=new["qb"], rho=rhat + 0.5 * dt * new["k"])
        if p.q3d:
            out["qyy"] = new["qc"]
        self.f = out
        return feat

    def state(self):
        f = dict(self.f, x=self.f["x"] % self.p.L, y=self.f["y"] % self.p.L)
        if self.p.q3d:
            f["qzz"] = -f["qxx"] - f["qyy"]
        return f


def _mlp64(w, z):
    """The network on normalised inputs z, in 64 bits, and its hidden layers."""
    W1, b1, W2, b2, W3, b3 = _split(w)
    h1 = torch.tanh(z @ W1 + b1)
    h2 = torch.tanh(h1 @ W2 + b2)
    return h1, h2, h2 @ W3 + b3


def _split(w):
    return (w[:768].view(12, 64), w[768:832], w[832:4928].view(64, 64), w[4928:4992], w[4992:5312].view(64, 5), w[5312:])


def _exact_train(case, seed, dev):
    X, T = (v.to(dev).double() for v in _samples(case, seed))
    z, t = ((a - a.mean(0)) / a.std(0, unbiased=False) for a in (X, T))
    w = torch.tensor(_network(seed)[0], dtype=torch.float64, device=dev)
    m, v, n, B, lr, it = torch.zeros_like(w), torch.zeros_like(w), case["samples"], case["batch"], 2e-3, 0
    stride = int(0.6180339887 * n) | 1      # the documented per-epoch permutation k -> (k stride + offset) mod n
    while math.gcd(stride, n) != 1:
        stride += 2
    loss = 0.0
    for e in range(case["epochs"]):
        off = (e + 1) * 2654435761 % n
        for first in range(0, n - B + 1, B):
            k = (torch.arange(first, first + B, device=dev) * stride + off) % n
            h1, h2, o = _mlp64(w, z[k])
            W1, b1, W2, b2, W3, b3 = _split(w)
            d = o - t[k]
            loss = 0.5 * (d * d).sum() / B
            d = d / B
            d2 = d @ W3.T * (1 - h2 * h2)
            d1 = d2 @ W2.T * (1 - h1 * h1)
            g = torch.cat([(z[k].T @ d1).reshape(-1), d1.sum(0), (h1.T @ d2).reshape(-1), d2.sum(0),
                           (h2.T @ d).reshape(-1), d.sum(0)])
            it += 1
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            w = w - lr * (m / (1 - 0.9 ** it)) / (torch.sqrt(v / (1 - 0.999 ** it)) + 1e-8)
    return dict(weights=w, loss=loss)


def _exact_diagnostics(case, seed, dev):
    side, M = case["side"], case["grid"]
    p = _params(side)
    box = _Box64(p, _fields(side, seed), dev)
    f = box.f
    V = box.volumes(f["x"], f["y"])
    F = Fg = 0.0
    grid = {k: torch.empty_like(f["x"]) for k in ("ux", "uy", "qxx", "qxy")}
    c = torch.arange(side, dtype=torch.float64, device=dev) + 0.5
    gx, gy = c.repeat(side), c.repeat_interleave(side)   # nodes at the lattice sites (M = side)
    for s in box.chunks():
        j, rx, ry, r, W, _, m, cc, B, g = box.gradients(s, f["x"], f["y"], V, [f["qxx"], f["qxy"]])
        la, lb = (box.laplacian(f[k], s, j, rx, ry, r, cc, B) for k in ("qxx", "qxy"))
        a, b = f["qxx"][s], f["qxy"][s]
        t2 = 2 * (a * a + b * b)
        bulk = 0.5 * p.A * t2 + 0.25 * p.C * t2 * t2
        F = F + (V[s] * (bulk - p.K * (a * la + b * lb))).sum()
        Fg = Fg + (V[s] * (bulk + p.K * sum(q * q for d in g for q in d))).sum()
        j, rx, ry, r, W, _, m = box.pairs(s, f["x"], f["y"], gx, gy)
        w0x, w0y = gx[s] - f["x"][s], gy[s] - f["y"][s]          # the site's own particle is not in the table
        w0x, w0y = w0x - p.L * torch.round(w0x / p.L), w0y - p.L * torch.round(w0y / p.L)
        q = torch.sqrt(w0x ** 2 + w0y ** 2) / p.h
        W0 = box.W0 / 66 * ((3 - q) ** 5 - 6 * (2 - q) ** 5 + 15 * (1 - q).clamp(min=0) ** 5)
        for k in grid:
            grid[k][s] = ((W * f[k][j]).sum(1) + W0 * f[k][s]) / (W.sum(1) + W0)
    ux, uy = grid["ux"].view(M, M), grid["uy"].view(M, M)
    zx, zy = torch.fft.fft2(ux), torch.fft.fft2(uy)
    k = torch.fft.fftfreq(M, 1 / M, dtype=torch.float64, device=dev)
    shell = torch.floor(torch.sqrt(k[:, None] ** 2 + k[None, :] ** 2) + 0.5).long()
    nb = int(math.floor(math.sqrt(2.0) * (M // 2) + 0.5)) + 1
    e = 0.5 * (zx.abs() ** 2 + zy.abs() ** 2) / float(M) ** 4
    E = torch.zeros(nb, dtype=torch.float64, device=dev).index_add_(0, shell.reshape(-1), e.reshape(-1))
    kd = torch.where(k == -M // 2, torch.zeros_like(k), 2 * math.pi / p.L * k)
    om = kd[None, :] * zy - kd[:, None] * zx
    corr = torch.fft.ifft2(om.abs() ** 2).real
    speed = torch.sqrt(f["ux"] ** 2 + f["uy"] ** 2)
    ids = torch.tensor(np.random.default_rng(seed).choice(side * side, min(4096, side * side), replace=False), device=dev)
    diag = dict(px=None, py=None, ke=0.5 * (speed ** 2).mean(), F=F, F_grad=Fg, umax=speed.max(), c0=None,
                qmax=torch.sqrt(2 * (f["qxx"] ** 2 + f["qxy"] ** 2)).max())
    return dict(diag=diag, spectrum=E, slope=None, defects=(None, None), cx=corr[0, :M // 2 + 1] / corr[0, 0],
                cy=corr[:M // 2 + 1, 0] / corr[0, 0], lx=None, ly=None, track=(f["x"][ids], f["y"][ids]),
                mixing=(None, None))


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] == "train":
        return _exact_train(case, seed, dev)
    if case["kind"] == "diagnostics":
        return _exact_diagnostics(case, seed, dev)
    if case["kind"] == "ensemble":
        if sum(s * s for s, _, _ in _replicas(case)) * case["steps"] > 3e8:
            return None
        got = []
        for r, (s, z, k) in enumerate(_replicas(case)):
            box = _Box64(_params(s, z, k), _fields(s, 1000 * seed + r, start="lattice"), dev)
            for _ in range(case["steps"]):
                box.step(DT)
            got.append(box.state())
        return {k: torch.cat([g[k] for g in got]) for k in got[0]}
    side = case["side"]
    if case["kind"] == "box":
        if side * side * case["steps"] > 3e8:   # about 20 seconds
            return None
        box = _Box64(_params(side, **{k: case[k] for k in PHYS}),
                     _fields(side, seed, case["start"], case["angles"], q3d=case["q3d"]), dev)
        for _ in range(case["steps"]):
            box.step(DT)
        return box.state()
    if side * side * case["macro"] > 3e8:
        return None
    box = _Box64(_params(side), _fields(side, seed), dev)
    w, norm = (torch.tensor(v, dtype=torch.float64, device=dev) for v in _network(seed))
    worst = 0.0
    for _ in range(case["macro"]):
        X = box.step(case["mult"] * DT)
        y = _mlp64(w, (X - norm[:12]) / norm[12:24])[2]
        worst = max(worst, float(y.norm(dim=1).max()))
        c = y * norm[29:] + norm[24:29]
        box.f["qxx"], box.f["qxy"] = box.f["qxx"] + 0.5 * (c[:, 0] - c[:, 2]), box.f["qxy"] + c[:, 1]
        box.f["ux"], box.f["uy"] = box.f["ux"] + c[:, 3], box.f["uy"] + c[:, 4]
    return dict(box.state(), fallbacks=None, worst=worst)
