"""Timed cases of the Coordinate Condensation library on one MI355X.

Each case is one pass through the public entry points as a simulation or a
training loop calls them.  The sizes are the repository's own: the 17 x 17
square of the resolution sweep, the struck 41 x 2 x 2 rod, the 21 x 6 x 6 bar,
the batch of 6 x 6 x 6 .. 41 x 11 x 11 bars, the 81 x 21 x 21 beam, and the
warm-start network's batches.

A step is taken from a saved state (displaced and moving smoothly, as in the
middle of a trajectory) that every pass restores first, as a rollout that is
replayed from a checkpoint does; so every pass does the same work.  With
float32 local arithmetic ("fp32") the positions, velocities and directions
are returned as float32, the precision a program keeps of such a solve; with
"fp64" they are returned as the library holds them.
"""
import math
import random

import numpy as np
import torch

import paper_2510_12053_amd.ccgpu as cg

DEV = "cuda:0"
GRAV = 9.81
DT = 1.0 / 60
STEP_ITERS = 5          # iterations of a step to 1e-6 that work() counts


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def listed():
    return [
        # one quasistatic solve of a small 2D square, as in the mesh-resolution sweep: launch latency
        dict(name="square17_stretch_fp64", kind="square", n=17, E=1e5, nu=0.4, prec="fp64"),
        # one implicit step of one free rod struck at its end, the smallest 3D mesh (no held vertex)
        dict(name="rod41_step_fp64", kind="step", nx=41, ny=2, nz=2, logE=3.0, nu=0.3, h=0.025, face=-1,
             prec="fp64", corot=False, radius=0, material="snh", gs=False),
        # interactive stepping of a single bar in float64, one call per step
        dict(name="bar21_step_fp64", kind="step", nx=21, ny=6, nz=6, logE=5.0, nu=0.45, h=0.2, face=0,
             prec="fp64", corot=False, radius=0, material="snh", gs=False),
        # the four bars of the float64 stiffness comparison, stepped as one batch
        dict(name="bars4_step_fp64", kind="batch", bars=4, nx=21, ny=6, nz=6, draw=0, prec="fp64",
             corot=False, gs=False, steps=1, warm=False),
        # one sweep's directions on a ragged bar (a user's own outer solver or a diagnostic)
        dict(name="bar29x9x7_directions_fp32", kind="directions", nx=29, ny=9, nz=7, logE=6.0, nu=0.4, h=0.1,
             face=0, prec="fp32", corot=True, radius=0),
        # the basis rebuilt from the current state before a quasistatic load step, Fixed Corotational
        dict(name="cantilever21_restart_fp64", kind="restart", nx=21, ny=6, nz=6, logE=7.0, nu=0.45, h=0.2,
             face=0, prec="fp64", corot=False, material="fcr"),
        # the benchmark's batch: 64 uneven bars, exact corotated bases, one step to 1e-6
        dict(name="bars64_step_fp32", kind="batch", bars=64, nx=0, ny=0, nz=0, draw=20251012, prec="fp32",
             corot=True, gs=False, steps=1, warm=False),
        # a short rollout of a smaller batch with the learned warm start
        dict(name="bars16_rollout_warm_fp32", kind="batch", bars=16, nx=0, ny=0, nz=0, draw=20251100,
             prec="fp32", corot=True, gs=False, steps=4, warm=True),
        # the same solver with coloured Gauss-Seidel sweeps
        dict(name="bars16_gs_step_fp32", kind="batch", bars=16, nx=0, ny=0, nz=0, draw=20251200, prec="fp32",
             corot=True, gs=True, steps=1, warm=False),
        # the large twisted beam with its exact basis, one step (the largest case)
        dict(name="beam81_twist_fp32", kind="step", nx=81, ny=21, nz=21, logE=7.0, nu=0.45, h=0.05, face=6,
             prec="fp32", corot=True, radius=0, material="snh", gs=False),
        # the same beam, soft, with a one-ring patch basis: the sparse sweep
        dict(name="beam81_patch_step_fp32", kind="step", nx=81, ny=21, nz=21, logE=3.0, nu=0.45, h=0.05, face=6,
             prec="fp32", corot=False, radius=1, material="snh", gs=False),
        # the warm-start network: one training gradient, and one pass over the vertices of a batch
        dict(name="network_gradient_and_forward", kind="network", rows=4096, infer=105438),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(["square", "step", "step", "step", "batch", "batch", "batch", "directions", "directions",
                       "restart", "network"])
    if kind == "square":
        return dict(kind=kind, n=rng.randint(5, 29), E=float(10.0 ** rng.uniform(4, 6)), nu=rng.uniform(0.3, 0.45),
                    prec="fp64")
    if kind == "network":
        return dict(kind=kind, rows=_logint(rng, 256, 16384), infer=_logint(rng, 1000, 400000))
    prec = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "batch":
        return dict(kind=kind, bars=_logint(rng, 2, 48 if prec == "fp32" else 12), nx=0, ny=0, nz=0,
                    draw=rng.randint(1, 10 ** 6), prec=prec, corot=rng.random() < 0.7, gs=rng.random() < 0.2,
                    steps=rng.choice([1, 1, 2]), warm=rng.random() < 0.25)
    # bars from a few vertices across to thick ones; float64 bases are kept for the smaller ones
    while True:
        c = dict(kind=kind, nx=_logint(rng, 6, 61), ny=_logint(rng, 3, 21), nz=_logint(rng, 3, 21))
        n = c["nx"] * c["ny"] * c["nz"]
        if n <= (16000 if prec == "fp32" and kind != "restart" else 2600) and n >= 54:
            break
    c.update(logE=rng.uniform(4.5, 7.0), nu=rng.uniform(0.3, 0.48), h=0.1, face=rng.randint(0, 6), prec=prec)
    c["corot"] = rng.random() < 0.6
    if kind == "step":
        c.update(radius=0, material=rng.choice(["snh", "snh", "fcr"]), gs=rng.random() < 0.15)
        if rng.random() < 0.25:      # patch bases serve soft materials
            c.update(radius=rng.randint(1, 2), logE=rng.uniform(3.0, 3.6), corot=False, gs=False, face=6)
    elif kind == "directions":
        c.update(radius=rng.choice([0, 0, 0, 1, 2]))
    else:
        c.update(nx=min(c["nx"], 24), corot=True, material=rng.choice(["snh", "fcr"]), face=0,
                 logE=rng.uniform(6.0, 7.0))
    return c


# --------------------------------------------------------------------------
# inputs: structured grids, seeded smooth states
# --------------------------------------------------------------------------

def _grid3(nx, ny, nz, h):
    k, j, i = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    X = np.stack([i.ravel(), j.ravel(), k.ravel()], axis=1) * float(h)
    cell = np.stack([a.ravel() for a in np.meshgrid(np.arange(nx - 1), np.arange(ny - 1), np.arange(nz - 1),
                                                    indexing="ij")], axis=1)
    tets = []
    for p in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)):
        at, path = cell.copy(), [cell.copy()]
        for ax in p:
            at = at.copy()
            at[:, ax] += 1
            path.append(at)
        ids = [q[:, 0] + nx * (q[:, 1] + ny * q[:, 2]) for q in path]
        if p in ((0, 2, 1), (1, 0, 2), (2, 1, 0)):
            ids[2], ids[3] = ids[3], ids[2]
        tets.append(np.stack(ids, axis=1))
    return X, np.stack(tets, axis=1).reshape(-1, 4).astype(np.int32)


def _grid2(n):
    j, i = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
    X = np.stack([i.ravel(), j.ravel()], axis=1) / float(n - 1)
    cj, ci = np.meshgrid(np.arange(n - 1), np.arange(n - 1), indexing="ij")
    a = (ci + n * cj).ravel()
    tris = np.stack([np.stack([a, a + 1, a + n + 1], 1), np.stack([a, a + n + 1, a + n], 1)], 1)
    return X, tris.reshape(-1, 3).astype(np.int32)


def _unit(rng):
    v = rng.normal(size=3)
    return v / np.linalg.norm(v)


def _bar(c, rng, quasistatic=False):
    """One bar: mesh, material, and a smooth state drawn from rng.  face 0..5 holds one face, 6 holds both
    ends along x (the far one turning), -1 none."""
    nx, ny, nz, h, face = c["nx"], c["ny"], c["nz"], c["h"], c["face"]
    X, el = _grid3(nx, ny, nz, h)
    L = np.array([nx - 1, ny - 1, nz - 1]) * h
    s = X / L
    bc, fixed = X.copy(), np.zeros(len(X), bool)
    g = GRAV * _unit(rng) * (1.0 if not quasistatic else 0.05)   # quasistatic: one load step of twenty
    amp, speed = (0.02 * L.min(), 0.3) if not quasistatic else (0.001 * L.min(), 0.0)
    if face == -1:
        ramp = np.ones(len(X))
        v = np.zeros_like(X)
        v[s[:, 0] == 1.0, 0] = -0.1 * rng.uniform(0.5, 1.5)
        u, g = np.zeros_like(X), np.zeros(3)
    else:
        if face == 6:
            a, b = s[:, 0] == 0.0, s[:, 0] == 1.0
            fixed = a | b
            t = np.pi / 60 * rng.uniform(0.7, 1.3)
            y, z = X[b, 1] - L[1] / 2, X[b, 2] - L[2] / 2
            bc[b, 1] = L[1] / 2 + np.cos(t) * y - np.sin(t) * z
            bc[b, 2] = L[2] / 2 + np.sin(t) * y + np.cos(t) * z
            ramp, g, speed = 4 * s[:, 0] * (1 - s[:, 0]), np.zeros(3), 0.1
        else:
            r = s[:, face // 2] if face % 2 == 0 else 1 - s[:, face // 2]
            fixed, ramp = r == 0.0, r * r
        wave = sum(np.sin(np.pi * (k + 1) * s @ rng.uniform(0.2, 1.0, 3))[:, None] * rng.normal(size=3) / (k + 1)
                   for k in range(2))
        u = amp * ramp[:, None] * (_unit(rng) + 0.3 * wave)
        v = speed * ramp[:, None] * (_unit(rng) + 0.3 * wave)
    return dict(X=X, el=el, fixed=fixed, E=10.0 ** c["logE"], nu=c["nu"], g=g, x=X + u, v=v, bc=bc, dim=3,
                dt=1.0 if quasistatic else DT, quasi=quasistatic, fcr=c.get("material") == "fcr")


def _scenes(case, seed):
    """The bodies of a case with their states."""
    rng = np.random.default_rng([int(seed) & 0xffffffff, 77])
    if case["kind"] == "square":
        X, el = _grid2(case["n"])
        left, right = X[:, 0] == 0.0, X[:, 0] == 1.0
        bc = X.copy()
        bc[right, 0] += 0.5 * rng.uniform(0.9, 1.1)
        x = X + 0.02 / (case["n"] - 1) * rng.normal(size=X.shape)
        x[left | right] = bc[left | right]
        return [dict(X=X, el=el, fixed=left | right, E=case["E"], nu=case["nu"], g=np.zeros(3), x=x,
                     v=np.zeros_like(X), bc=bc, dim=2, dt=1.0, quasi=True, fcr=False)]
    if case["kind"] == "batch":
        shape, out = random.Random(case["draw"]), []
        for b in range(case["bars"]):
            c = dict(nx=case["nx"] or shape.randint(6, 41), ny=case["ny"] or shape.randint(6, 11),
                     nz=case["nz"] or shape.randint(6, 11), h=0.2 if case["nx"] else 0.1,
                     logE=4.0 + b if case["nx"] else shape.uniform(4, 7), nu=0.45 if case["nx"] else shape.uniform(0.3, 0.48),
                     face=0 if case["nx"] else shape.randint(0, 5))
            out.append(_bar(c, rng))
        return out
    return [_bar(case, rng, quasistatic=case["kind"] == "restart")]


def _network(seed):
    """Initial parameters of the 32-64-64-16 network (16 inputs and 3 outputs used), packed."""
    r = np.random.default_rng([int(seed) & 0xffffffff, 5])
    W1, W3 = np.zeros((32, 64)), np.zeros((64, 16))
    W1[:16] = r.normal(size=(16, 64)) / 4
    W2 = r.normal(size=(64, 64)) / 8
    W3[:, :3] = 0.1 * r.normal(size=(64, 3)) / 8
    return np.concatenate([W1.ravel(), np.zeros(64), W2.ravel(), np.zeros(64), W3.ravel(), np.zeros(16)])


def _rows(case, seed):
    r = np.random.default_rng([int(seed) & 0xffffffff, 6])
    X = r.normal(size=(case["rows"], 16)).astype(np.float32)
    T = (0.05 * r.normal(size=(case["rows"], 3))).astype(np.float32)
    idx = r.permutation(case["rows"]).astype(np.int32)
    return X, T, idx


def _rows_infer(case, seed):
    r = np.random.default_rng([int(seed) & 0xffffffff, 8])
    return r.normal(size=(case["infer"], 16)).astype(np.float32)


# --------------------------------------------------------------------------
# what a program has in hand, and one pass
# --------------------------------------------------------------------------

def prepare(case, seed):
    stream = torch.cuda.Stream(device=DEV)
    st = dict(case=case, stream=stream)
    st["ctx"] = ctx = cg.cc_create(0, stream)
    if case["kind"] == "network":
        X, T, idx = _rows(case, seed)
        cg.cc_mlp_set(ctx, _network(seed))
        st.update(X=torch.tensor(X, device=DEV), T=torch.tensor(T, device=DEV), idx=torch.tensor(idx, device=DEV),
                  Xi=torch.tensor(_rows_infer(case, seed), device=DEV))
        torch.cuda.synchronize()
        return st
    sc = _scenes(case, seed)
    # positions and velocities of all bodies in one buffer, each body a view
    state0 = torch.tensor(np.stack([np.concatenate([s[k] for s in sc]) for k in ("x", "v")]), device=DEV)
    state = state0.clone()
    off = np.cumsum([0] + [len(s["X"]) for s in sc])
    st.update(state0=state0, state=state, dt=sc[0]["dt"], g=np.stack([s["g"] for s in sc]),
              xs=[state[0, a:b] for a, b in zip(off, off[1:])], vs=[state[1, a:b] for a, b in zip(off, off[1:])],
              bcs=[torch.tensor(s["bc"], device=DEV) for s in sc], ids=[])
    for s in sc:
        mid = cg.cc_mesh_upload(ctx, s["X"], s["el"], s["fixed"], s["E"], s["nu"], 1000.0)
        cg.cc_mesh_set_material(ctx, mid, cg.MATERIAL_FCR if s["fcr"] else cg.MATERIAL_SNH)
        if case["kind"] != "restart":
            cg.cc_subspace_build(ctx, mid, case.get("radius", 0), s["dt"], s["quasi"])
        st["ids"].append(mid)
    if case["kind"] == "directions":
        st["xt"] = st["xs"][0] + DT * st["vs"][0]
    if case.get("warm"):
        cg.cc_mlp_set(ctx, _network(seed))
    st["par"] = cg.cc_params_default(
        method=cg.METHOD_CC, sweep=cg.SWEEP_COLORED_GS if case.get("gs") else cg.SWEEP_JACOBI,
        precision=cg.FP64 if case["prec"] == "fp64" else cg.FP32_MIXED, line_search=int(case["kind"] != "square"),
        max_iters=500 if case["kind"] == "square" else 200, quasistatic=int(sc[0]["quasi"]), gravity=sc[0]["g"],
        warm_start=int(bool(case.get("warm"))), corotate=int(bool(case.get("corot"))))
    torch.cuda.synchronize()
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    with torch.cuda.stream(st["stream"]):
        if case["kind"] == "network":
            grad, loss = cg.cc_mlp_gradient(ctx, st["X"], st["T"], st["idx"])
            return {"grad": grad, "forward": cg.cc_mlp_forward(ctx, st["Xi"])}
        if case["kind"] == "directions":
            e, g, dx = cg.cc_probe_sweep(ctx, st["ids"][0], st["xs"][0], st["xt"], DT, st["par"])
            return {"energy": e, "g": g, "dx": dx if case["prec"] == "fp64" else dx.float()}
        st["state"].copy_(st["state0"])
        if case["kind"] == "batch":
            for _ in range(case["steps"]):
                cg.cc_step_batch(ctx, st["ids"], st["xs"], st["vs"], st["bcs"], st["dt"], st["par"], 1e-6,
                                 gravity=st["g"])
        else:
            if case["kind"] == "restart":
                cg.cc_subspace_build_at(ctx, st["ids"][0], st["xs"][0], 0, st["dt"], True)
            tol = 1e-4 if case["kind"] == "square" else 1e-6
            cg.cc_step(ctx, st["ids"][0], st["xs"][0], st["vs"][0], st["bcs"][0], st["dt"], st["par"], tol)
        out = st["state"].clone() if case["prec"] == "fp64" else st["state"].float()
        # quasistatic: positions only
        return {"x": out[0]} if case["kind"] in ("square", "restart") else {"x": out[0], "v": out[1]}


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def _sizes(nx, ny, nz, face):
    n = nx * ny * nz
    dims = (nx, ny, nz)
    held = 0 if face == -1 else 2 * ny * nz if face == 6 else n // dims[face // 2]
    return n, n - held, 6 * (nx - 1) * (ny - 1) * (nz - 1)


def _iteration(n, nf, m, d, S, radius):
    """Bytes and flops of one Jacobi iteration: the basis and the element data read once, positions in and
    out; the condensation's block products (half of H by symmetry, about 8 upper blocks a vertex in 3D, 4 in
    2D), projected element Hessians and gradients."""
    up = 8 if d == 3 else 4
    supp = nf if radius == 0 else (14 if radius == 1 else 60)
    b = nf * supp * d * d * S + m * (4 * (d + 1) + d * d * (S + 8) + S + 8) + 6 * n * d * 8
    f = nf * supp * (2.0 * d ** 3 * (up + 1) + 2 * d * d) + m * (3400.0 if d == 3 else 500.0)
    return b, f


def work(case):
    if case["kind"] == "network":
        per = 2.0 * (16 * 64 + 64 * 64 + 64 * 3)
        return {"bytes": case["rows"] * 80 + 7312 * 8 + case["infer"] * 76,
                "flops": per * (3 * case["rows"] + case["infer"])}
    S, d, it, b, f = (8 if case["prec"] == "fp64" else 4), 3, STEP_ITERS, 0.0, 0.0
    if case["kind"] == "square":
        n = case["n"] ** 2
        b, f = _iteration(n, n - 2 * case["n"], 2 * (case["n"] - 1) ** 2, 2, S, 0)
        return {"bytes": it * b, "flops": it * f}
    if case["kind"] == "batch":
        shape = random.Random(case["draw"])
        for _ in range(case["bars"]):
            if case["nx"]:
                sz = _sizes(case["nx"], case["ny"], case["nz"], 0)
            else:
                nx, ny, nz = shape.randint(6, 41), shape.randint(6, 11), shape.randint(6, 11)
                shape.uniform(4, 7), shape.uniform(0.3, 0.48)
                sz = _sizes(nx, ny, nz, shape.randint(0, 5))
            bb, ff = _iteration(*sz, d, S, 0)
            b, f = b + bb, f + ff
        it *= case["steps"]
        return {"bytes": it * b, "flops": it * f}
    n, nf, m = _sizes(case["nx"], case["ny"], case["nz"], case["face"])
    b, f = _iteration(n, nf, m, d, S, case.get("radius", 0))
    if case["kind"] == "directions":
        it = 1
    if case["kind"] == "restart":       # the basis written once more, its columns by a block-tridiagonal solve
        lev = max(768, 3 * case["ny"] * case["nz"])
        return {"bytes": it * b + nf * nf * 36, "flops": it * f + 8.0 * (3 * nf) ** 2 * lev}
    return {"bytes": it * b, "flops": it * f}


# --------------------------------------------------------------------------
# the same values in 64 bits, in plain torch
# --------------------------------------------------------------------------

class _Bodies:
    """All bodies of a case as one system, float64."""

    def __init__(self, sc):
        self.d = d = sc[0]["dim"]
        n = np.cumsum([0] + [len(s["X"]) for s in sc])
        t = lambda a, dt=torch.float64: torch.tensor(np.ascontiguousarray(a), dtype=dt, device=DEV)  # noqa: E731
        cat = lambda f: np.concatenate([f(s) for s in sc])  # noqa: E731
        self.X, self.x, self.v, self.bc = (t(cat(lambda s, k=k: s[k])) for k in ("X", "x", "v", "bc"))
        self.el = t(np.concatenate([s["el"] + o for s, o in zip(sc, n)]), torch.int64)
        self.fixed = t(cat(lambda s: s["fixed"]), torch.bool)
        per = lambda f: t(np.concatenate([np.full(len(s["el"]), f(s)) for s in sc]))  # noqa: E731
        self.mu = per(lambda s: s["E"] / (2 * (1 + s["nu"])))
        lamL = per(lambda s: s["E"] * s["nu"] / ((1 + s["nu"]) * (1 - 2 * s["nu"])))
        self.fcr, self.quasi, self.h = sc[0]["fcr"], sc[0]["quasi"], sc[0]["dt"]
        self.lam = lamL if self.fcr else lamL + self.mu
        self.grav = t(np.concatenate([np.broadcast_to(s["g"][:d], s["X"].shape) for s in sc]))
        D = (self.X[self.el[:, 1:]] - self.X[self.el[:, :1]]).transpose(1, 2)
        self.vol = torch.linalg.det(D) / math.factorial(d)
        b = torch.linalg.inv(D)
        self.beta = torch.cat([-b.sum(1, keepdim=True), b], 1)
        self.mass = torch.zeros(len(self.X), dtype=torch.float64, device=DEV)
        self.mass.index_add_(0, self.el.reshape(-1), (1000.0 * self.vol / (d + 1)).repeat_interleave(d + 1))
        self.s = 1.0 if self.quasi else self.h ** 2
        self.w = 0.0 if self.quasi else 1.0
        self.free = (~self.fixed).nonzero().reshape(-1)
        dof = torch.full((len(self.X),), -1, dtype=torch.int64, device=DEV)
        dof[self.free] = torch.arange(len(self.free), device=DEV)
        self.rank = dof

    def F(self, x):
        return torch.einsum("eai,eaj->eij", x[self.el], self.beta)

    def cof(self, F):
        if self.d == 2:
            return torch.stack([torch.stack([F[:, 1, 1], -F[:, 1, 0]], -1), torch.stack([-F[:, 0, 1], F[:, 0, 0]], -1)], 1)
        return torch.stack([torch.linalg.cross(F[:, 1], F[:, 2], dim=-1), torch.linalg.cross(F[:, 2], F[:, 0], dim=-1),
                            torch.linalg.cross(F[:, 0], F[:, 1], dim=-1)], 1)

    def grad(self, x, xt):
        F = self.F(x)
        J = torch.linalg.det(F)
        mu, lam = self.mu[:, None, None], self.lam[:, None, None]
        if self.fcr:
            U, _, V = torch.linalg.svd(F.cpu())
            P = 2 * mu * (F - (U @ V).to(DEV)) + lam * (J - 1)[:, None, None] * self.cof(F)
        else:
            P = mu * F + (lam * (J - 1)[:, None, None] - mu) * self.cof(F)
        fe = torch.einsum("eij,eaj->eai", P, self.beta) * self.vol[:, None, None]
        g = self.w * self.mass[:, None] * (x - xt) - self.s * self.mass[:, None] * self.grav
        g.index_add_(0, self.el.reshape(-1), self.s * fe.reshape(-1, self.d))
        return g[self.free]

    def energy(self, x, xt):
        F = self.F(x)
        J = torch.linalg.det(F)
        psi = self.mu / 2 * (F.square().sum((1, 2)) - self.d) - self.mu * (J - 1) + self.lam / 2 * (J - 1) ** 2
        fr, m = self.free, self.mass[self.free]
        return (self.s * (self.vol * psi).sum() + self.w * 0.5 * (m * (x - xt)[fr].square().sum(1)).sum()
                - self.s * (m[:, None] * self.grav[fr] * x[fr]).sum())

    def element_hessians(self, x, project):
        """(m, (d+1) d, (d+1) d), of the stable neo-Hookean energy."""
        d, F = self.d, self.F(x)
        m = len(F)
        J, C = torch.linalg.det(F), self.cof(F).reshape(m, d * d)
        lam = self.lam if not self.fcr else self.lam + self.mu
        E = torch.zeros(d * d, m, d, d, dtype=torch.float64, device=DEV)
        for k in range(d * d):
            E[k, :, k // d, k % d] = 1
        if d == 2:
            dC = torch.stack([self.cof(E[k]).reshape(m, 4) for k in range(4)], 1)
        else:      # cof is quadratic: its derivative along E is half of cof(F + E) - cof(F - E)
            dC = torch.stack([(self.cof(F + E[k]) - self.cof(F - E[k])).reshape(m, 9) / 2 for k in range(9)], 1)
        A = (lam[:, None, None] * C[:, :, None] * C[:, None, :] + (lam * (J - 1) - self.mu)[:, None, None] * dC
             + self.mu[:, None, None] * torch.eye(d * d, dtype=torch.float64, device=DEV))
        if project:
            w, Q = torch.linalg.eigh(((A + A.transpose(1, 2)) / 2).cpu())
            A = ((Q * w.clamp(min=0)[:, None, :]) @ Q.transpose(1, 2)).to(DEV)
        H = torch.einsum("eijkl,eaj,ebl->eaibk", A.reshape(m, d, d, d, d), self.beta, self.beta)
        return (self.s * self.vol)[:, None, None] * H.reshape(m, (d + 1) * d, (d + 1) * d)

    def dofs(self):
        d = self.d
        r = self.rank[self.el]
        return torch.where(r[:, :, None] >= 0, r[:, :, None] * d + torch.arange(d, device=DEV), -1).reshape(len(self.el), -1)

    def dense(self, x, project):
        N = len(self.free) * self.d
        He, D = self.element_hessians(x, project), self.dofs()
        ok = (D[:, :, None] >= 0) & (D[:, None, :] >= 0)
        H = torch.zeros(N * N, dtype=torch.float64, device=DEV)
        H.index_add_(0, (D[:, :, None] * N + D[:, None, :])[ok], He[ok])
        H = H.reshape(N, N)
        H += torch.diag(self.w * self.mass[self.free].repeat_interleave(self.d))
        return H

    def solve(self, x, xt, g):
        """H^{-1} g at x by conjugate gradients with the inverse diagonal blocks (H not projected)."""
        d, D = self.d, self.dofs()
        He = self.element_hessians(x, False)
        nf = len(self.free)
        pad = torch.where(D >= 0, D, nf * d)
        mass = self.w * self.mass[self.free].repeat_interleave(d)
        B = torch.zeros(nf + 1, d, d, dtype=torch.float64, device=DEV)
        r = torch.where(self.rank[self.el] >= 0, self.rank[self.el], nf)
        for a in range(d + 1):
            B.index_add_(0, r[:, a], He[:, a * d:(a + 1) * d, a * d:(a + 1) * d])
        B = torch.linalg.inv(B[:nf] + torch.diag_embed(mass.reshape(nf, d)))
        N, m, k = nf * d, len(He), (d + 1) * d
        ij = torch.stack([pad[:, :, None].expand(m, k, k).reshape(-1), pad[:, None, :].expand(m, k, k).reshape(-1)])
        keep = (ij < N).all(0)
        H = torch.sparse_coo_tensor(ij[:, keep], He.reshape(-1)[keep], (N, N)).coalesce().to_sparse_csr()
        z = torch.zeros(N, dtype=torch.float64, device=DEV)
        res = g.reshape(-1).clone()
        pre = lambda v: (B @ v.reshape(nf, d, 1)).reshape(-1)  # noqa: E731
        y = pre(res)
        p, rho = y.clone(), res @ y
        stop = 1e-9 * float(res.norm())
        for k in range(4000):
            q = H @ p + mass * p
            a = rho / (p @ q)
            z += a * p
            res -= a * q
            if k % 25 == 24 and float(res.norm()) < stop:
                break
            y = pre(res)
            rho, old = res @ y, rho
            p = y + (rho / old) * p
        return z.reshape(nf, d)

    def step(self, x, v):
        """The minimiser of the step energy by Newton's method: (x, v) after the step; None if not reached."""
        xt = x.clone() if self.quasi else x + self.h * v
        xt[self.fixed] = self.bc[self.fixed]
        y = xt.clone()
        g = self.grad(y, xt)
        first = max(float(g.norm()), float((self.s * self.mass[:, None] * self.grav)[self.free].norm()))
        for it in range(30):
            if float(g.norm()) < 1e-11 * first:
                break
            if len(self.free) * self.d <= 6000 or self.fcr:
                if it < 4 or not self.fcr or it % 6 == 0:
                    L, bad = torch.linalg.cholesky_ex(self.dense(y, len(self.el) <= 20000))
                    if int(bad):
                        return None
                dy = torch.cholesky_solve(g.reshape(-1, 1), L).reshape(-1, self.d)
            else:
                dy = self.solve(y, xt, g)
            for k in range(6):           # shortened while the gradient grows tenfold
                new = y.clone()
                new[self.free] -= 0.5 ** k * dy
                gn = self.grad(new, xt)
                if float(gn.norm()) < 10 * float(g.norm()):
                    break
            y, g = new, gn
        if not float(g.norm()) < 1e-9 * first:
            return None
        return y, (y - x) / self.h

    def rotations(self, x):
        pairs = torch.cat([self.el[:, [a, b]] for a in range(self.d + 1) for b in range(self.d + 1) if a != b])
        pairs = torch.unique(pairs, dim=0)
        dx, dX = x[pairs[:, 1]] - x[pairs[:, 0]], self.X[pairs[:, 1]] - self.X[pairs[:, 0]]
        M = torch.zeros(len(x), self.d, self.d, dtype=torch.float64, device=DEV)
        M.index_add_(0, pairs[:, 0], dx[:, :, None] * dX[:, None, :])
        U, _, V = torch.linalg.svd(M[self.free].cpu())
        S = torch.ones(len(U), self.d, dtype=torch.float64)
        S[:, -1] = torch.linalg.det(U @ V).sign()
        return ((U * S[:, None, :]) @ V).to(DEV)

    def directions(self, x, xt, corot, radius):
        """One Jacobi sweep's directions with the rest basis."""
        d, nf = self.d, len(self.free)
        N = nf * d
        H0 = self.dense(self.X, True)
        if radius == 0:
            Z = torch.linalg.inv(H0.cpu()).to(DEV)
            at = torch.arange(nf, device=DEV)
            Zii = Z.reshape(nf, d, nf, d)[at, :, at, :]
            U = torch.einsum("nia,iab->nib", Z.reshape(N, nf, d), torch.linalg.inv(Zii.cpu()).to(DEV)).reshape(nf, d, nf, d)
            U[at, :, at, :] = 0
        else:
            near = (H0.reshape(nf, d, nf, d).abs().sum((1, 3)) > 0).double()
            r = self.rank[self.el]
            for a in range(d + 1):
                for b in range(d + 1):
                    ok = (r[:, a] >= 0) & (r[:, b] >= 0)
                    near[r[ok, a], r[ok, b]] = 1
            reach = near.clone()
            for _ in range(radius - 1):
                reach = ((reach @ near) > 0).double()
            U = torch.zeros(nf, d, nf, d, dtype=torch.float64)
            reach, Hc = reach.cpu().numpy() > 0, H0.cpu().numpy()
            for i in range(nf):
                c = np.nonzero(reach[i])[0]
                c = c[c != i]
                if len(c):
                    q = (c[:, None] * d + np.arange(d)).reshape(-1)
                    o = i * d + np.arange(d)
                    U[c, :, i, :] = torch.from_numpy(-np.linalg.solve(Hc[np.ix_(q, q)], Hc[np.ix_(q, o)]).reshape(len(c), d, d))
            U = U.to(DEV)
        if corot:
            U = torch.einsum("jab,jbic->jaic", self.rotations(x), U)
        U = U.reshape(N, N)
        H, g = self.dense(x, True), self.grad(x, xt)
        W = H @ U
        at = torch.arange(nf, device=DEV)
        A = W.reshape(nf, d, nf, d)[at, :, at, :]
        Ht = torch.stack([torch.stack([(U[:, a::d] * W[:, b::d]).sum(0) for b in range(d)], -1) for a in range(d)], 1)
        b = (U.T @ g.reshape(-1)).reshape(nf, d, 1)
        Y = torch.linalg.solve(Ht.cpu(), torch.cat([A.transpose(1, 2), b], 2).cpu()).to(DEV)
        Hii = H.reshape(nf, d, nf, d)[at, :, at, :]
        dx = torch.zeros_like(x)
        K, r = Hii - A @ Y[:, :, :d], g[:, :, None] - A @ Y[:, :, d:]
        dx[self.free] = -torch.linalg.solve(K.cpu(), r.cpu()).to(DEV)[:, :, 0]
        return dx


def exact(case, seed):
    if case["kind"] == "network":
        p = torch.tensor(_network(seed).astype(np.float32).astype(np.float64), device=DEV, requires_grad=True)
        def net(X):
            W1, b1, W2, b2, W3, b3 = torch.split(p, [2048, 64, 4096, 64, 1024, 16])
            h = torch.nn.functional.silu(X @ W1.reshape(32, 64)[:16] + b1)
            h = torch.nn.functional.silu(h @ W2.reshape(64, 64) + b2)
            return (h @ W3.reshape(64, 16) + b3)[:, :3]
        X, T, idx = _rows(case, seed)
        loss = (net(torch.tensor(X.astype(np.float64), device=DEV)) - torch.tensor(T.astype(np.float64), device=DEV)).square().mean()
        loss.backward()
        with torch.no_grad():
            return {"grad": p.grad, "forward": net(torch.tensor(_rows_infer(case, seed).astype(np.float64), device=DEV))}
    sc = _scenes(case, seed)
    b = _Bodies(sc)
    if case["kind"] == "directions":
        if len(b.free) > (2500 if case["radius"] == 0 else 1500):
            return None
        xt = b.x + DT * b.v
        g = torch.zeros_like(b.x)
        g[b.free] = b.grad(b.x, xt)
        return {"energy": float(b.energy(b.x, xt)), "g": g, "dx": b.directions(b.x, xt, case["corot"], case["radius"])}
    if case.get("material") == "fcr" and len(b.free) > 3000:
        return None
    x, v = b.x.clone(), b.v.clone()
    for _ in range(case.get("steps", 1)):
        try:
            r = b.step(x, v)
        except torch.linalg.LinAlgError:
            r = None
        if r is None:
            return None
        x, v = r
    return {"x": x} if case["kind"] in ("square", "restart") else {"x": x, "v": v}
