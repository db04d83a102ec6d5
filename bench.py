#!/usr/bin/env python
"""Benchmark of the Coordinate Condensation hot path on one MI355X.

Workload "batch64_bars" (the batched configuration of the scope): 64
seed-drawn tet bars of 6x6x6 to 41x11x11 vertices (116,527 vertices, 105,438
free, 522,624 tets; log10 E ~ U(4, 7), nu ~ U(0.3, 0.48), a random clamped
face, gravity 9.81 m/s^2 along a random direction, rho 1000, h = 1/60), each
with its exact perturbation basis (built on the GPU before timing).  One bench
step advances all 64 bars by one implicit Euler step, every bar solved by
Jacobi Coordinate Condensation (basis blocks rotated by the vertices'
neighbourhood rotations, as the bars swing and bend under gravity) with
backtracking line search to
rel|grad E| <= 1e-6, in FP32 local arithmetic with FP64 positions, gradients,
energies and reductions.  Three paths are timed on the same trajectory:

  plain CC        one bar after another, single-mesh launches, host-driven
                  iteration (one synchronisation per iteration);
  batched         all bars in every launch, graph replays, autotuned schedule;
  learned+batched the batched path started from the learned per-vertex
                  proposal (accepted only when it lowers the step energy).

The warm-start network is trained at start-up (untimed) on trajectories of
50 seeded 21x6x6 training bars generated by the solver itself.  Inputs are
resident on the GPU before timing.  The JSON line reports vertex updates per
second of the learned+batched path as `value`, the time to tolerance per step
of every path, the roofline position of the dominant kernel (HIP events on
the library stream, in an uncaptured rerun of the same launches) and the CPU
oracle timed on a bounded sample of the same bars.  Further sections time the
81x21x21 twisted beam to tolerance with its exact, corotated basis
(`beam81x21x21_twist`) and the four 21x6x6 bars of the stiffness sweep in
float64 (`bar21x6x6_Esweep_fp64`).
"""
import argparse
import gc
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = ("time-to-rel‖∇E‖≤1e-6 per step and vertex-updates/s; "
          "learned+batched vs plain CC")
HBM_PEAK_GBS = 8000.0
FP64_PEAK_TFLOPS = 78.6
FP32_PEAK_TFLOPS = 157.3          # published vector peak: counts packed FP32 (two FMAs per lane)
# the library is built without packed FP32 instructions, so its FP32 code
# issues at most one FMA per lane per clock: 256 CUs x 64 lanes x 2 flops x
# 2.4 GHz, the same figure as the FP64 vector peak
FP32_SCALAR_PEAK_TFLOPS = 78.6
FP32_MATRIX_PEAK_TFLOPS = 157.3   # published float32 matrix peak: the condensation's, unless a row count is forced
TOL = 1e-6
MAX_ITERS = 10000          # per step; the headline Jacobi solves never come near it
GS_MAX_ITERS = 200
TRAIN_SEEDS = range(1000, 1050)
TRAIN_STEPS = 10
E_SWEEP = (1e4, 1e5, 1e6, 1e7)
MASK = (1 << 6) - 1
T_START = time.perf_counter()


def log(msg):
    """Progress line on stderr (the JSON result alone goes to stdout)."""
    print(f"[bench {time.perf_counter() - T_START:7.1f} s] {msg}", file=sys.stderr, flush=True)


def block_pattern(s):
    """Row lengths (diagonal included) of the free-vertex block Hessian, by vertex id."""
    fixed = s.fixed.astype(bool)
    nbr = [set() for _ in range(s.n)]
    for e in s.elems:
        fr = [int(a) for a in e if not fixed[a]]
        for a in fr:
            nbr[a].update(fr)
    return np.array([len(nbr[i]) for i in range(s.n)])


def kernel_model(s, S):
    """Algorithmic bytes and flops of each kernel for one Jacobi iteration of
    one mesh with the exact basis (S: bytes of the local float type).

    Condensation (band kernel + finish): every basis row once (n_f^2 blocks,
    own block included), the upper blocks of H with their band positions
    once, the rows of H for A_i, g, and K, L, b out.  With n_up the number of
    blocks (j, k) with k at or after j, vertex i costs one d x d x d product
    per upper block (W_j) and one per row j (U_j^T W_j), plus U_j^T g_j and
    one product per block of its own row (A_i)."""
    d = s.X.shape[1]
    k, dd = d + 1, d * d
    nb = k * (k + 1) // 2
    rl = block_pattern(s)
    free = ~s.fixed.astype(bool)
    nf = int(free.sum())
    nnzb = int(rl[free].sum())
    nup = (nnzb + nf) // 2
    fma3 = 2.0 * d ** 3
    byts = {
        "cc_prep": nf * nf * dd * S + nup * (dd * S + 4) + nnzb * (dd * S + 4)
        + nf * (d * 8 + 2 * dd * S + d * 8),
        "elem_hess": s.m * (k * 4 + dd * S + S + k * d * 8 + nb * dd * S),
        "assemble": s.m * nb * dd * S + nnzb * dd * S + nup * dd * S,
        "gradient": s.m * (k * 4 + dd * 8 + 8) + s.n * d * 8 * 2 + nf * d * 8,
        "energy": s.m * (k * 4 + dd * 8 + 8) + s.n * d * 8 * 2,
    }
    flops = {
        "cc_prep": nf * (fma3 * nup + (fma3 + 2 * dd) * nf) + fma3 * nnzb,
        "elem_hess": s.m * 3.4e3,
        "assemble": nnzb * dd * 1.0,
        "gradient": 4 * s.m * 150.0,
        "energy": s.m * 100.0,
    }
    return byts, flops


def measured_traffic(summary, kernel=None):
    """HBM bytes of one condensation launch from the counter summary written
    by bench_counters.py, or None when the summary is missing, was taken on
    another version of the kernel source, or (kernel given) of another kernel."""
    import hashlib
    path = os.path.join(ROOT, "profiles", summary)
    src = os.path.join(ROOT, "paper_2510_12053_amd", "csrc", "cc_kernels.hip")
    if not os.path.exists(path):
        return None
    rec = None
    for line in open(path):
        if line.startswith("traffic_json: "):
            rec = json.loads(line[len("traffic_json: "):])
    with open(src, "rb") as f:
        h = hashlib.sha256(f.read()).hexdigest()[:16]
    if rec is None or rec.get("source_sha256_16") != h or kernel not in (None, rec.get("kernel")):
        return None
    return rec


def cpu_baseline(scenes, budget_s):
    """Time the oracle on a bounded sample of the bench bars: the smallest
    bars (whose exact bases the oracle builds in seconds) are stepped from
    t = 1, round-robin, until the solve time exceeds the budget."""
    from oracle import solvers as S
    from oracle.basis import exact_basis
    from oracle.fem import Problem
    from oracle.timestep import step
    try:
        from threadpoolctl import threadpool_info
        threads = max([t.get("num_threads", 1) for t in threadpool_info()] or [1])
    except Exception:  # pragma: no cover
        threads = 1
    order = np.argsort([int((~s.fixed.astype(bool)).sum()) for s in scenes])[:4]
    sample = [scenes[i] for i in order]
    prm = S.Params(method=S.CC, sweep=S.JACOBI, line_search=True, max_iters=200)
    probs = [Problem.from_scene(s) for s in sample]
    bases = [exact_basis(p) for p in probs]             # precompute, untimed
    states = [s.initial_state() for s in sample]
    upd, t_solve, nsteps, iters = 0, 0.0, 0, 0
    t = 0
    while t_solve < budget_s and t < 50:
        t += 1
        for k, s in enumerate(sample):
            x, v = states[k]
            t0 = time.perf_counter()
            x, v, res, _ = step(probs[k], x, v, s.targets(t), bases[k], prm, TOL)
            t_solve += time.perf_counter() - t0
            states[k] = (x, v)
            upd += res.iters * probs[k].free.size
            iters += res.iters
            nsteps += 1
    names = ", ".join(s.name for s in sample)
    return {"value": round(upd / t_solve, 1), "unit": "vertex-updates/s", "cores": int(threads),
            "kind": "oracle",
            "sample": f"{nsteps} bar-steps ({t} time steps of the four smallest bench bars, {names}; "
                      f"{iters} CC iterations; exact basis, Jacobi CC + line search to 1e-6, float64), "
                      f"{t_solve:.1f} s of oracle solve time; BLAS threads {threads}, "
                      f"host os.cpu_count()={os.cpu_count()}"}


class Workload:
    """Meshes of one scene list with their bases, and a state per path."""

    def __init__(self, cg, ctx, dev, scenes, precision, corotate=0, build=True):
        import torch
        self.cg, self.ctx, self.dev, self.scenes = cg, ctx, dev, scenes
        self.nf = [int((~s.fixed.astype(bool)).sum()) for s in scenes]
        self.mids = []
        t0 = time.perf_counter()
        for s in scenes:
            mid = cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho)
            if build:
                cg.cc_subspace_build(ctx, mid, 0, s.dt, False)      # exact basis, untimed
            self.mids.append(mid)
        torch.cuda.synchronize()
        self.build_s = time.perf_counter() - t0
        self.grav = np.stack([s.gravity for s in scenes])
        self.precision, self.corotate = precision, corotate
        self._bcs = {}

    sweep = 0
    max_iters = 10000

    def params(self, s, warm):
        return self.cg.cc_params_default(method=self.cg.METHOD_CC, sweep=self.sweep,
                                         precision=self.precision, line_search=1, max_iters=self.max_iters,
                                         gravity=s.gravity, warm_start=int(warm),
                                         corotate=self.corotate)

    def bcs(self, t):
        import torch
        if t not in self._bcs:
            self._bcs[t] = [torch.tensor(s.targets(t), dtype=torch.float64, device=self.dev)
                            for s in self.scenes]
        return self._bcs[t]

    def fresh_state(self):
        import torch
        xs = [torch.tensor(s.initial_state()[0], dtype=torch.float64, device=self.dev) for s in self.scenes]
        vs = [torch.tensor(s.initial_state()[1], dtype=torch.float64, device=self.dev) for s in self.scenes]
        return xs, vs

    def run_plain(self, st, t, rec, warm=False):
        cg = self.cg
        xs, vs = st
        for k, (s, mid) in enumerate(zip(self.scenes, self.mids)):
            t0 = time.perf_counter()
            code, it, rg = cg.cc_step(self.ctx, mid, xs[k], vs[k], self.bcs(t)[k], s.dt,
                                      self.params(s, warm), TOL)
            if rec is not None:
                rec.append((code, it, rg, (time.perf_counter() - t0) * 1e3, it * self.nf[k], 0, 0))

    def run_batch(self, st, t, rec, warm=False):
        cg = self.cg
        xs, vs = st
        t0 = time.perf_counter()
        _, its, rgs, sts = cg.cc_step_batch(self.ctx, self.mids, xs, vs, self.bcs(t), self.scenes[0].dt,
                                            self.params(self.scenes[0], warm), TOL, gravity=self.grav)
        ms = (time.perf_counter() - t0) * 1e3
        if rec is not None:
            coloured = self.sweep != cg.SWEEP_JACOBI
            for k, mid in enumerate(self.mids):
                info = cg.cc_step_info(self.ctx, mid) if (warm or coloured) else None
                acc = int(info["warm_accepted"]) if warm else 0
                sfb = int(info["sweep_fallbacks"]) if coloured else 0
                rec.append((int(sts[k]), int(its[k]), float(rgs[k]), ms, int(its[k]) * self.nf[k], acc, sfb))


def timed(cg, ctx, wl, runner, warmup, steps, warm=False, profile=False):
    """warmup untimed steps, then steps timed ones, from the rest state."""
    import torch
    st = wl.fresh_state()
    for t in range(1, warmup + 1):
        runner(st, t, None, warm)
    torch.cuda.synchronize()
    cg.cc_profile_enable(ctx, MASK if profile else 0)
    rec = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for t in range(warmup + 1, warmup + steps + 1):
        runner(st, t, rec, warm)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    kern = {cg.K_NAMES[k]: cg.cc_profile_read(ctx, k) for k in range(6)}
    cg.cc_profile_enable(ctx, 0)
    return rec, elapsed, kern


def summary(rec, elapsed, steps, nmesh, per_mesh_time):
    upd = sum(r[4] for r in rec)
    # time to tolerance of one step: the bars' own solves one after another
    # (plain) or the batch call (batched)
    if per_mesh_time:
        ttt = np.array([sum(r[3] for r in rec[i:i + nmesh]) for i in range(0, len(rec), nmesh)])
    else:
        ttt = np.array([rec[i][3] for i in range(0, len(rec), nmesh)])
    out = {"vertex_updates_per_s": round(upd / elapsed, 1),
           "ms_per_step": round(elapsed / steps * 1e3, 3),
           "time_to_tol_ms": {"median": round(float(np.median(ttt)), 3),
                              "p90": round(float(np.percentile(ttt, 90)), 3)},
           "iters_per_mesh_step": round(float(np.mean([r[1] for r in rec])), 2),
           "max_iters": int(max(r[1] for r in rec)),
           "not_ok": sum(1 for r in rec if r[0] != 0),
           "max_rel_grad": float(max(r[2] for r in rec))}
    if not per_mesh_time:
        out["warm_accepted"] = int(sum(1 for r in rec if r[5]))
        out["warm_network_taken"] = int(sum(1 for r in rec if r[5] == 1))
    return out


def roofline(wl, rec, kern, S, peak_f, dense_rows):
    """Dominant kernel class of the profiled launches against HBM and the
    arithmetic peak of the unit that does its products.  dense_rows: the
    tuning's rows per workgroup of the condensation (0: matrix cores in
    float32, on launches as large as these workloads')."""
    models = [kernel_model(s, S) for s in wl.scenes]
    its_mesh = [0] * len(wl.scenes)
    for k, r in enumerate(rec):
        its_mesh[k % len(wl.scenes)] += r[1]
    dom = max(kern, key=lambda k: kern[k][0])
    ms_tot, launches = kern[dom]
    secs = ms_tot * 1e-3
    alg = sum(i * m[0][dom] for i, m in zip(its_mesh, models))
    fl = sum(i * m[1][dom] for i, m in zip(its_mesh, models))
    gbs, tfl = alg / secs / 1e9, fl / secs / 1e12
    tile = S == 4 and dense_rows == 0
    if tile and dom == "cc_prep":
        peak_f = FP32_MATRIX_PEAK_TFLOPS
    hbm = {"achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": round(gbs / HBM_PEAK_GBS, 4)}
    alu = {"achieved": round(tfl, 3), "peak": peak_f, "unit": "TFLOP/s", "frac": round(tfl / peak_f, 4)}
    if peak_f == FP32_SCALAR_PEAK_TFLOPS and S == 4:
        alu["published_peak"] = FP32_PEAK_TFLOPS
        alu["frac_of_published_peak"] = round(tfl / FP32_PEAK_TFLOPS, 4)
    bound = "alu" if alu["frac"] >= hbm["frac"] else "hbm"
    roof = dict(alu if bound == "alu" else hbm)
    roof = {"bound": bound, **roof}
    prep = "kb_prep_tile" if tile else "kb_prep_band"
    roof.update({"kernel": prep + "+kb_dm_finish" if dom == "cc_prep" else "kb_" + dom,
                 "avg_launch_us": round(ms_tot / max(launches, 1) * 1e3, 2), "launches": launches,
                 "algorithmic_bytes_per_launch": round(alg / max(launches, 1)),
                 "flops_per_launch": round(fl / max(launches, 1)),
                 "hbm": hbm, "valu": alu,
                 "share_of_kernel_time": round(ms_tot / sum(v[0] for v in kern.values()), 3)})
    per_class = {}
    for name, (ms_k, n_k) in kern.items():
        if name not in models[0][0] or n_k == 0 or ms_k <= 0:
            continue
        sec_k = ms_k * 1e-3
        per_class[name] = {
            "us_per_launch": round(ms_k / n_k * 1e3, 2), "launches": n_k,
            "GBps_algorithmic": round(sum(i * m[0][name] for i, m in zip(its_mesh, models)) / sec_k / 1e9, 1),
            "TFLOPs": round(sum(i * m[1][name] for i, m in zip(its_mesh, models)) / sec_k / 1e12, 3)}
    return roof, per_class, dom


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--precision", choices=["fp32", "fp64"], default="fp32")
    ap.add_argument("--beam-steps", type=int, default=4)
    ap.add_argument("--no-beam", action="store_true")
    ap.add_argument("--no-esweep", action="store_true")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-budget", type=float, default=20.0)
    ap.add_argument("--retune", action="store_true", help="ignore the autotuner's cache")
    ap.add_argument("--train-epochs", type=int, default=40)
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only; --gpus {args.gpus} is not supported "
              "(this path is measured on one GPU; sharding across GPUs is a design, not built)",
              file=sys.stderr)
        sys.exit(2)
    if args.steps < 1 or args.warmup < 0:
        print("--steps must be >= 1 and --warmup >= 0", file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2510_12053_amd.ccgpu as cg
    from paper_2510_12053_amd import warmstart as W
    from ccscenes import batch_bars, mlp_init, tet_bar, twist_beam, warm_start_train_scene

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    stream = torch.cuda.Stream(device=dev)          # capturable stream for the batched graphs
    torch.cuda.set_stream(stream)
    ctx = cg.cc_create(0, stream)
    prec = cg.FP64 if args.precision == "fp64" else cg.FP32_MIXED
    S = 8 if prec == cg.FP64 else 4
    peak_f = FP64_PEAK_TFLOPS if prec == cg.FP64 else FP32_SCALAR_PEAK_TFLOPS

    # ---- untimed: warm-start network trained on solver-generated data ----
    log("generating warm-start training data")
    t0 = time.perf_counter()
    train_scenes = [warm_start_train_scene(sd) for sd in TRAIN_SEEDS]
    Xtr, Ttr, _ = W.generate(ctx, train_scenes, TRAIN_STEPS, dev, precision=prec)
    t_gen = time.perf_counter() - t0
    log(f"training the warm-start network on {Xtr.shape[0]} samples")
    losses, t_train = W.train(ctx, Xtr, Ttr, mlp_init(7), epochs=args.train_epochs, batch=4096, lr=2e-3)
    training = {"samples": int(Xtr.shape[0]), "episodes": len(train_scenes), "steps": TRAIN_STEPS,
                "generate_s": round(t_gen, 2), "train_s": round(t_train, 2), "epochs": args.train_epochs,
                "loss_first": round(losses[0], 5), "loss_last": round(losses[-1], 5)}
    del Xtr, Ttr
    torch.cuda.empty_cache()
    # everything alive now (torch, scenes, meshes) leaves the collector's
    # view, so a full collection inside a timed step stays short
    gc.collect()
    gc.freeze()

    # ---- headline: the 64-bar batch ----
    bars = batch_bars(64)
    log("building the exact bases of the 64 bars")
    wl = Workload(cg, ctx, dev, bars, prec, corotate=1)
    log(f"bases built in {wl.build_s:.1f} s; autotuning")
    from paper_2510_12053_amd import autotune
    xs0, vs0 = wl.fresh_state()
    tuning, tune_table = autotune.tune(ctx, wl.mids, xs0, vs0, [wl.bcs(1), wl.bcs(2)], bars[0].dt,
                                       wl.params(bars[0], False), TOL, wl.grav,
                                       sum(wl.nf), any_dense=True, any_sparse=False,
                                       use_cache=not args.retune)
    del xs0, vs0
    log(f"tuning: {tuning}")
    nb = len(bars)
    log("plain CC")
    rec_p, el_p, _ = timed(cg, ctx, wl, wl.run_plain, args.warmup, args.steps)
    log(f"plain CC: {el_p / args.steps * 1e3:.1f} ms per step; batched")
    rec_b, el_b, _ = timed(cg, ctx, wl, wl.run_batch, args.warmup, args.steps)
    log(f"batched: {el_b / args.steps * 1e3:.1f} ms per step; learned+batched")
    rec_l, el_l, _ = timed(cg, ctx, wl, wl.run_batch, args.warmup, args.steps, warm=True)
    log(f"learned+batched: {el_l / args.steps * 1e3:.1f} ms per step")
    # the coloured Gauss-Seidel sweep on the same bars and trajectory (one
    # colour at a time, Hessians refreshed per colour on the elements the
    # previous colour moved), batched, beside Jacobi.  With the exact basis
    # every colour's move is a whole Newton-like step taken while the other
    # colours stand still, and on stiff bars the sweep's full step can raise
    # E; such an iteration takes the Jacobi sweep instead (as the oracle
    # does), and the section reports how many iterations did.
    log("coloured Gauss-Seidel, batched")
    wl.sweep, wl.max_iters = cg.SWEEP_COLORED_GS, GS_MAX_ITERS
    rec_g, el_g, _ = timed(cg, ctx, wl, wl.run_batch, args.warmup, args.steps)
    wl.sweep, wl.max_iters = cg.SWEEP_JACOBI, MAX_ITERS
    gs_batched = summary(rec_g, el_g, args.steps, nb, False)
    gs_batched["max_iters_cap"] = GS_MAX_ITERS
    gs_batched["jacobi_fallback_iters"] = int(sum(r[6] for r in rec_g))
    # the learned+batched launches again, uncaptured, with HIP events around
    # every kernel class: per-kernel durations for the roofline (last of the
    # bar sections, so that a kernel trace finds its dispatches just before
    # the beam's)
    log("profiled rerun")
    rec_k, _, kern_k = timed(cg, ctx, wl, wl.run_batch, args.warmup, args.steps, warm=True, profile=True)
    plain = summary(rec_p, el_p, args.steps, nb, True)
    batched = summary(rec_b, el_b, args.steps, nb, False)
    learned = summary(rec_l, el_l, args.steps, nb, False)
    roof, kernel_roofline, dom = roofline(wl, rec_k, kern_k, S, peak_f, tuning["dense_rows"])
    prep = roof["kernel"].split("+")[0]
    tr = (measured_traffic(f"traffic_{prep}_batch64_{args.precision}.md", roof["kernel"])
          if dom == "cc_prep" else None)
    # counter bytes per bar-iteration times the bar-iterations of a mean launch
    if tr is not None:
        per_it = (tr["fetch_bytes_per_launch"] + tr["write_bytes_per_launch"]) / tr["mesh_iters_per_launch"]
        mesh_iters = sum(r[1] for r in rec_k)
        roof["traffic"] = round(per_it * mesh_iters / max(roof["launches"], 1))
    else:
        roof["traffic"] = None
    value = learned["vertex_updates_per_s"]
    headline_build_s = round(wl.build_s, 2)
    del wl
    gc.collect()
    torch.cuda.empty_cache()

    out = {
        "metric": METRIC,
        "value": value,
        "unit": "vertex-updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": learned["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if prec == cg.FP64 else "f32+f64",
        "data": "synthetic",
        "config": {"workload": "batch64_bars", "bars": nb, "verts": int(sum(s.n for s in bars)),
                   "free_verts": int(sum(int((~s.fixed.astype(bool)).sum()) for s in bars)),
                   "tets": int(sum(s.m for s in bars)), "basis": "exact", "method": "cc",
                   "sweep": "jacobi", "line_search": True, "corotated": True, "tol": TOL,
                   "dt": bars[0].dt,
                   "precision": args.precision, "path": "learned+batched", "tuning": tuning,
                   "basis_build_s": headline_build_s},
        "learned_batched": learned,
        "batched": batched,
        "plain_cc": plain,
        "coloured_gs_batched": gs_batched,
        "speedup_time_to_tol_learned_batched_vs_plain": round(plain["ms_per_step"] / learned["ms_per_step"], 3),
        "speedup_time_to_tol_batched_vs_plain": round(plain["ms_per_step"] / batched["ms_per_step"], 3),
        "training": training,
        "autotune": tune_table,
        "kernel_ms_learned_batched_uncaptured": {k: round(v[0], 3) for k, v in kern_k.items()},
        "roofline": roof,
        "kernel_roofline": kernel_roofline,
    }

    # ---- the 81x21x21 twisted beam, exact corotated basis, to tolerance ----
    if not args.no_beam:
        beam = twist_beam()
        log("beam: building the exact basis")
        bw = Workload(cg, ctx, dev, [beam], cg.FP32_MIXED, corotate=1)
        log(f"beam: basis built in {bw.build_s:.1f} s")
        nsteps = min(args.beam_steps, beam.n_steps)
        res = {"workload": "beam81x21x21_twist", "verts": beam.n, "tets": beam.m,
               "free_verts": bw.nf[0], "basis": "exact, corotated", "precision": "fp32",
               "basis_build_s": round(bw.build_s, 2), "steps": nsteps}
        for name, warm in (("batched", False), ("learned_batched", True)):
            log(f"beam: {name}")
            rec, el, _ = timed(cg, ctx, bw, bw.run_batch, 0, nsteps, warm=warm)
            res[name] = summary(rec, el, nsteps, 1, False)
            res[name]["iters_per_step"] = [r[1] for r in rec]
        rec, _, kern = timed(cg, ctx, bw, bw.run_batch, 0, min(nsteps, 2), profile=True)
        broof, bcls, _ = roofline(bw, rec, kern, 4, FP32_SCALAR_PEAK_TFLOPS, tuning["dense_rows"])
        res["roofline"] = broof
        res["kernel_roofline"] = bcls
        out["beam81x21x21_twist"] = res
        del bw
        gc.collect()
        torch.cuda.empty_cache()

    # ---- the four 21x6x6 bars of the stiffness sweep in float64 ----
    if not args.no_esweep:
        log("float64 stiffness sweep bars")
        es = [tet_bar(E=E) for E in E_SWEEP]
        ew = Workload(cg, ctx, dev, es, cg.FP64)
        n_es = min(args.steps + args.warmup, 10)
        res = {"workload": "bar21x6x6_Esweep", "E": list(E_SWEEP), "precision": "fp64", "steps": n_es}
        for name, runner, per in (("plain_cc", ew.run_plain, True), ("batched", ew.run_batch, False)):
            rec, el, _ = timed(cg, ctx, ew, runner, 0, n_es)
            res[name] = summary(rec, el, n_es, len(es), per)
        out["bar21x6x6_Esweep_fp64"] = res
        del ew

    if not args.no_cpu_baseline:
        log("CPU oracle baseline")
        out["cpu_baseline"] = cpu_baseline(bars, args.cpu_budget)
    log("done")
    print(json.dumps(out), flush=True)
    cg.cc_destroy(ctx)


if __name__ == "__main__":
    main()
