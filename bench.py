#!/usr/bin/env python
"""Benchmark of the batched multi-Debye fitting hot path on one MI355X.

Default workload: 65,536 user-style tables (each a seeded sum of one to three
Havriliak-Negami terms with 1 % multiplicative Gaussian noise), F = 4096
log-spaced points on 1e5-1e11 Hz, N = 20 poles, 128 particles per material:
8,388,608 candidates, inputs resident in HBM.

One step = one swarm iteration over the whole batch: the swarm move of every
particle, then the batched cost evaluation of all 8.4M candidates (the
paper's hybrid fit, Sec. III-B: swarm over the relaxation times, damped least
squares for the weights, flip, eps_inf, cost).  value = cost evaluations per
second over the timed steps, counting only the share of a sampled parity
check that is within 1e-10 of the FP64 oracle (or of its 80-bit instance).

The JSON line also carries:
  - roofline: the cost kernel (the only kernel of an evaluation at this shape),
    timed with HIP events on the stream it is launched on, against the FP64
    vector peak;
  - fwd_adjoint_kernel_evals_per_s: the forward + variable-projection adjoint
    kernel over the same 8.4M candidates;
  - fwd_no_refine_kernel_evals_per_s: the forward kernel without the
    refinement step (DEBYE_FLAG_NO_REFINE; not the tolerance of `value`);
  - fwd_dd_refine_kernel_evals_per_s: the forward kernel with the refinement
    step in double-double (DEBYE_FLAG_DD_REFINE), and in parity_sample_dd_refine
    the parity sample's candidates evaluated that way, judged like the others;
  - polish: 50 L-BFGS steps (adjoint gradients, up to 30 Armijo trials) on
    every material's swarm best, timed once;
  - batched_vs_per_material: a shard of the materials fitted whole (all swarm
    iterations + polish) in one batch, against the plain per-material loop
    (forward evaluations only) run until each material reaches the batched
    final cost;
  - cpu_baseline: the oracle on the host cores, on a bounded sample of the
    same workload, and parity_sample: that sample judged against the oracle.

Usage: python bench.py [--gpus 1] [--steps 3] [--warmup 1] [--workload tables]
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP64_VALU = 78.6e12   # 256 CUs x 4 SIMD x 16 lanes x 2 flop (FMA) x 2.4 GHz
T_TRIALS, MEM = 30, 10


def algorithmic_flops(F, N):
    """Useful FP64 work of one cost evaluation, basis counted once:
    basis 5FN, Gram FN(N+1), rhs 2FN, column sums FN, residuals 4FN + F,
    cost 4F, dense solve N^3/3 + 2N^2."""
    return F * (N * N + 13 * N + 5) + N ** 3 / 3 + 2 * N * N


def algorithmic_bytes(F, N, P_per_mat):
    """HBM bytes one evaluation must move: its log10(tau) row in, cost out,
    and its share of the material's three spectra."""
    return 8 * N + 8 + 24 * F / P_per_mat


def kernel_source_hash():
    import hashlib
    # the cost kernel's own source: its file and the device helpers it includes
    src = b"".join(open(os.path.join(ROOT, "paper_2109_01928_amd", "csrc", f), "rb").read()
                   for f in ("fit_kernel.hpp", "fit_eval.hip", "common.hpp"))
    return hashlib.sha256(src).hexdigest()[:16]


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def make_workload(W, args):
    it = args.iters
    if args.workload == "mixed":
        wl = W.mixed_uniform(M=args.materials or 1024, N=args.poles or 8, iters=it if it >= 0 else 200)
    elif args.workload == "single":
        wl = W.single_hn()
    elif args.workload == "ragged":
        wl = W.mixed_ragged(M=args.materials or 4096, iters=it if it >= 0 else 300)
    elif args.workload == "hncc":
        wl = W.hn_cc(M=args.materials or 1024, N=args.poles or 12, iters=it if it >= 0 else 200)
    else:
        wl = W.tables(M=args.materials or 65536, iters=it if it >= 0 else 400)
    if it >= 0:
        wl.iters = it
    return wl


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="tables", choices=["tables", "mixed", "single", "ragged", "hncc"],
                    help="tables (default): 65536 HN-sum tables, F=4096, N=20, 128 particles; mixed: 1024 mixed "
                         "materials, F=1000, N=8, 256 particles; single: one HN, F=50, N=5, 40 particles; ragged: "
                         "4096 materials of uneven F/N/swarm size; hncc: 1024 HN/CC, F=2000, N=12")
    ap.add_argument("--optimizer", default="pso", choices=["pso", "de", "da"],
                    help="global search: particle swarm (default), differential evolution (rand/1/bin) or "
                         "annealing (batched generalized simulated annealing chains)")
    ap.add_argument("--materials", type=int, default=0, help="override the workload's material count")
    ap.add_argument("--poles", type=int, default=0, help="override the pole count (mixed and hncc workloads)")
    ap.add_argument("--iters", type=int, default=-1, help="override the workload's swarm iterations (shard fit)")
    ap.add_argument("--polish-steps", type=int, default=-1)
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--per-material", type=int, default=8,
                    help="materials timed in the plain per-material loop (0: only the batched whole fit of the "
                         "shard; -1: skip both)")
    ap.add_argument("--shard", type=int, default=512,
                    help="materials of the batched whole fit that the per-material loop is compared with")
    ap.add_argument("--no-extras", action="store_true",
                    help="only the timed steps (no adjoint rate, polish leg or per-material comparison)")
    ap.add_argument("--launch", default="auto", choices=["auto", "buckets", "persistent"],
                    help="several pole counts: per-bucket launches, one persistent launch, or the autotuner's choice")
    ap.add_argument("--no-autotune", action="store_true", help="keep the plan's default frequency splits")
    ap.add_argument("--autotune-reps", type=int, default=1)
    ap.add_argument("--freq-split", type=int, default=0,
                    help="fixed frequency split for every pole count (implies --no-autotune)")
    ap.add_argument("--only-eval", type=int, default=0,
                    help="profiling: run this many forward launches of the swarm batch and exit")
    ap.add_argument("--only-grad", type=int, default=0,
                    help="profiling: run this many forward+adjoint launches of the swarm batch and exit")
    ap.add_argument("--copy-bytes", type=int, default=0,
                    help="profiling: time a device-to-device copy of this many bytes (counter calibration) and exit")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU: the fit shards by material with no communication, "
              "so the per-GPU rate is the figure; run it with --gpus 1 on a single MI355X.", file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2109_01928_amd as D
    import workloads as W

    dev = "cuda:0"
    torch.cuda.set_device(0)
    if args.copy_bytes:
        src = torch.ones(args.copy_bytes // 8, dtype=torch.float64, device=dev)
        dst = torch.empty_like(src)
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes": src.numel() * 8, "launches": 5}), flush=True)
        return
    wl = make_workload(W, args)
    if args.polish_steps < 0:
        args.polish_steps = wl.polish_steps
    M, P = wl.M, wl.P
    uniform = len(set(np.diff(wl.f_off))) == 1 and len(set(wl.n_poles)) == 1
    N = int(wl.n_poles.max())
    F = int(np.max(np.diff(wl.f_off)))
    P_per = int(np.max(np.diff(wl.cand_off)))
    log(f"workload {wl.name}: {M} materials, {P} candidates")

    # ---- set-up (outside the timed region): inputs resident in HBM, targets, plan
    zeros = torch.zeros(len(wl.omega), dtype=torch.float64, device=dev)
    b = D.Batch(wl.f_off, wl.cand_off, wl.n_poles, wl.omega, zeros, zeros, dev)
    kind_t = torch.tensor(wl.kind, dtype=torch.int8, device=dev)
    params_t = torch.tensor(wl.params, dtype=torch.float64, device=dev)
    er, ei = D.material_eval(kind_t, params_t, b, noise_seed=wl.noise_seed)
    bb = b.with_targets(er, ei)
    del zeros
    lb = torch.tensor(wl.lb, device=dev)
    ub = torch.tensor(wl.ub, device=dev)
    plan = D.Plan(b)
    theta0 = torch.tensor(W.draw_theta(wl.cand_off, wl.n_poles, wl.lb, wl.ub, wl.ld, seed=77), device=dev)
    if args.launch != "auto":
        plan.set_launch(D.LAUNCH_BUCKETS if args.launch == "buckets" else D.LAUNCH_PERSISTENT)
    if args.freq_split:
        plan.set_freq_split(args.freq_split)
    elif not args.no_autotune:
        t = time.perf_counter()
        plan.autotune(bb, theta0, reps=args.autotune_reps)
        log(f"autotuned in {time.perf_counter() - t:.1f} s: {plan.info()}")
    work_per_eval = float(np.sum(np.diff(wl.cand_off) * np.array(
        [algorithmic_flops(int(f), int(n)) for f, n in zip(np.diff(wl.f_off), wl.n_poles)])))
    cost = torch.empty(P, dtype=torch.float64, device=dev)
    status = torch.empty(P, dtype=torch.int8, device=dev)
    out = (cost, None, None, status)
    stream = torch.cuda.current_stream()

    if args.only_eval or args.only_grad:
        for _ in range(args.only_eval):
            D.fit_eval(plan, bb, theta0, want_weights=False, out=out)
        for _ in range(args.only_grad):
            D.fit_eval_grad(plan, bb, theta0)
        torch.cuda.synchronize()
        print(json.dumps({"launches": args.only_eval + args.only_grad, "evals_per_launch": P,
                          "flops_per_eval": algorithmic_flops(F, N),
                          "alg_bytes_per_eval": algorithmic_bytes(F, N, P_per)}), flush=True)
        return

    sw = D.Swarm.empty(P, M, wl.ld, 1, dev)
    pop = D.Population.empty(P, M, wl.ld, 1, dev) if args.optimizer in ("de", "da") else None

    def evaluate(theta, evs):
        if evs is not None:
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
        D.fit_eval(plan, bb, theta, want_weights=False, out=out)
        if evs is not None:
            e1.record(stream)
            evs.append((e0, e1))

    # iteration 0: initial swarm / population and its evaluation
    if args.optimizer == "de":
        D.de_init(bb, lb, ub, pop, seed=wl.seed)
        evaluate(pop.x, None)
        D.de_select(bb, pop, 0, pop.x, cost, history=False)
    elif args.optimizer == "da":
        D.da_init(bb, lb, ub, pop, seed=wl.seed)
        evaluate(pop.x, None)
        D.da_accept(bb, pop, 0, pop.x, cost, seed=wl.seed, history=False)
    else:
        D.pso_init(bb, lb, ub, sw, wl.inertia, wl.c1, wl.c2, wl.seed)
        evaluate(sw.x, None)

    def iteration(t, evs=None):
        if args.optimizer == "de":
            D.de_trial(bb, lb, ub, pop, t, seed=wl.seed)
            evaluate(pop.u, evs)
            D.de_select(bb, pop, t, pop.u, cost, history=False)
        elif args.optimizer == "da":
            D.da_visit(bb, lb, ub, pop, t, seed=wl.seed)
            evaluate(pop.u, evs)
            D.da_accept(bb, pop, t, pop.u, cost, seed=wl.seed, history=False)
        else:
            D.pso_step(bb, lb, ub, sw, t, True, cost, wl.inertia, wl.c1, wl.c2, wl.seed, history=False)
            evaluate(sw.x, evs)

    for t in range(1, args.warmup + 1):
        iteration(t)
    torch.cuda.synchronize()
    events = []
    log(f"timing {args.steps} steps")
    t0 = time.perf_counter()
    for t in range(args.warmup + 1, args.warmup + args.steps + 1):
        iteration(t, events)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    ms_per_step = 1e3 * dt / args.steps
    value = P * args.steps / dt
    durs = np.array([a.elapsed_time(c) for a, c in events]) * 1e-3
    avg = float(durs.mean())
    achieved = work_per_eval / avg
    log(f"{ms_per_step:.1f} ms per step, evaluation {1e3 * avg:.1f} ms")
    if args.optimizer == "pso":
        D.pso_step(bb, lb, ub, sw, args.warmup + args.steps + 1, False, cost, wl.inertia, wl.c1, wl.c2, wl.seed,
                   history=False)

    sched = plan.info()
    kernel = "fit_kernel (all pole-count buckets of one evaluation)"
    if uniform:
        s0 = sched[0]
        kernel = (f"fit_kernel<{N},{s0['pole_split']},false,"
                  f"{(1 if s0['freq_split'] == 1 else 2) if s0['uniform'] else 0}>")
    line = {
        "metric": "Debye-fit cost evals/s (fwd, fwd+adjoint), rel err <=1e-10 vs FP64 oracle",
        "value": value,
        "unit": "evals/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic (seeded materials; no dataset in the paper)",
        "config": {"workload": f"{wl.name.split(' I')[0]}: one {args.optimizer.upper()} iteration (move + cost "
                               f"evaluation of every candidate) per step",
                   "materials": M, "freq_points": F if uniform else "ragged", "poles": N if uniform else "ragged",
                   "particles": P_per if uniform else "ragged", "evals_per_step": P},
        "schedule": {f"N{i['n_poles']}": f"{i['pole_split']}x{i['freq_split']} lanes" for i in sched},
        "launch": "one launch" if len(sched) == 1 else
                  ("persistent" if plan.launch() == D.LAUNCH_PERSISTENT else "per-bucket launches"),
        "roofline": {"bound": "alu", "achieved": achieved / 1e12, "peak": PEAK_FP64_VALU / 1e12,
                     "unit": "TFLOP/s", "frac": achieved / PEAK_FP64_VALU,
                     "traffic": measured_traffic(wl, kernel, sched), "kernel": kernel, "avg_launch_s": avg,
                     "flops_per_eval": work_per_eval / P, "evals_per_launch": P},
        "fwd_kernel_evals_per_s": P / avg,
    }

    if not args.no_extras:
        theta = (pop.x if pop is not None else sw.x)
        line["fwd_adjoint_kernel_evals_per_s"] = adjoint_rate(D, plan, bb, theta, stream)
        line["fwd_no_refine_kernel_evals_per_s"] = flagged_rate(D, plan, bb, theta, stream, D.FLAG_NO_REFINE)
        line["fwd_dd_refine_kernel_evals_per_s"] = flagged_rate(D, plan, bb, theta, stream, D.FLAG_DD_REFINE)
        best = (pop.best_x if pop is not None else sw.gbest_x).clone()
        if args.polish_steps > 0:
            line["polish"] = polish_leg(D, wl, er, ei, best, lb, ub, args.polish_steps, stream)
        if args.per_material >= 0:
            line["batched_vs_per_material"] = shard_comparison(D, W, wl, er, ei, args)
        del theta, best
    if not args.no_cpu_baseline:
        line["cpu_baseline"], line["parity_sample"], dd = cpu_leg(D, W, wl, er, ei, plan, args.cpu_seconds,
                                                                   dd_refine=not args.no_extras)
        if dd is not None:
            line["parity_sample_dd_refine"] = dd
        # counted evaluations: only those within the parity tolerance (sampled rate)
        ps = line["parity_sample"]
        line["value_raw"] = value
        line["value"] = value * ps["within_1e-10"] / ps["candidates"]
    print(json.dumps(line), flush=True)


def measured_traffic(wl, kernel, sched):
    """HBM bytes per launch from the rocprofv3 FETCH_SIZE / WRITE_SIZE record in
    profiles/ (scaled by a plain copy's readings), used only while the kernel
    source, the workload and the schedule are the ones it was taken on."""
    tfile = os.path.join(ROOT, "profiles", "fit_eval_traffic.json")
    if not os.path.exists(tfile):
        return None
    for rec in json.load(open(tfile)).get("records", []):
        if (rec.get("source_sha256_16") == kernel_source_hash() and rec.get("workload") == wl.name.split(" I")[0]
                and rec.get("kernel") == kernel and rec.get("freq_split") == sched[0]["freq_split"]):
            return rec["bytes_per_launch"]
    return None


def adjoint_rate(D, plan, bb, theta, stream, reps=2):
    import torch
    log("forward + adjoint kernel rate")
    D.fit_eval_grad(plan, bb, theta)
    torch.cuda.synchronize()
    g0, g1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    g0.record(stream)
    for _ in range(reps):
        D.fit_eval_grad(plan, bb, theta)
    g1.record(stream)
    torch.cuda.synchronize()
    return bb.P * reps / (g0.elapsed_time(g1) * 1e-3)


def flagged_rate(D, plan, bb, theta, stream, flags, reps=2):
    """Forward kernel rate under `flags`: DEBYE_FLAG_NO_REFINE (no refinement
    pass; accuracy limited by the conditioning of the normal equations) or
    DEBYE_FLAG_DD_REFINE (the refinement pass in double-double)."""
    import torch
    log(f"forward kernel rate with flags {flags}")
    D.fit_eval(plan, bb, theta, flags=flags, want_weights=False)
    torch.cuda.synchronize()
    g0, g1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    g0.record(stream)
    for _ in range(reps):
        D.fit_eval(plan, bb, theta, flags=flags, want_weights=False)
    g1.record(stream)
    torch.cuda.synchronize()
    return bb.P * reps / (g0.elapsed_time(g1) * 1e-3)


def polish_leg(D, wl, er, ei, best, lb, ub, steps, stream):
    """50 L-BFGS steps on every material's swarm best: per step one batched
    forward launch of every material's full step, then launches of further
    Armijo trials only for the materials still undecided (the next four
    halvings, then the rest), and one forward + adjoint launch at the accepted
    points; materials that accept no trial stall and drop out of the
    launches."""
    import torch
    log(f"polish leg: {steps} steps x {T_TRIALS} trials on {wl.M} materials")
    b1 = D.Batch(wl.f_off, np.arange(wl.M + 1), wl.n_poles, wl.omega, er, ei)
    pol = D.Polish(b1, wl.ld, steps=steps, mem=MEM, max_trials=T_TRIALS)   # set-up: allocates
    hist = torch.empty((wl.M, steps + 1), dtype=torch.float64, device=best.device)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    pol.run(b1, best, lb, ub, cost_hist=hist)
    e1.record(stream)
    torch.cuda.synchronize()
    s = e0.elapsed_time(e1) * 1e-3
    h = hist.cpu().numpy()
    drop = 1 - h[:, -1] / h[:, 0]
    # materials whose last step still moved (the others stalled: no acceptable trial)
    moving = float(np.mean(h[:, -1] < h[:, -2])) if steps > 0 else 0.0
    return {"materials": wl.M, "steps": steps, "trials": T_TRIALS, "seconds": s, "ms_per_step": 1e3 * s / max(steps, 1),
            "median_rel_cost_drop": float(np.median(drop)), "moving_at_last_step": moving,
            "monotone": bool(np.all(np.diff(h, axis=1) <= 0))}


def shard_comparison(D, W, wl, er, ei, args):
    """Batched fit vs the plain per-material loop at equal final residual: the
    first `shard` materials fitted together (the chosen optimiser with the
    workload's population and iteration count, enqueued at once, then the L-BFGS
    polish); then, for the swarm only, the first `per_material` of them, each
    material alone (its own plan and swarm,
    forward evaluations only, the host reading the best cost after every
    iteration) until its best cost is within 1e-3 of the batched final cost, or
    10x the iterations.  Times per material are compared; the per-material
    time is extrapolated linearly to the shard."""
    import torch
    S = min(args.shard, wl.M)
    log(f"batched whole fit of {S} materials ({wl.iters} iterations), then the per-material loop")
    f_end = int(wl.f_off[S])
    fo = wl.f_off[:S + 1]
    co = wl.cand_off[:S + 1]
    bs = D.Batch(fo, co, wl.n_poles[:S], wl.omega[:f_end], er[:f_end].contiguous(), ei[:f_end].contiguous())
    plan = D.Plan(bs)
    plan.autotune(bs, torch.tensor(W.draw_theta(co, wl.n_poles[:S], wl.lb[:S], wl.ub[:S], wl.ld, seed=5),
                                   device="cuda"), reps=1)
    sw = D.Swarm.empty(bs.P, S, wl.ld, wl.iters + 1)
    lbs, ubs = torch.tensor(wl.lb[:S], device="cuda"), torch.tensor(wl.ub[:S], device="cuda")
    b1 = D.Batch(fo, np.arange(S + 1), wl.n_poles[:S], wl.omega[:f_end], bs.eps_re, bs.eps_im)
    steps = args.polish_steps
    pol = D.Polish(b1, wl.ld, steps=max(steps, 1), mem=MEM, max_trials=T_TRIALS)
    plan1 = D.Plan(b1)

    pop = D.Population.empty(bs.P, S, wl.ld, wl.iters + 1) if args.optimizer != "pso" else None

    def batched(mode):
        if args.optimizer == "de":
            D.de_run(plan, bs, lbs, ubs, pop, wl.iters, seed=wl.seed, use_graph=mode)
        elif args.optimizer == "da":
            D.da_run(plan, bs, lbs, ubs, pop, wl.iters, seed=wl.seed, use_graph=mode)
        else:
            D.pso_run(plan, bs, lbs, ubs, sw, wl.iters, wl.inertia, wl.c1, wl.c2, wl.seed, use_graph=mode)
        best = (pop.best_x if pop is not None else sw.gbest_x).clone()
        if steps > 0:
            pol.run(b1, best, lbs, ubs)
        return best

    times = {}
    for mode in (False, True):
        batched(mode)
        torch.cuda.synchronize()
        t = time.perf_counter()
        best = batched(mode)
        c1, w1, e1, _ = D.fit_eval(plan1, b1, best)
        torch.cuda.synchronize()
        times["graph" if mode else "eager"] = time.perf_counter() - t
    final = c1.cpu().numpy()
    afe = D.afe(b1, best, w1, e1).cpu().numpy()
    batched_s = times["graph"]
    # the plain per-material loop (the swarm's; for DE and DA only the batched fit is timed)
    K = min(args.per_material, S) if args.optimizer == "pso" else 0
    cap = 10 * wl.iters
    t_mat, reached, used = [], 0, []
    for m in range(K):
        f0, f1 = int(wl.f_off[m]), int(wl.f_off[m + 1])
        Pm, Nm = int(wl.cand_off[m + 1] - wl.cand_off[m]), int(wl.n_poles[m])
        bm = D.Batch([0, f1 - f0], [0, Pm], [Nm], wl.omega[f0:f1], er[f0:f1].contiguous(), ei[f0:f1].contiguous())
        pm = D.Plan(bm)
        swm = D.Swarm.empty(Pm, 1, Nm, 1)
        lbm, ubm = lbs[m:m + 1], ubs[m:m + 1]
        goal = final[m] * (1 + 1e-3)
        torch.cuda.synchronize()
        t = time.perf_counter()
        D.pso_init(bm, lbm, ubm, swm, wl.inertia, wl.c1, wl.c2, wl.seed)
        cm = D.fit_eval(pm, bm, swm.x, want_weights=False)[0]
        it, best_c = 0, float("inf")
        while best_c > goal and it < cap:
            it += 1
            D.pso_step(bm, lbm, ubm, swm, it, True, cm, wl.inertia, wl.c1, wl.c2, wl.seed, history=False)
            cm = D.fit_eval(pm, bm, swm.x, want_weights=False)[0]
            best_c = float(swm.gbest_cost.item())
        torch.cuda.synchronize()
        t_mat.append(time.perf_counter() - t)
        reached += best_c <= goal
        used.append(it)
    out = {"optimizer": args.optimizer, "shard_materials": S, "iterations": wl.iters, "polish_steps": steps,
           "batched_s": batched_s, "batched_eager_s": times["eager"], "batched_s_per_material": batched_s / S,
           "afe_percent_median": float(np.median(afe)), "afe_below_5_percent": float(np.mean(afe < 5.0))}
    if K > 0:
        per_mat = float(np.mean(t_mat))
        out.update({"per_material_timed": K, "per_material_s_mean": per_mat, "per_material_extrapolated_s": per_mat * S,
                    "speedup": per_mat * S / batched_s, "reached_batched_cost": f"{reached}/{K}",
                    "median_iterations": float(np.median(used)), "iteration_cap": cap})
    return out


def cpu_leg(D, W, wl, er, ei, plan, seconds, dd_refine=False):
    """The oracle on the host cores over a bounded sample of the workload (whole
    materials in order, the uniform initial candidates, until `seconds` of
    oracle time), and a parity check of the same candidates: the GPU evaluates
    the full batch in the timed launch configuration with the oracle's own
    targets in the sampled materials' segments, and each sampled cost is
    judged by oracle.judge_costs (within 1e-10 of the FP64 oracle, or of its
    80-bit instance).  With dd_refine the same candidates are evaluated again
    with DEBYE_FLAG_DD_REFINE and judged the same way."""
    import torch

    import oracle

    log("oracle leg on the host cores")
    theta = W.draw_theta(wl.cand_off, wl.n_poles, wl.lb, wl.ub, wl.ld, seed=77)
    nthreads = oracle.num_threads()

    def targets(m0, m1):
        mats = np.arange(m0, m1)
        f0, f1 = wl.f_off[m0], wl.f_off[m1]
        return oracle.material_eval_sample(wl.kind[mats], wl.params[mats], wl.f_off[m0:m1 + 1] - f0, wl.omega[f0:f1],
                                           mats, noise_seed=wl.noise_seed, nthreads=nthreads)

    def sub_batch(m0, m1, oer, oei):
        f0, f1 = wl.f_off[m0], wl.f_off[m1]
        return oracle.Batch(wl.f_off[m0:m1 + 1] - f0, wl.cand_off[m0:m1 + 1] - wl.cand_off[m0], wl.n_poles[m0:m1],
                            wl.omega[f0:f1], oer, oei)

    # timed sample: whole materials in order until `seconds` of oracle time
    done_m, t_cpu, costs, ers, eis = 0, 0.0, [], [], []
    chunk = max(1, min(16, int(2048 // max(1, np.max(np.diff(wl.cand_off))))))
    while t_cpu < seconds and done_m < wl.M:
        m1 = min(done_m + chunk, wl.M)
        oer, oei = targets(done_m, m1)
        th = theta[wl.cand_off[done_m]:wl.cand_off[m1]]
        t = time.perf_counter()
        c = oracle.fit_eval(sub_batch(done_m, m1, oer, oei), th, nthreads=nthreads)[0]
        t_cpu += time.perf_counter() - t
        costs.append(c)
        ers.append(oer)
        eis.append(oei)
        done_m = m1
    c64 = np.concatenate(costs)
    n = len(c64)
    oer, oei = np.concatenate(ers), np.concatenate(eis)
    # the same oracle on one core, about a fifth of the time budget
    m, t1, n1 = 0, 0.0, 0
    while t1 < seconds / 5 and m < done_m:
        m1 = min(m + 1, done_m)
        f0, f1 = wl.f_off[m] - wl.f_off[0], wl.f_off[m1] - wl.f_off[0]
        t = time.perf_counter()
        n1 += len(oracle.fit_eval(sub_batch(m, m1, oer[f0:f1], oei[f0:f1]), theta[wl.cand_off[m]:wl.cand_off[m1]],
                                  nthreads=1)[0])
        t1 += time.perf_counter() - t
        m = m1
    # GPU: identical targets in the sampled segments, full batch, the bench's plan
    fe = int(wl.f_off[done_m])
    gr, gi = er.clone(), ei.clone()
    gr[:fe] = torch.tensor(oer, device=er.device)
    gi[:fe] = torch.tensor(oei, device=er.device)
    tgt_err = float(max(np.max(np.abs(er[:fe].cpu().numpy() - oer) / np.maximum(np.abs(oer), 1e-300)),
                        np.max(np.abs(ei[:fe].cpu().numpy() - oei) / np.maximum(np.abs(oei), 1e-300))))
    bg = D.Batch(wl.f_off, wl.cand_off, wl.n_poles, wl.omega, gr, gi, er.device)
    tg = torch.tensor(theta, device=er.device)
    cg, _, _, stg = D.fit_eval(plan, bg, tg, want_weights=False)
    cg = cg.cpu().numpy()[:n]
    cdd = D.fit_eval(plan, bg, tg, flags=D.FLAG_DD_REFINE, want_weights=False)[0].cpu().numpy()[:n] if dd_refine else None
    del gr, gi, bg, tg
    per_m = np.array([np.sum(oer[wl.f_off[m]:wl.f_off[m + 1]] ** 2 + oei[wl.f_off[m]:wl.f_off[m + 1]] ** 2)
                      for m in range(done_m)])
    floor = 1e-12 * np.repeat(per_m, np.diff(wl.cand_off[:done_m + 1]))
    log(f"judging {n} sampled candidates")
    rel, judged = oracle.judge_costs(sub_batch(0, done_m, oer, oei), theta[:n], cg, c64, floor, 1e-10)
    cpu = {"value": n / t_cpu, "unit": "evals/s", "cores": nthreads, "kind": "oracle",
           "sample": f"the first {done_m} materials of the workload ({n} candidate evaluations: uniform log10 tau, "
                     f"the timed batch's layout), Householder-QR FP64 oracle, {t_cpu:.1f} s; one core: {n1} "
                     f"evaluations in {t1:.1f} s",
           "value_1core": n1 / t1}
    parity = {"candidates": n, "max_cost_rel_err": float(rel.max()), "oracle_limited": judged["oracle_limited"],
              "failed": judged["failed"], "within_1e-10": int((rel <= 1e-10).sum()),
              "max_err_vs_80bit_of_judged": judged["max_rel_80"],
              "status_ok": int(np.sum(stg.cpu().numpy()[:n] == 0)), "target_max_rel_err": tgt_err}
    if judged["over"]:
        parity["over"] = judged["over"][:8]
    dd = None
    if cdd is not None:
        log(f"judging the {n} candidates with the double-double refinement")
        rel_dd, jd = oracle.judge_costs(sub_batch(0, done_m, oer, oei), theta[:n], cdd, c64, floor, 1e-10)
        dd = {"candidates": n, "max_cost_rel_err": float(rel_dd.max()), "oracle_limited": jd["oracle_limited"],
              "failed": jd["failed"], "within_1e-10": int((rel_dd <= 1e-10).sum()),
              "max_err_vs_80bit_of_judged": jd["max_rel_80"]}
    return cpu, parity, dd


if __name__ == "__main__":
    main()
