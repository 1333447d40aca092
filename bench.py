"""Benchmark: propagation steps/s of the one-way Helmholtz propagator on one MI355X.

Workload (named `scalar1024`): scalar field, 1024 x 1024 grid at lambda/4,
sine-product medium n = 1 + 0.02 sin(2 pi x) sin(2 pi y), Gaussian beam waist
32 lambda, 16-pole AAA-Lawson rational approximation, dz = lambda, GMRES tol
1e-8 (restart 30), edge layer 128 cells.  A "step" is one full propagation
step: every pole's preconditioned GMRES solve plus the residue-weighted sum.

Both precisions run from the same initial field for warmup + steps steps; the
mixed-precision field must agree with the all-FP64 field to 1e-6 relative L2
and the faster mode that meets it is reported.  Inputs are resident in HBM
before timing; the timed region is bracketed by torch.cuda.synchronize().

The warmup steps time every kernel class with HIP events (the per-class
breakdown and the dominant class); in the timed steps every fourth launch of
the dominant class is bracketed by events (on the plan's stream: an event
record costs about 6 us of stream time, so timing every launch would slow the
step it measures), and its roofline figure is the algorithmic bytes the library
counts for the timed launches over their event time.  cpu_baseline times the CPU
oracle on a bounded sample of the same workload.

Other workloads (--config): batch64 (64 independent propagations of uneven
sizes run concurrently), learned (a U-Net trained on the GPU from the
propagator's own solves supplies GMRES starting points; timed against the plain
method and the previous-step start on scalar1024), unet (training steps of that
U-Net at its training shape), copy (the HBM reference for the counters) and
pml512 and pml512v (absorbing layers, scalar and vector: 512^2 with PML layers
of 64 cells, the eigen-route Sylvester preconditioner's dense products), fit (the rational fit on the device
against the host's), sqrt1024 (the scalar1024 workload
through the pseudo-differential form: 25
Cauchy-integral terms of sqrt(1+z), alpha = 1, eight RK4 substeps of lambda/8
per lambda step, FP64; the field is compared with the exponential form's after
the same number of steps) and sineprod768 (z-dependent rotated sine-product
media, one n^2 plane per step: the coefficient refresh of every step).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
SQRT_TERMS, SQRT_ALPHA, SQRT_SUBSTEPS = 25, 1.0, 8
KERNEL_SOURCES = ("kernels.hip", "fft.hpp", "wave.hpp", "cplx.hpp", "state.hpp", "kernels.hpp")
COUNTERS = os.path.join(ROOT, "profiles", "row_apply_scalar1024_fp64_hbm_counters.md")


def counter_traffic(kernel, workload="scalar1024"):
    """HBM bytes per launch of `kernel` on `workload` (FP64) from the committed FETCH_SIZE / WRITE_SIZE
    summary, or None when there is none for that pair or the kernel sources changed since it was
    taken."""
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2410_17446_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    try:
        with open(COUNTERS) as fh:
            kv = dict(line.split(" = ", 1) for line in fh.read().splitlines() if " = " in line)
    except OSError:
        return None
    if (kv.get("source_sha256", "").strip() != h.hexdigest() or kv.get("traffic_kernel", "").strip() != kernel
            or kv.get("traffic_workload", "").strip() != workload):
        return None
    return float(kv["traffic_bytes_per_launch"])


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", default="scalar1024")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--modes", default="mixed,mixed64,fp64")
    ap.add_argument("--autotune", type=int, default=4,
                    help="timed steps per column-pass variant before the warmup (0: the default variant)")
    ap.add_argument("--cpu-poles", type=int, default=8, help="poles of one oracle step in the CPU sample")
    ap.add_argument("--workers", type=int, default=8, help="batch workers (batch64 workload)")
    ap.add_argument("--unet-base", type=int, default=32, help="U-Net base channels (learned workload)")
    ap.add_argument("--train-n", type=int, default=256, help="training grid (learned workload)")
    ap.add_argument("--learned-workload", default="scalar1024", choices=["scalar1024", "vector2048"],
                    help="workload the learned guesses are timed on")
    ap.add_argument("--learned-chunk", type=int, default=None,
                    help="poles per U-Net forward pass (learned; default 8, and 4 for vector2048, whose 206 GB "
                         "workspace leaves room for the activations of 4)")
    ap.add_argument("--train-draws", type=int, default=48, help="(medium, beam) draws for training")
    ap.add_argument("--train-seconds", type=float, default=90.0, help="training time budget")
    ap.add_argument("--event-period", type=int, default=EVENT_PERIOD,
                    help="time every n-th launch of the dominant kernel in the timed steps")
    ap.add_argument("--no-exp-compare", action="store_true",
                    help="sqrt1024: skip the exponential-form run the field is compared with")
    ap.add_argument("--unet-precision", default="bf16", choices=["bf16", "f32"],
                    help="U-Net 3x3 convolutions: bf16 matrix cores or float32")
    ap.add_argument("--bytes-out", default=None,
                    help="write {mode: {kernel class: [launches, algorithmic bytes]}} over every launch of the "
                         "warmup and timed steps (to pair with a profiler's per-dispatch counters)")
    return ap.parse_args()


def run_batch(args):
    """The batch64 workload: 64 independent propagations (N in 256..1024, 8/12/16 poles, sine or random
    media), each `steps` steps after `warmup`, run concurrently by the library's batch workers."""
    import numpy as np
    import torch

    from paper_2410_17446_amd import hp, inputs, tables
    probs = inputs.batch_configs(64)
    tabs = {}
    problems, ins, meds = [], [], []
    for cfg in probs:
        key = cfg["npoles"]
        if key not in tabs:
            tabs[key] = tables.plan_tables(inputs.K0 * cfg["dz"], key)
        poles, residues, r_inf, d2, d1 = tabs[key]
        N = cfg["N"]
        problems.append(dict(nx=N, ny=N, dx=cfg["dx"], dy=cfg["dx"], k0=inputs.K0, n0=1.0, dz=cfg["dz"], ncomp=1,
                             poles=poles, residues=residues, r_inf=r_inf, d2=d2, d1=d1, edge_width=cfg["W"],
                             edge_eta=cfg["eta_max"], tol=cfg["tol"], restart=cfg["restart"]))
        ins.append(torch.from_numpy(inputs.beam(cfg)).cuda())
        meds.append(torch.from_numpy(inputs.medium_n2(cfg)).cuda())
    b = hp.Batch(problems, nworkers=args.workers)
    # launch-shape autotuner once per grid size (on that size's first problem), outside the timed
    # region; every problem of the size takes the choice
    variants = {}
    if args.autotune:
        for i, pr in enumerate(problems):
            if pr["nx"] not in variants:
                plan = hp.Plan(**pr, max_cycles=20)
                plan.set_medium(meds[i])
                variants[pr["nx"]] = plan.autotune(ins[i], reps=args.autotune)[1]
                plan.close()
        b.set_launch([variants[pr["nx"]] for pr in problems])
    if args.warmup:
        ins = b.propagate(ins, meds, [args.warmup] * len(problems))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    outs = b.propagate(ins, meds, [args.steps] * len(problems))
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    it, sec = b.stats()
    total_steps = args.steps * len(problems)
    finite = all(bool(torch.isfinite(torch.view_as_real(o)).all()) for o in outs)
    b.close()
    # what the concurrency buys: the same problems and steps with 1 worker (one problem at a time,
    # one stream) and with 2 and 4 workers; the library's workers share the box's hardware queues
    sweep = {}
    for nw in sorted({1, 2, 4} - {args.workers}):
        bw = hp.Batch(problems, nworkers=nw)
        if variants:
            bw.set_launch([variants[pr["nx"]] for pr in problems])
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        bw.propagate(ins, meds, [args.steps] * len(problems))
        torch.cuda.synchronize()
        sweep[nw] = total_steps / (time.perf_counter() - t1)
        bw.close()
        print(f"# {nw} workers: {sweep[nw]:.1f} steps/s", file=sys.stderr, flush=True)
    sweep[args.workers] = total_steps / dt
    # spot check: three problems (smallest, middle, largest) stepped by single plans equal the batch
    order = sorted(range(len(problems)), key=lambda i: problems[i]["nx"])
    spot = {}
    for i in (order[0], order[len(order) // 2], order[-1]):
        plan = hp.Plan(**problems[i], max_cycles=20)
        if variants:
            plan.set_launch(variants[problems[i]["nx"]])
        ref = plan.propagate(ins[i], args.steps, n2=meds[i])
        plan.close()
        spot[i] = bool(torch.equal(ref, outs[i]))
    line = {"metric": "batch propagation steps/s (64 problems, N 256..1024, 8-16 poles)",
            "value": total_steps / dt, "unit": "steps/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
            "ms_per_step": 1e3 * dt / total_steps, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
            "dtype": "c128", "data": "synthetic",
            "config": {"workload": "batch64", "problems": len(problems), "workers": args.workers,
                       "sizes": sorted({p["nx"] for p in problems}),
                       "column_variant_by_size": {str(k): v for k, v in sorted(variants.items())}},
            "gmres_iterations": int(sum(it)), "all_finite": finite,
            "busiest_problem_s": max(sec),
            "steps_per_s_by_workers": {str(k): v for k, v in sorted(sweep.items())},
            "speedup_vs_one_worker": (total_steps / dt) / sweep[1],
            "single_plan_equal": {str(k): v for k, v in spot.items()}}
    print(json.dumps(line))
    return 0


def unet_forward_flops(levels, base, cin, cout, H, W):
    """Multiply-adds x 2 of one forward pass (3x3 and 1x1 convolutions)."""
    ch = lambda l: base << l
    f = 2 * ch(0) * cout * H * W
    for l in range(levels):
        pl = (H >> l) * (W >> l)
        f += 18 * ((cin if l == 0 else ch(l - 1)) * ch(l) + ch(l) * ch(l)) * pl
        if l + 1 < levels:
            f += 18 * ((ch(l + 1) + ch(l)) * ch(l) + ch(l) * ch(l)) * pl
    return f


def run_learned(args):
    """Learned initial guesses (the plan's HP_GUESS_LEARNED mode: U-Net guesses for every pole,
    computed in batched forward passes, with the lockstep solves of all poles) against the plain
    method and the previous-step start, on the scalar1024 workload (the headline's second arm) or,
    with --learned-workload vector2048, on the 2048^2 vector workload (E_x, E_y, 24 poles): train
    a U-Net on FP64 solve pairs the propagator makes at --train-n (random media and beams, the same
    pole table), then time steps of all three modes from the same field (the plain method's field
    after the warmup steps)."""
    import numpy as np
    import torch

    from paper_2410_17446_amd import hp, inputs, learn, tables
    from paper_2410_17446_amd.unet import HP_UNET_BF16, HP_UNET_F32, UNet
    cfg = dict(inputs.CONFIGS[args.learned_workload])
    nc = cfg["ncomp"]
    if args.learned_chunk is None:
        args.learned_chunk = 4 if args.learned_workload == "vector2048" else 8
    cin, cout = 4 * nc + 3, 2 * nc
    poles, residues, r_inf, d2, d1 = tables.plan_tables(inputs.K0 * cfg["dz"], cfg["npoles"])
    fit = dict(poles=poles, residues=residues, r_inf=r_inf)
    levels, base = 4, args.unet_base
    prec = HP_UNET_BF16 if args.unet_precision == "bf16" else HP_UNET_F32
    net = UNet(levels, base, cin, cout, seed=0, precision=prec)
    t0 = time.perf_counter()
    X, T = learn.generate(net, fit, d2, d1, args.train_n, nc, count=args.train_draws, seed=1, tol=1e-10,
                          poles_per_field=8)
    Xv, Tv = learn.generate(net, fit, d2, d1, args.train_n, nc, count=8, seed=2, tol=1e-10, poles_per_field=8)
    t_gen = time.perf_counter() - t0
    print(f"# training pairs: {X.shape[0]} at {args.train_n}^2 in {t_gen:.1f} s", file=sys.stderr, flush=True)
    learn.train(net, X, T, steps=3, batch=8, lr=1e-3)   # first calls allocate; not timed
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    learn.train(net, X, T, steps=20, batch=8, lr=1e-3)
    torch.cuda.synchronize()
    per = (time.perf_counter() - t0) / 20
    nsteps = max(10, int(args.train_seconds / per))
    net = UNet(levels, base, cin, cout, seed=0, precision=prec)
    t0 = time.perf_counter()
    losses = learn.train(net, X, T, steps=nsteps, batch=8, lr=1e-3, lr_final=1e-4, log_every=max(1, nsteps // 5))
    torch.cuda.synchronize()
    t_train = time.perf_counter() - t0
    mse, mse0 = learn.evaluate(net, Xv, Tv)
    print(f"# trained {nsteps} Adam steps in {t_train:.1f} s; held-out mse {mse:.3e} vs free-space {mse0:.3e}",
          file=sys.stderr, flush=True)
    del X, T
    N = cfg["N"]
    mk = lambda: hp.Plan(nx=N, ny=N, dx=cfg["dx"], dy=cfg["dx"], k0=inputs.K0, n0=1.0, dz=cfg["dz"], ncomp=nc,
                         poles=poles, residues=residues, r_inf=r_inf, d2=d2, d1=d1, edge_width=cfg["W"],
                         edge_eta=cfg["eta_max"], tol=cfg["tol"], restart=cfg["restart"], max_cycles=20)
    w0 = torch.from_numpy(inputs.beam(cfg)).cuda()
    n2 = torch.from_numpy(inputs.medium_n2(cfg)).cuda()
    base_plan = mk()
    start = base_plan.propagate(w0, args.warmup, n2=n2) if args.warmup else w0.clone()
    base_plan.close()
    res = {}
    for mode in ("plain", "prev", "learned"):
        plan = mk()
        plan.set_medium(n2)
        if mode == "prev":
            plan.set_guess(hp.HP_GUESS_PREV)
            plan.step(start)           # the first step has no previous solutions; untimed
        # the learned mode: the library computes every pole's guess from the net at the start of
        # each step (hp_set_guess_net + HP_GUESS_LEARNED); its time is the "guess" kernel class
        lg = learn.LearnedGuess(plan, net, chunk=args.learned_chunk) if mode == "learned" else None
        if lg is not None:
            lg.step(start)             # allocate activations; untimed
            plan.profile(True, classes=["guess"])
        a = start.clone()
        b = torch.empty_like(a)
        its, acc_total = [], 0
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for s in range(args.steps):
            if lg is None:
                plan.step(a, E_out=b)
            else:
                _, acc = lg.step(a, E_out=b)
                acc_total += sum(acc)
            its.append(sum(plan.stats()[0]))
            a, b = b, a
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        res[mode] = dict(steps_per_s=args.steps / dt, iters_per_step=float(np.mean(its)), field=a)
        if lg is not None:
            res[mode]["guess_ms_per_step"] = plan.profile_read()["guess"][1] / args.steps
            res[mode]["accepted_frac"] = acc_total / (args.steps * plan.npoles)
            plan.profile(False)
        plan.close()
        print(f"# {mode}: {res[mode]['steps_per_s']:.2f} steps/s, {res[mode]['iters_per_step']:.1f} iterations "
              f"per step", file=sys.stderr, flush=True)
    ref = res["plain"]["field"].cpu().numpy()
    for mode in res:
        f = res[mode].pop("field").cpu().numpy()
        res[mode]["err_vs_plain"] = float(np.linalg.norm(f - ref) / np.linalg.norm(ref))
    # U-Net forward throughput at the inference shape (learned_chunk poles per launch)
    x = torch.randn(args.learned_chunk, cin, N, N, device="cuda")
    net.forward(x)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(3):
        net.forward(x)
    torch.cuda.synchronize()
    fwd = (time.perf_counter() - t0) / 3
    tflops = unet_forward_flops(levels, base, cin, cout, N, N) * args.learned_chunk / fwd / 1e12
    what = f"{N}^2{' vector' if nc == 2 else ''}, {cfg['npoles']} poles, tol {cfg['tol']:g}"
    line = {"metric": f"propagation steps/s ({what}) with learned initial guesses, all poles batched",
            "value": res["learned"]["steps_per_s"], "unit": "steps/s", "n_gpus": 1, "steps": args.steps,
            "warmup": args.warmup, "ms_per_step": 1e3 / res["learned"]["steps_per_s"], "higher_is_better": True,
            "scaling": "weak", "vs_baseline": None, "dtype": "c128+f32", "data": "synthetic",
            "config": {"workload": args.learned_workload, "grid": N, "poles": cfg["npoles"], "tol": cfg["tol"],
                       "unet": {"levels": levels, "base": base, "params": net.nparam,
                                "convolutions": args.unet_precision, "poles_per_forward": args.learned_chunk},
                       "training": {"grid": args.train_n, "components": nc, "pairs": args.train_draws * 8,
                                    "adam_steps": nsteps, "batch": 8, "seconds": t_train,
                                    "datagen_seconds": t_gen, "final_loss": float(np.mean(losses[-20:])),
                                    "heldout_mse": mse, "heldout_mse_free_space": mse0}},
            "modes": res,
            "roofline": ({"bound": "mfma", "kernel": "unet forward (k_conv3_mfma, bf16)", "achieved": tflops,
                          "peak": 2500.0, "unit": "TFLOP/s", "frac": tflops / 2500.0, "traffic": None}
                         if args.unet_precision == "bf16" else
                         {"bound": "alu", "kernel": "unet forward (k_conv3, fp32)", "achieved": tflops, "peak": 157.3,
                          "unit": "TFLOP/s", "frac": tflops / 157.3, "traffic": None})}
    print(json.dumps(line))
    return 0


def run_unet(args):
    """U-Net training throughput (the learned-guess network, 4 levels, --unet-base channels, 7 inputs,
    2 outputs) at the training shape: batches of 8 synthetic 256^2 samples (--train-n), one step =
    forward, reverse pass and Adam update.  FLOPs per step: 3x the forward's multiply-adds x 2
    (data and weight gradients each cost a forward); roofline against the bf16 matrix-core peak
    (or the fp32 vector peak with --unet-precision f32)."""
    import torch

    from paper_2410_17446_amd.unet import HP_UNET_BF16, HP_UNET_F32, UNet
    levels, base, B, H = 4, args.unet_base, 8, args.train_n
    prec = HP_UNET_BF16 if args.unet_precision == "bf16" else HP_UNET_F32
    net = UNet(levels, base, 7, 2, seed=0, precision=prec)
    g = torch.Generator(device="cuda").manual_seed(0)
    x = torch.randn((B, 7, H, H), device="cuda", generator=g)
    t = torch.randn((B, 2, H, H), device="cuda", generator=g)
    for _ in range(args.warmup):
        net.grad(x, t)
        net.adam(1e-4)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        net.grad(x, t)
        net.adam(1e-4)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / max(args.steps, 1)
    flops = 3 * unet_forward_flops(levels, base, 7, 2, H, H) * B
    tf = flops / dt / 1e12
    peak, bound = (2500.0, "mfma") if args.unet_precision == "bf16" else (157.3, "alu")
    line = {"metric": "U-Net training steps/s (forward + gradients + Adam, batch 8)", "value": 1.0 / dt,
            "unit": "steps/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": 1e3 * dt,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
            "dtype": "bf16 operands, f32 accumulate" if args.unet_precision == "bf16" else "f32",
            "data": "synthetic",
            "config": {"workload": "unet_train", "levels": levels, "base": base, "batch": B, "grid": H,
                       "params": net.nparam},
            "roofline": {"bound": bound, "kernel": "whole training step", "achieved": tf, "peak": peak,
                         "unit": "TFLOP/s", "frac": tf / peak, "traffic": None}}
    print(json.dumps(line))
    return 0


def run_copy(args):
    """Reference for HBM counters: `steps` launches of a plain elementwise copy (torch.add(a, 0)) of
    a 1 GiB float64 buffer into another; algorithmic bytes 2 GiB per launch."""
    import torch
    n = (1 << 30) // 8
    a = torch.arange(n, dtype=torch.float64, device="cuda")
    b = torch.empty_like(a)
    for _ in range(args.warmup):
        torch.add(a, 0, out=b)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        torch.add(a, 0, out=b)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / max(args.steps, 1)
    print(json.dumps({"config": "copy", "bytes_per_launch": 2 * n * 8, "seconds_per_launch": dt,
                      "GBps": 2 * n * 8 / dt / 1e9}))
    return 0


EVENT_PERIOD = 4  # the timed steps bracket every 4th launch of the dominant kernel with events


def run_mode(hp, torch, cfg, tables, precision, w0, n2, warmup, steps, form=None, event_period=EVENT_PERIOD,
             autotune=0, pml=None):
    poles, residues, r_inf, d2, d1 = tables
    N = cfg["N"]
    plan = hp.Plan(nx=N, ny=N, dx=cfg["dx"], dy=cfg["dx"], k0=hp_k0(), n0=1.0, dz=cfg["dz"], ncomp=cfg["ncomp"],
                   poles=poles, residues=residues, r_inf=r_inf, d2=d2, d1=d1, edge_width=cfg["W"],
                   edge_eta=cfg["eta_max"], tol=cfg["tol"], restart=cfg["restart"], max_cycles=20,
                   precision=precision)
    if form is not None:
        plan.set_form(*form)
    if pml is not None:
        plan.set_pml(*pml)
    plan.set_medium(n2)
    create_status = plan.create_status
    a = w0.clone()
    b = torch.empty_like(a)
    # launch-shape autotuner (before the warmup, outside the timed region): `autotune` timed steps
    # per column-pass variant, the plan keeps the fastest
    variant = plan.autotune(a, reps=autotune, E_out=b)[1] if autotune else 1
    # warmup: every kernel class timed (the per-class breakdown, and which class dominates)
    plan.profile(True)
    if warmup:
        plan.propagate(a, warmup, E_out=b)
        a, b = b, a
    breakdown = plan.profile_read()
    warm_totals = plan.profile_totals()
    dom = max(breakdown, key=lambda k: breakdown[k][1]) if warmup else "row_apply"
    # timed steps: events around every event_period-th launch of the dominant class only
    plan.profile(True, classes=[dom])
    plan.profile_sample(event_period)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    plan.propagate(a, steps, E_out=b)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    prof = plan.profile_read()
    totals = plan.profile_totals()
    iters, relres = plan.stats()
    plan.profile(False)
    plan.close()
    run_totals = {k: [warm_totals[k][0] + totals[k][0], warm_totals[k][1] + totals[k][1]] for k in totals}
    return dict(seconds=dt, field=b, prof=prof, totals=totals, run_totals=run_totals, dom=dom, breakdown=breakdown,
                iters=iters, relres=relres, variant=variant, create_status=create_status)


def spectrum_max_abs_r(cfg, tab):
    """max |e^{-iK} r(mu_p + mu_q)| over the plan's discrete free-space spectrum (host check of the
    PF table; the library's hp_plan_create reports HP_WARN_UNSTABLE when it exceeds 1 + 1e-6)."""
    import numpy as np
    poles, residues, r_inf, d2, _ = tab
    N, dx = cfg["N"], cfg["dx"]
    q = np.arange(1, N)
    sym = d2[0] + 2.0 * np.cos(np.outer(q * np.pi / N, np.arange(1, 7))) @ np.asarray(d2[1:])
    mu = sym / (hp_k0() * dx) ** 2
    lam = np.unique(np.round((mu[:, None] + mu[None, :]).ravel(), 13))
    r = r_inf + (1.0 / (lam[:, None] - np.asarray(poles)[None, :])) @ np.asarray(residues)
    return float(np.abs(r).max())


def hp_k0():
    from paper_2410_17446_amd import inputs
    return inputs.K0


def cpu_model():
    """The host CPU's model name (Linux), for the CPU baseline's record."""
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(cfg, npoles_sample, sqrt_form=False, one_core_poles=2):
    """Oracle on a bounded sample: `npoles_sample` pole solves of step 1 (of its first RK stage for the
    pseudo-differential form), scaled to steps/s."""
    import numpy as np

    from oracle import fit, stencil
    from oracle import operator as op
    from oracle import sqrt_form as sf
    from oracle import step as st
    from paper_2410_17446_amd import inputs
    c, d = stencil.stencils()
    if sqrt_form:
        pf = sf.cauchy_sqrt_pf(cfg["npoles"], SQRT_ALPHA)
        f = {"poles": pf.poles}
        solves_per_pole = 4 * SQRT_SUBSTEPS
    else:
        f = fit.fit_exp_sqrt(inputs.K0 * cfg["dz"], cfg["npoles"])
        solves_per_pole = 1
    g = op.Grid(N=cfg["N"], dx=cfg["dx"], dy=cfg["dx"], k0=inputs.K0, n0=1.0, c=c, d=d, W=cfg["W"],
                eta_max=cfg["eta_max"])
    n2 = inputs.medium_n2(cfg)
    w = inputs.beam(cfg)
    co = op.coefficients(g, n2, cfg["ncomp"] == 2)
    k = min(npoles_sample, cfg["npoles"])
    picks = [int(i * cfg["npoles"] / k) for i in range(k)]   # spread over the pole list
    threads = min(os.cpu_count() or 1, int(os.environ.get("OMP_NUM_THREADS") or os.cpu_count() or 1))
    t0 = time.perf_counter()
    iters = []
    for j in picks:
        r = st.solve_pole(g, co, w, f["poles"][j], cfg["tol"], cfg["restart"], workers=threads)
        iters.append(r.iters)
    dt = time.perf_counter() - t0
    step_s = dt * cfg["npoles"] * solves_per_pole / k
    where = "the first RK stage of step 1" if sqrt_form else "step 1"
    scale = f"{cfg['npoles']} x {solves_per_pole}/{k}" if sqrt_form else f"{cfg['npoles']}/{k}"
    out = dict(value=1.0 / step_s, unit="steps/s", cores=threads, kind="oracle", cpu=cpu_model(),
               sample=f"GMRES solves of poles {picks} (of {cfg['npoles']}) in {where} of the {cfg['N']}^2 "
                      f"workload ({dt:.1f} s, iterations {iters}); per-step time = sample time x "
                      f"{scale}; scipy.fft uses {threads} threads, the rest of numpy one")
    if one_core_poles > 0:
        # the same oracle on one core (FFTs and BLAS both single-threaded), a smaller sample
        from threadpoolctl import threadpool_limits
        k1 = min(one_core_poles, k)
        picks1 = picks[::max(1, k // k1)][:k1]
        t0 = time.perf_counter()
        with threadpool_limits(limits=1):
            for j in picks1:
                st.solve_pole(g, co, w, f["poles"][j], cfg["tol"], cfg["restart"], workers=1)
        dt1 = time.perf_counter() - t0
        out["one_core"] = dict(value=k1 / (dt1 * cfg["npoles"] * solves_per_pole), unit="steps/s", cores=1,
                               sample=f"poles {picks1} of {where} ({dt1:.1f} s), scaled by "
                                      f"{cfg['npoles'] * solves_per_pole}/{k1}")
    return out


def run_sineprod(args):
    """z-dependent media (Sec. 2: n and psi refreshed for every new step; the rotated sine-product
    media of Sec. 5.3): a Gaussian beam (1/e radius 25 lambda) over 240 lambda, n0 = 1.2,
    dn = 0.025, steps of a quarter of the medium's wavelength, q = 1 (medium wavenumber k0 n0) and
    q = 2 (0.5 k0 n0), 768^2 cells of lambda/4 (192 lambda; edge layer 24 lambda), 16 poles, FP64,
    tol 1e-8.  Every step takes its own n^2 plane (hp_propagate with a plane stride: coefficient
    refresh each step); the planes are generated on the device before the timed region.  Reports
    steps/s over both runs and the beam's power."""
    import numpy as np
    import torch

    from paper_2410_17446_amd import hp, inputs, tables
    N, dx, L, n0, dn, w0 = 768, 0.25, 240.0, 1.2, 0.025, 25.0
    k0 = inputs.K0
    R = inputs.rotation_matrix()
    xs = torch.tensor(inputs.coords(N, dx), dtype=torch.float64, device="cuda")
    Y, X = torch.meshgrid(xs, xs, indexing="ij")
    d2, d1 = tables.stencil_d2(), tables.stencil_d1()
    runs, total_steps, total_s = {}, 0, 0.0
    for q in (1.0, 2.0):
        dz = q / (4 * n0)
        nsteps = int(round(L / dz))
        ks = k0 * n0 / (np.sqrt(3.0) * q)
        stack = torch.empty((nsteps, N, N), dtype=torch.float64, device="cuda")
        for st in range(nsteps):
            z = st * dz
            xt = R[0, 0] * X + R[0, 1] * Y + R[0, 2] * z
            yt = R[1, 0] * X + R[1, 1] * Y + R[1, 2] * z
            zt = R[2, 0] * X + R[2, 1] * Y + R[2, 2] * z
            n = n0 + dn * torch.sin(ks * xt) * torch.sin(ks * yt) * torch.sin(ks * zt)
            stack[st] = n * n
        for st in (0, nsteps // 2):   # the device planes are the input module's planes
            ref = inputs.rotated_sine_n2(N, dx, st * dz, n0=n0, dn=dn, q=q)
            assert np.abs(stack[st].cpu().numpy() - ref).max() < 1e-12
        f = tables.RationalFit(k0 * n0 * dz, 16)
        plan = hp.Plan(nx=N, ny=N, dx=dx, dy=dx, k0=k0, n0=n0, dz=dz, ncomp=1, poles=f.poles, residues=f.residues,
                       r_inf=f.r_inf, d2=d2, d1=d1, edge_width=N // 8, edge_eta=0.25, tol=1e-8, restart=30,
                       max_cycles=20)
        w = torch.from_numpy(inputs.gaussian_beam(N, dx, w0)).cuda()
        out = torch.empty_like(w)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        plan.propagate(w, nsteps, n2=stack, n2_step_stride=N * N, E_out=out)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        iters, _ = plan.stats()
        plan.close()
        power = float((out[0].abs() ** 2).sum() / (w[0].abs() ** 2).sum())
        runs[f"q{q:g}"] = {"steps": nsteps, "dz": dz, "seconds": dt, "steps_per_s": nsteps / dt,
                           "last_step_iters": int(sum(iters)), "power_ratio": power}
        print(f"# q={q:g}: {nsteps} steps in {dt:.1f} s ({nsteps / dt:.1f} steps/s), power ratio {power:.6f}",
              file=sys.stderr, flush=True)
        total_steps += nsteps
        total_s += dt
        del stack
    line = {
        "metric": "propagation steps/s (768^2, 16 poles, z-dependent rotated sine-product media, 240 lambda)",
        "value": total_steps / total_s, "unit": "steps/s", "n_gpus": 1, "steps": total_steps, "warmup": 0,
        "ms_per_step": 1e3 * total_s / total_steps, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "c128", "data": "synthetic",
        "config": {"workload": "sineprod768", "grid": N, "poles": 16, "tol": 1e-8, "n0": n0, "dn": dn,
                   "beam_radius": w0, "range": L},
        "runs": runs,
    }
    print(json.dumps(line))
    return 0


FP64_VALU_PEAK_TFS = 78.6   # MI355X FP64 vector (and FP64 matrix) peak
PML_SIGMA = 10.0


def run_pml(args, ncomp=1):
    """Absorbing layers (Sec. 4.1): the workload of the sine-product runs of Sec. 5 on 512^2 cells of
    lambda/4 (128 lambda) with PML layers of 64 cells (16 lambda) on every side, sigma_max = 10, a
    Gaussian beam (1/e radius 8 lambda; x-polarised for vector fields) tilted 20 degrees off axis and
    16 lambda off centre toward the layer, sine-product medium n = 1 + 0.02 sin(2 pi x) sin(2 pi y),
    16 poles, dz = lambda, tol 1e-8, FP64; scalar (pml512) or vector (pml512v: coupled E_x, E_y).
    The preconditioner is the eigen route of the stretched Sylvester equation: four dense complex
    products per pole, component and Arnoldi step."""
    import numpy as np
    import torch

    from paper_2410_17446_amd import hp, inputs, tables
    N, W = 512, 64
    cfg = dict(N=N, dx=0.25, ncomp=ncomp, W=W, eta_max=0.25, dz=1.0, npoles=16, tol=1e-8, restart=30,
               medium=("sine", 0.02, 1.0), w0=8.0)
    tab = tables.plan_tables(inputs.K0 * cfg["dz"], cfg["npoles"])
    Q, Qi, lam = tables.pml_eigen(N, cfg["dx"], inputs.K0, 1.0, W, PML_SIGMA, tab[3], tab[4])
    cond = float(np.linalg.cond(Q))
    w = inputs.tilted_beam(N, cfg["dx"], cfg["w0"], np.sin(np.radians(20.0)), x0=16.0)
    if ncomp == 2:
        w = np.concatenate([w, np.zeros_like(w)])
    w0 = torch.from_numpy(w).cuda()
    n2 = torch.from_numpy(inputs.medium_n2(cfg)).cuda()
    r = run_mode(hp, torch, cfg, tab, hp.HP_FP64, w0, n2, args.warmup, args.steps, event_period=args.event_period,
                 pml=(PML_SIGMA, Q, Qi, lam), autotune=args.autotune)
    value = args.steps / r["seconds"]
    prof, brk, dom = r["prof"], r["breakdown"], r["dom"]
    n_l, ms, amount = prof[dom]
    if dom == "pml_gemm":
        achieved = amount / (ms * 1e-3) / 1e12 if ms > 0 else 0.0
        roof = {"bound": "alu", "kernel": "pml_gemm (the four dense stages of a round)", "achieved": achieved,
                "peak": FP64_VALU_PEAK_TFS, "unit": "TFLOP/s", "frac": achieved / FP64_VALU_PEAK_TFS,
                "traffic": None, "algorithmic_flops_per_launch": amount / max(n_l, 1),
                "flops_convention": "8 (N-1)^3 per complex product actually needed: four per pole that did the "
                                    "round, and in the step's first round two shared by all poles plus two per pole",
                "peak_is": "FP64 vector ALU (256 CUs x 2.4 GHz x 128 FP64 flops/clock; the FP64 matrix "
                           "cores have the same rate)"}
    else:
        achieved = amount / (ms * 1e-3) / 1e9 if ms > 0 else 0.0
        roof = {"bound": "hbm", "kernel": dom, "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": achieved / HBM_PEAK_GBS, "traffic": None}
    roof.update({"launches": n_l, "avg_launch_us": 1e3 * ms / max(n_l, 1),
                 "timed": f"every {args.event_period}th launch in the timed steps"})
    f_in, f_out = w0.cpu().numpy(), r["field"].cpu().numpy()
    gemm_ms = brk["pml_gemm"][1]
    line = {
        "metric": f"propagation steps/s ({N}^2{' vector' if ncomp == 2 else ''}, {cfg['npoles']} poles, "
                  f"PML layers of {W} cells)",
        "value": value, "unit": "steps/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": 1e3 * r["seconds"] / args.steps, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "c128", "data": "synthetic",
        "config": {"workload": "pml512v" if ncomp == 2 else "pml512", "grid": N, "pml_cells": W, "sigma_max": PML_SIGMA, "poles": cfg["npoles"],
                   "tol": cfg["tol"], "mode": "fp64", "beam": "1/e radius 8 lambda, 20 degrees, 16 lambda off axis",
                   "dense_stage_variant": r["variant"]},
        "last_step_iters": r["iters"], "last_step_true_relres_max": max(r["relres"]),
        "eigenvector_condition": cond,
        "power_ratio": float(np.sum(np.abs(f_out) ** 2) / np.sum(np.abs(f_in) ** 2)),
        "roofline": roof,
        "warmup_kernel_ms": {k: brk[k][1] for k in brk},
        "warmup_pml_gemm_TFLOPs": (brk["pml_gemm"][2] / (gemm_ms * 1e-3) / 1e12) if gemm_ms > 0 else None,
    }
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline_pml(cfg, tab, w, inputs.medium_n2(cfg))
    if ncomp == 2:
        line["power_in_E_y"] = float(np.sum(np.abs(f_out[1]) ** 2) / np.sum(np.abs(f_out) ** 2))
    print(json.dumps(line))
    return 0


def cpu_baseline_pml(cfg, tab, w, n2):
    """The oracle's PML solve (Bartels-Stewart preconditioner) of one pole of step 1, scaled to steps/s."""
    from oracle import operator as op
    from oracle import pml
    from paper_2410_17446_amd import inputs
    poles = tab[0]
    g = pml.PMLGrid(N=cfg["N"], h=cfg["dx"], k0=inputs.K0, n0=1.0, c=tab[3], d=tab[4], W=cfg["W"],
                    sigma_max=PML_SIGMA)
    threads = min(os.cpu_count() or 1, int(os.environ.get("OMP_NUM_THREADS") or os.cpu_count() or 1))
    j = len(poles) // 2
    t0 = time.perf_counter()
    if cfg["ncomp"] == 2:
        co = op.coefficients(pml.vector_grid(g), n2, True)
        r = pml.solve_pole_vector(g, co, w, poles[j], cfg["tol"], cfg["restart"])
    else:
        r = pml.solve_pole(g, pml.medium(g, n2), w[0], poles[j], cfg["tol"], cfg["restart"])
    dt = time.perf_counter() - t0
    return dict(value=1.0 / (dt * cfg["npoles"]), unit="steps/s", cores=threads, kind="oracle", cpu=cpu_model(),
                sample=f"GMRES solve of pole {j} (of {cfg['npoles']}) in step 1 of the {cfg['N']}^2 PML workload "
                       f"({dt:.1f} s, {r.iters} iterations); per-step time = sample time x {cfg['npoles']}; "
                       f"numpy/scipy BLAS and LAPACK threads as the box sets them")


def run_fit(args):
    """The rational fit of Sec. 3.1 on the device (hp_fit_exp_sqrt) against the host's (tables.RationalFit):
    time per fit and the largest sample error of each, for the step sizes of the workloads (dz = lambda,
    16 poles), the beam runs (dz = lambda/20, n0 = 1.0003, 25 poles) and a quarter-wave step."""
    import numpy as np
    import torch

    from paper_2410_17446_amd import hp, inputs, tables
    torch.cuda.synchronize()
    hp.fit_exp_sqrt(inputs.K0, 8)           # module load and first launch, outside the timings
    cases = [("dz=lambda", inputs.K0, 16), ("dz=lambda/4", inputs.K0 / 4, 12),
             ("beam dz=lambda/20", inputs.K0 * 1.0003 * 0.05, 25)]
    out = {}
    for name, K, deg in cases:
        t0 = time.perf_counter()
        p, r, ri, e_dev = hp.fit_exp_sqrt(K, deg)
        t_dev = time.perf_counter() - t0
        t0 = time.perf_counter()
        f = tables.RationalFit(K, deg)
        t_host = time.perf_counter() - t0
        z = np.linspace(-4, 2, 4001)
        e_host = float(np.abs(f(z) - tables.exp_sqrt(z, K)).max())
        out[name] = {"K": K, "poles": deg, "device_s": t_dev, "host_s": t_host, "device_max_err": e_dev,
                     "host_max_err": e_host}
        print(f"# {name}: device {t_dev * 1e3:.0f} ms ({e_dev:.2e}), host {t_host * 1e3:.0f} ms ({e_host:.2e})",
              file=sys.stderr, flush=True)
    tot_dev = sum(v["device_s"] for v in out.values())
    line = {"metric": "rational fits/s (AAA-Lawson of exp(iK sqrt(1+z)), 4001 samples, 40 Lawson steps)",
            "value": len(out) / tot_dev, "unit": "fits/s", "n_gpus": 1, "steps": len(out), "warmup": 1,
            "ms_per_step": 1e3 * tot_dev / len(out), "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": "f64", "data": "synthetic",
            "config": {"workload": "fit", "cases": [c[0] for c in cases]},
            "fits": out,
            "host_fits_per_s": len(out) / sum(v["host_s"] for v in out.values())}
    print(json.dumps(line))
    return 0


def run_sqrt(args):
    """scalar1024 through the pseudo-differential form (FP64), compared with the exponential form."""
    import numpy as np
    import torch

    from paper_2410_17446_amd import hp, inputs, tables
    cfg = dict(inputs.CONFIGS["scalar1024"], npoles=SQRT_TERMS)
    b, a, r = tables.cauchy_sqrt_table(SQRT_TERMS, SQRT_ALPHA)
    tab = (b, a, r, tables.stencil_d2(), tables.stencil_d1())
    w0 = torch.from_numpy(inputs.beam(cfg)).cuda()
    n2 = torch.from_numpy(inputs.medium_n2(cfg)).cuda()
    res = run_mode(hp, torch, cfg, tab, hp.HP_FP64, w0, n2, args.warmup, args.steps,
                   form=(hp.HP_FORM_SQRT, SQRT_SUBSTEPS), event_period=args.event_period)
    value = args.steps / res["seconds"]
    cmp = None
    if not args.no_exp_compare:
        ecfg = dict(inputs.CONFIGS["scalar1024"])
        ex = run_mode(hp, torch, ecfg, tables.plan_tables(inputs.K0 * ecfg["dz"], ecfg["npoles"]), hp.HP_FP64, w0,
                      n2, args.warmup, args.steps)
        f, g = res["field"].cpu().numpy(), ex["field"].cpu().numpy()
        cmp = {"steps_per_s": args.steps / ex["seconds"],
               "rel_l2_difference": float(np.linalg.norm(f - g) / np.linalg.norm(g))}
        print(f"# exponential form {cmp['steps_per_s']:.2f} steps/s; fields differ by "
              f"{cmp['rel_l2_difference']:.3e} (relative L2) after {args.warmup + args.steps} steps", file=sys.stderr)
    print(f"# sqrt form: {value:.3f} steps/s", file=sys.stderr)
    prof, brk, dom = res["prof"], res["breakdown"], res["dom"]
    n_l, ms, by = prof[dom]
    achieved = by / (ms * 1e-3) / 1e9 if ms > 0 else 0.0
    line = {
        "metric": (f"propagation steps/s ({cfg['N']}^2, pseudo-differential form: {SQRT_TERMS} Cauchy-integral terms "
                   f"of sqrt(1+z), RK4 with {SQRT_SUBSTEPS} substeps per lambda step)"),
        "value": value, "unit": "steps/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": 1e3 * res["seconds"] / args.steps, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "c128", "data": "synthetic",
        "config": {"workload": "sqrt1024", "grid": cfg["N"], "terms": SQRT_TERMS, "alpha": SQRT_ALPHA,
                   "substeps": SQRT_SUBSTEPS, "tol": cfg["tol"], "mode": "fp64"},
        "last_step_iters_summed_over_stages": res["iters"],
        "exponential_form": cmp,
        "roofline": {"bound": "hbm", "kernel": dom, "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": None,
                     "algorithmic_bytes_per_launch": by / max(n_l, 1), "launches": n_l,
                     "avg_launch_us": 1e3 * ms / max(n_l, 1),
                     "timed": f"every {args.event_period}th launch in the timed steps"},
        "warmup_kernel_ms": {k: brk[k][1] for k in brk},
    }
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline(cfg, 2, sqrt_form=True, one_core_poles=0)
    print(json.dumps(line))
    return 0


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (got --gpus {args.gpus}); run it with --gpus 1", file=sys.stderr)
        return 2
    if args.config == "batch64":
        return run_batch(args)
    if args.config == "learned":
        return run_learned(args)
    if args.config == "copy":
        return run_copy(args)
    if args.config == "unet":
        return run_unet(args)
    if args.config == "sqrt1024":
        return run_sqrt(args)
    if args.config == "sineprod768":
        return run_sineprod(args)
    if args.config == "pml512":
        return run_pml(args)
    if args.config == "pml512v":
        return run_pml(args, ncomp=2)
    if args.config == "fit":
        return run_fit(args)
    import numpy as np
    import torch

    from paper_2410_17446_amd import hp, inputs, tables
    cfg = dict(inputs.CONFIGS[args.config])
    K = inputs.K0 * cfg["dz"]
    tab = tables.plan_tables(K, cfg["npoles"])
    w0 = torch.from_numpy(inputs.beam(cfg)).cuda()
    n2 = torch.from_numpy(inputs.medium_n2(cfg)).cuda()
    res = {}
    modes = args.modes.split(",")
    if "fp64" not in modes:
        modes.append("fp64")   # the reference every other mode's field is compared with
    for mode in modes:
        prec = {"mixed": hp.HP_MIXED, "mixed64": hp.HP_MIXED64}.get(mode, hp.HP_FP64)
        res[mode] = run_mode(hp, torch, cfg, tab, prec, w0, n2, args.warmup, args.steps, autotune=args.autotune,
                             event_period=args.event_period)
        print(f"# {mode}: {args.steps / res[mode]['seconds']:.2f} steps/s, last-step iterations "
              f"{res[mode]['iters']}", file=sys.stderr, flush=True)
    if args.bytes_out:
        with open(args.bytes_out, "w") as fh:
            json.dump({m: res[m]["run_totals"] for m in res}, fh, indent=1)
    errs = {}
    if "fp64" in res:
        ref = res["fp64"]["field"].cpu().numpy()
        for m in res:
            if m != "fp64":
                f = res[m]["field"].cpu().numpy()
                errs[m] = float(np.linalg.norm(f - ref) / np.linalg.norm(ref))
    choices = [m for m in modes if m == "fp64" or errs.get(m, 1.0) <= 1e-6]
    best = min(choices, key=lambda m: res[m]["seconds"])
    r = res[best]
    value = args.steps / r["seconds"]
    prof, brk, dom = r["prof"], r["breakdown"], r["dom"]
    n_l, ms, by = prof[dom]
    achieved = by / (ms * 1e-3) / 1e9 if ms > 0 else 0.0
    inner_ms = brk["col"][1] + brk["row_apply"][1]
    inner_b = brk["col"][2] + brk["row_apply"][2]
    n_all, b_all = r["totals"][dom]
    f_in, f_out = w0.cpu().numpy(), r["field"].cpu().numpy()
    power = {"initial": float(np.sum(np.abs(f_in) ** 2)), "final": float(np.sum(np.abs(f_out) ** 2)),
             "steps": args.warmup + args.steps}
    power["ratio"] = power["final"] / power["initial"]
    line = {
        "metric": (f"propagation steps/s ({cfg['N']}^2{' vector' if cfg['ncomp'] == 2 else ''}, {cfg['npoles']} poles, "
                   f"err<=1e-6 vs FP64), plain GPU method"),
        "value": value,
        "unit": "steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * r["seconds"] / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"mixed": "c64+f64", "mixed64": "c64 storage, f64 arithmetic"}.get(best, "c128"),
        "data": "synthetic",
        "config": {"workload": args.config, "grid": cfg["N"], "poles": cfg["npoles"], "tol": cfg["tol"],
                   "mode": best, "method": "plain (zero initial guess)", "column_variant": r["variant"]},
        "err_vs_fp64": errs.get(best, 0.0 if best == "fp64" else None),
        "err_vs_fp64_by_mode": errs,
        "modes": {m: {"steps_per_s": args.steps / res[m]["seconds"], "last_step_iters": res[m]["iters"]}
                  for m in res},
        "roofline": {"bound": "hbm", "kernel": dom, "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS,
                     "traffic": counter_traffic(dom, args.config) if best == "fp64" else None,
                     "traffic_is": "FETCH_SIZE + WRITE_SIZE per launch (L2-to-fabric bytes: HBM and the "
                                   "Infinity Cache), scaled by a plain copy's reading",
                     "algorithmic_bytes_per_launch": by / max(n_l, 1),
                     "bytes_convention": "each distinct field once per launch (the first basis vector S_x w, "
                                         "shared by every pole in its first cycle, counted once)",
                     "launches": n_l, "avg_launch_us": 1e3 * ms / max(n_l, 1),
                     "timed": f"every {args.event_period}th launch in the timed steps",
                     "all_launches_timed_steps": n_all,
                     "algorithmic_bytes_per_launch_all": b_all / max(n_all, 1)},
        "mfma": {"used_by_propagator": False,
                 "why": "no dense contraction on the path: the preconditioner is a DST-I (FFT), the operator a "
                        "13-point stencil and a pointwise medium product, and each pole's Gram-Schmidt inner "
                        "products are matrix-vector products against its own Krylov basis (no basis is shared "
                        "between poles), all HBM-bound"},
        "plan": {"create_status": r["create_status"],
                 "max_abs_e_iK_r_on_spectrum": spectrum_max_abs_r(cfg, tab)},
        "power": power,
        "inner_loop_roofline": {"kernels": ["col", "row_apply"], "steps": "warmup",
                                "achieved": inner_b / (inner_ms * 1e-3) / 1e9 if inner_ms > 0 else 0.0,
                                "frac": (inner_b / (inner_ms * 1e-3) / 1e9) / HBM_PEAK_GBS if inner_ms > 0 else 0.0},
        "warmup_kernel_ms": {k: brk[k][1] for k in brk},
        "warmup_kernel_GBps": {k: brk[k][2] / (brk[k][1] * 1e-3) / 1e9 for k in brk if brk[k][1] > 0 and brk[k][2] > 0},
    }
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline(cfg, args.cpu_poles)
    print(json.dumps(line))
    return 0


if __name__ == "__main__":
    sys.exit(main())
