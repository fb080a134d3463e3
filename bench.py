#!/usr/bin/env python3
"""Benchmark: time to a 1e-6 relative residual at 256^3, mixed (FP32 sweeps) vs plain FP64.

One step = one complete solve of the batched workload: the 256^3 layered medium
(eight layers, velocities U[1.5, 4.5] times (1 + 0.1 g), 8 points per wavelength,
8-cell absorbing layer), 8 point sources, 16 contour poles (eps and the exponential-Taylor
degree q chosen by the library's rules), FCI inside FP64 FGMRES(30), all 128 (pole, RHS)
shifted systems advanced together.  Inputs are resident in HBM before the timed region starts.

The run keeps to a wall-clock budget (--budget, counted from process start): the first
timed solve always runs; the metric's other arms (the oracle CPU baseline, the plain
FP64 solve, the learned preconditioner) run next if their estimated time fits; further
timed solves (up to --steps) fill what is left.  Anything the budget cuts is recorded
in the line ("skipped": "budget", or under "not_run"), and "steps"/"warmup" are the
counts actually run.  Opt-in arms: the 32^3 / 96^3 configurations (--small), uneven
batches (--uneven N), Alg. 1 step 4 (--k-in-list), case two (--case-two), contour
choices (--params), the Fourier-spectral operator (--spectral).

Prints ONE JSON line on stdout (everything else goes to stderr), carrying:
  value        time-to-1e-6 of the mixed-precision batched solve (s / solve batch),
               the mean over the timed solves
  roofline     the dominant kernel (middle factors of the product-form fixed-point step,
               complex64): algorithmic bytes / average launch time from HIP events on
               the library's stream during the timed solves, against 8 TB/s
  cpu_baseline the FP64 oracle on the host: per-stencil time on a bounded sample,
               projected to the matvec count of the timed solve
  fp64         the same solve with FP64 sweeps (plain method), and the speedup
  learned      training on the remainders FCI leaves on 128^3 random media, then the solve
               with the network as Alg. 1 step 4's inner preconditioner, on the headline
               workload and (against FCI alone) on an unseen 256^3 random-field medium
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

T_START = time.monotonic()  # the wall-clock budget counts from process start (before torch loads)

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "time-to-1e-6 residual & stencil GB/s at 256³: learned/FP32 vs plain FP64 (1 GPU)"
HBM_PEAK_GBS = 8000.0
PROFILES = os.path.join(ROOT, "profiles")
PROFILE_EVERY = 4


def traffic_file(shape):
    """Counter summary of the complex64 stage kernel at 256^3 for one launch shape."""
    return os.path.join(PROFILES, "traffic_fp_stage_c64_256_shape%s.json" % "-".join(str(v) for v in shape))


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def source_hash():
    h = hashlib.sha256()
    for name in ("stencil.hip", "zrows.h", "zrows_launch.h", "kernels.h"):
        with open(os.path.join(ROOT, "paper_1811_12378_amd", "csrc", name), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(shape, kernel):
    """Ratio of counter-measured HBM bytes to algorithmic bytes per launch of the middle
    kernel (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated), if the counters were
    taken on this source with the same launch shape and for this kernel."""
    try:
        with open(traffic_file(shape)) as fh:
            d = json.load(fh)
    except (OSError, ValueError):
        return None
    if d.get("source_hash") != source_hash() or list(d.get("shape", [])) != list(shape):
        return None
    if d.get("kernel") != kernel:
        return None
    if not d.get("alg_bytes_per_launch"):
        return None
    return d["bytes_per_launch"] / d["alg_bytes_per_launch"]


def middle_kernel_name(t, triple=False):
    """The library's kernel for the middle factors of a fixed-point step at launch shape t
    (triple: the three-factor passes of shapes with fuse 2)."""
    kern, ty, pd, _, fuse = t[:5]
    if fuse and kern <= 1:
        return "zrows_kernel (up to four middle factors of a fixed-point step per pass, planes in registers)"
    if triple:
        return ("ztrip_kernel (three middle factors of a fixed-point step per pass on 64 x 18 tiles, "
                "streams loaded straight into LDS)")
    if fuse and kern == 3:
        return ("zpair_tall_kernel (two middle factors of a fixed-point step per pass on 64 x 28 tiles, "
                "streams loaded straight into LDS)")
    if fuse and kern == 2:
        return ("zpair_dma_kernel<0, %d> (two middle factors of a fixed-point step per pass, streams loaded "
                "straight into LDS)" % (4 if pd >= 3 else 2))
    return "%s<float, EpiFactor<float, 0>, %d, %d> (middle factor of a fixed-point step)" % (
        "zlds_kernel" if kern == 1 else "zmarch_kernel", ty, pd)


def traffic_kernel(t, triple=False):
    """Kernel-name key of the counter summary for the middle kernel at launch shape t."""
    kern, _, pd, _, fuse = t[:5]
    if fuse and kern <= 1:
        return "zrows_kernel<float, 0, "  # the launches without residual or y1, of any width
    if triple:
        return "ztrip_kernel"
    if fuse and kern == 3:
        return "zpair_tall_kernel<0>"
    if fuse and kern == 2:
        return "zpair_dma_kernel<0, %d>" % (4 if pd >= 3 else 2)
    return "zlds_kernel" if kern == 1 else "zmarch_kernel"


def host_description():
    """CPU model, logical core count and the thread settings that could change the oracle's speed."""
    model = None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    env = {k: os.environ.get(k) for k in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS")}
    return {"cpu_model": model, "cpu_count": os.cpu_count(), "threads_env": env}


def cpu_baseline(wl, poles_oracle, n_matvecs, budget_s=15.0):
    """The FP64 oracle's fixed-point step (q stencil products each) on the same 256^3 input,
    timed on the host for a bounded sample and projected to the timed solve's product count.
    The oracle's stencil is NumPy element-wise work, which runs on one thread."""
    import numpy as np
    from oracle import fixed_point as OFP
    from oracle import operator as OO
    o = OO.Operator(wl.c, wl.omega, wl.damp_cells, wl.damp_rho2)
    p = poles_oracle[0]
    f = o.s * wl.rhs[0]
    y = np.zeros_like(f)
    Am = lambda x, s: o.apply(x, s)
    t0 = time.perf_counter()
    steps = 0
    while True:
        y = OFP.fixed_point_step(Am, y, f, p.z, p.z0, p.delta, p.q)
        steps += 1
        if time.perf_counter() - t0 > budget_s or steps >= 6:
            break
    dt = time.perf_counter() - t0
    per_mv = dt / (steps * p.q)
    out = {"value": per_mv * n_matvecs, "unit": "s", "cores": 1, "kind": "oracle", "projection": True,
           "sample": "%d fixed-point steps (q=%d, %d stencil products, %.1f s) of one pole at %d^3 in FP64 "
                     "NumPy on one host thread (%.3f s per product); value = that per-product time x the "
                     "%d stencil products of the timed solve (a projection: a full oracle solve at this "
                     "size would take days)" % (steps, p.q, steps * p.q, dt, wl.n, per_mv, n_matvecs),
           "per_matvec_s": per_mv, "sample_s": dt}
    out.update(host_description())
    return out


def cpu_full_solves(args):
    """Complete FP64 oracle solves on the host: the 32^3 constant medium to 1e-8 (8 poles,
    q = 8, FGMRES(30)), wall clock and iterations.  The 96^3 configuration is projected
    from its per-product time: a full oracle solve there runs for hours."""
    import numpy as np
    import workloads as W
    from oracle import fci as OF
    from oracle import operator as OO
    out = {}
    w1 = W.config_constant_32()
    o1 = OO.Operator(w1.c, w1.omega, w1.damp_cells, w1.damp_rho2)
    poles = OF.pole_parameters(o1, 8, 1.0, 0.5, 8)  # configuration 1 fixes degree 8
    t0 = time.perf_counter()
    u, info = OF.solve(o1, w1.rhs[0], poles, m=30, tol=1e-8, max_it=400)
    t = time.perf_counter() - t0
    b = o1.s * w1.rhs[0]
    rr = float(np.linalg.norm(b - o1.apply(np.asarray(u).reshape(o1.shape))) / np.linalg.norm(b))
    out["constant_32_fp64_tol1e-8"] = {"time_s": round(t, 2), "its": int(info["its"]), "relres": rr}
    w2 = W.config_grf_96()
    o2 = OO.Operator(w2.c, w2.omega, w2.damp_cells, w2.damp_rho2)
    x = np.asarray(w2.rhs[0])
    t0 = time.perf_counter()
    for _ in range(5):
        o2.apply(x, 0.1j)
    out["grf_96_per_product_s"] = round((time.perf_counter() - t0) / 5, 4)
    out.update(host_description())
    return out


def unet_flops_per_voxel():
    """Multiply-adds x 2 of the U-Net per fine voxel (3 real input channels)."""
    k = 2 * 27
    lvl1 = k * (3 * 16 + 16 * 16 + 48 * 16 + 16 * 16) + 2 * 16 * 2
    lvl2 = k * (16 * 32 + 32 * 32 + 96 * 32 + 32 * 32) / 8.0
    lvl3 = k * (32 * 64 + 64 * 64) / 64.0
    return lvl1 + lvl2 + lvl3


def small_configs_arm(args, ctx):
    """The two small configurations, timed with direct launches and with each fixed-point
    step replayed from a captured HIP graph:
      constant c = 1, 32^3, 10 ppw, 8 poles (eps 0.5), q = 8, FP64, FGMRES(30) to 1e-8;
      GRF medium, 96^3, 10 ppw, 12 poles, 4 Gaussian RHS, plain FP64 and mixed, to 1e-6.
    Every solution's FP64 residual is recomputed by the oracle."""
    import numpy as np
    import torch
    import workloads as W
    from oracle import operator as OO
    from paper_1811_12378_amd import hfci

    def run(wl, J, eps, prec, tol, graphs, reps=3, q=None):
        g = hfci.Operator(ctx, torch.from_numpy(wl.c).cuda(), wl.h, wl.omega, wl.damp_cells, wl.damp_rho2)
        g.autotune(prec, 2)
        c = hfci.Contour(g, J, 1.0, eps, args.q if q is None else q)
        f = torch.from_numpy(np.stack(wl.rhs)).cuda()
        o = hfci.default_opts(precision=prec, tol=tol, max_it=args.max_it, graphs=graphs)
        hfci.solve(g, c, f, opts=o)  # warm-up: workspace, graph instantiation
        torch.cuda.synchronize()
        best = None
        for _ in range(reps):
            t0 = time.perf_counter()
            u, st = hfci.solve(g, c, f, opts=o)
            torch.cuda.synchronize()
            dt = time.perf_counter() - t0
            best = dt if best is None else min(best, dt)
        oo = OO.Operator(wl.c, wl.omega, wl.damp_cells, wl.damp_rho2)
        un = u.cpu().numpy()
        rr = max(float(np.linalg.norm(oo.s * wl.rhs[k] - oo.apply(un[k])) / np.linalg.norm(oo.s * wl.rhs[k]))
                 for k in range(len(wl.rhs)))
        c.close()
        g.close()
        return {"time_s": round(best, 4), "its": st["its"], "relres_oracle": rr}

    out = {}
    w1 = W.config_constant_32()
    # configuration 1 fixes degree 8
    out["constant_32_fp64_tol1e-8"] = {"direct": run(w1, 8, 0.5, 64, 1e-8, 0, q=8),
                                       "graphs": run(w1, 8, 0.5, 64, 1e-8, 1, q=8)}
    w2 = W.config_grf_96()
    out["grf_96_4rhs_fp64"] = {"direct": run(w2, 12, args.eps, 64, args.tol, 0),
                               "graphs": run(w2, 12, args.eps, 64, args.tol, 1, reps=1)}
    out["grf_96_4rhs_mixed"] = {"direct": run(w2, 12, args.eps, 32, args.tol, 0),
                                "graphs": run(w2, 12, args.eps, 32, args.tol, 1, reps=1)}
    for k, v in out.items():
        v["graph_speedup"] = round(v["direct"]["time_s"] / v["graphs"]["time_s"], 3)
        log("%s: direct %.3f s, graphs %.3f s, its %d, oracle relres %.2e"
            % (k, v["direct"]["time_s"], v["graphs"]["time_s"], v["graphs"]["its"], v["graphs"]["relres_oracle"]))
    out["grf_96_speedup_mixed_vs_fp64"] = round(
        min(out["grf_96_4rhs_fp64"]["direct"]["time_s"], out["grf_96_4rhs_fp64"]["graphs"]["time_s"]) /
        min(out["grf_96_4rhs_mixed"]["direct"]["time_s"], out["grf_96_4rhs_mixed"]["graphs"]["time_s"]), 3)
    return out


def uneven_arm(args, ctx, verbose):
    """Config-4 style uneven batch: independent GRF instances of sizes {48,64,96,128}^3 with
    ppw ~ U[6,12] and 8 poles each, solved to the same tolerance as one hfci_solve_batch call
    and one instance at a time; every solution's FP64 residual is recomputed by the oracle."""
    import numpy as np
    import torch
    import workloads as W
    from oracle import operator as OO
    from paper_1811_12378_amd import hfci
    wls = W.config_uneven_batch(count=args.uneven, seed=7)
    t0 = time.perf_counter()
    ops, cons, fs = [], [], []
    for wl in wls:
        g = hfci.Operator(ctx, torch.from_numpy(wl.c).cuda(), wl.h, wl.omega, wl.damp_cells, wl.damp_rho2)
        ops.append(g)
        cons.append(hfci.Contour(g, wl.n_poles, 1.0, args.eps, args.q))
        fs.append(torch.from_numpy(wl.rhs[0]).cuda())
    # a batch shares one degree: where the rule chose (eps, q) per instance, the instances
    # whose q differs from the most common one get eps chosen again for that q
    qs = [c.q for c in cons]
    q_batch = max(set(qs), key=qs.count)
    for k, (g, wl) in enumerate(zip(ops, wls)):
        if cons[k].q != q_batch:
            cons[k].close()
            cons[k] = hfci.Contour(g, wl.n_poles, 1.0, args.eps, q_batch)
    # untimed: every instance gets its autotuned complex64 shape, which the one-at-a-time
    # solves use (the batch launches have their own fixed shape)
    for g in ops:
        g.autotune(32, 2)
    setup_s = time.perf_counter() - t0
    opts = hfci.default_opts(precision=32, tol=args.tol, max_it=args.max_it)
    hfci.solve_batch(ops, cons, fs, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=1))  # allocate
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    us, sts, status = hfci.solve_batch(ops, cons, fs, opts=hfci.default_opts(precision=32, tol=args.tol,
                                                                            max_it=args.max_it, verbose=verbose))
    torch.cuda.synchronize()
    t_batch = time.perf_counter() - t1
    log("uneven batch of %d: %.3f s (%s), its %d..%d" % (len(ops), t_batch, status, min(s["its"] for s in sts),
                                                          max(s["its"] for s in sts)))
    for g, c, f in zip(ops, cons, fs):  # warm the single-instance workspaces
        hfci.solve(g, c, f[None], opts=hfci.default_opts(precision=32, tol=args.tol, max_it=1))
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    seq_its = []
    for k, (g, c, f) in enumerate(zip(ops, cons, fs)):
        _, st = hfci.solve(g, c, f[None], opts=opts)
        seq_its.append(st["its"])
        if k % 8 == 7:
            log("sequential: %d of %d solved" % (k + 1, len(ops)))
    torch.cuda.synchronize()
    t_seq = time.perf_counter() - t2
    log("one instance at a time: %.3f s" % t_seq)
    worst = 0.0
    for wl, u in zip(wls, us):
        o = OO.Operator(wl.c, wl.omega, wl.damp_cells, wl.damp_rho2)
        b = o.s * wl.rhs[0]
        worst = max(worst, float(np.linalg.norm(b - o.apply(u.cpu().numpy())) / np.linalg.norm(b)))
    sizes = {}
    for wl in wls:
        sizes[str(wl.c.shape[0])] = sizes.get(str(wl.c.shape[0]), 0) + 1
    points = sum(int(wl.c.size) for wl in wls)
    eps_used = [round(c.params()["eps"], 4) for c in cons]
    for g, c in zip(ops, cons):
        c.close()
        g.close()
    return {"instances": len(wls), "grid_sizes": sizes, "points": points, "time_batch_s": round(t_batch, 4),
            "q": q_batch, "q_chosen_per_instance": qs, "eps_min": min(eps_used), "eps_max": max(eps_used),
            "time_sequential_s": round(t_seq, 4), "speedup_batch_vs_sequential": round(t_seq / t_batch, 3),
            "its_min": min(s["its"] for s in sts), "its_max": max(s["its"] for s in sts),
            "stencil_products": int(sts[0]["matvecs"] + sum(s["matvecs"] for s in sts[1:])),
            "max_relres_oracle": worst, "status": status, "setup_s": round(setup_s, 2)}


def fp64_arm(args, ctx, op, cont, f_d, wl, t_mixed, verbose):
    """The plain method: the same solve with FP64 shifted sweeps (and FP64 FGMRES)."""
    import torch
    from paper_1811_12378_amd import hfci
    # FP64 sweeps need twice the bytes per shifted system: advance part of the poles at a
    # time once the batch would exceed ~64 GB of iterate storage
    sys_bytes = 3 * 16 * wl.n ** 3 * args.nrhs
    pb = 0 if sys_bytes * args.poles <= 64e9 else max(1, int(64e9 // sys_bytes))
    plain = hfci.default_opts(precision=64, tol=args.tol, max_it=args.max_it, pole_batch=pb, verbose=verbose)
    ctx.profile(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    u64, st64 = hfci.solve(op, cont, f_d, opts=plain)
    torch.cuda.synchronize()
    t64 = time.perf_counter() - t0
    p64 = ctx.profile_read()["fp_stage"]
    ctx.profile(False)
    gbs64 = p64["alg_bytes"] / (p64["total_ms"] * 1e-3) / 1e9 if p64["total_ms"] > 0 else 0.0
    log("plain FP64: %.3f s, its %d, relres %.3e, stage %.0f GB/s" % (t64, st64["its"], st64["final_relres"], gbs64))
    del u64
    return {"time_s": t64, "its": st64["its"], "matvecs": st64["matvecs"], "final_relres": st64["final_relres"],
            "stage_gbs": gbs64, "speedup_mixed_vs_fp64": t64 / t_mixed}


def learned_arm(args, ctx, op, cont, f_d, t_mixed, fp64, verbose):
    """Configuration 5: train the network (untimed) on the remainders FCI leaves on random
    128^3 media (about 2000 pairs from FCI-preconditioned FGMRES, the residual loss), then
    time FGMRES with the network as Alg. 1 step 4's inner preconditioner (k_in = 1: FCI(v)
    plus the best multiple of net(remainder)) on the headline workload, and FCI alone
    against FCI with the network on an unseen 256^3 random-field medium."""
    import torch
    from paper_1811_12378_amd import hfci
    from paper_1811_12378_amd import learned as L
    t0 = time.perf_counter()
    net, info = L.train(ctx, None, n=args.learn_n, media=args.learn_media, pairs=48, steps=args.learn_steps,
                        crop=min(64, args.learn_n))
    train_s = time.perf_counter() - t0
    log("learned: %d remainders at %d^3, harvest %.1f s, training %.1f s, final loss %.4f"
        % (info["pairs"], args.learn_n, info["harvest_s"], info["train_s"], info["final_loss"]))
    # network throughput on the benchmark grid (BF16 MFMA, FP32 accumulate)
    r = torch.randn((1,) + tuple(f_d.shape[1:]), dtype=torch.complex128, device="cuda")
    net.apply(op, r)
    torch.cuda.synchronize()
    reps = 3
    t1 = time.perf_counter()
    for _ in range(reps):
        net.apply(op, r)
    torch.cuda.synchronize()
    t_net = (time.perf_counter() - t1) / reps
    del r
    tflops = unet_flops_per_voxel() * op.n / t_net / 1e12
    lo = hfci.default_opts(precision=32, tol=args.tol, max_it=args.max_it, k_in=1, inner_precond=1, verbose=verbose)
    lo.net = net.h.value
    hfci.solve(op, cont, f_d, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=1, k_in=1, inner_precond=1,
                                                     net=net.h.value))  # untimed: workspace
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    _, st = hfci.solve(op, cont, f_d, opts=lo)
    torch.cuda.synchronize()
    t_l = time.perf_counter() - t2
    log("learned (step 4) + FP32: %.3f s, its %d, relres %.3e" % (t_l, st["its"], st["final_relres"]))
    out = {"mode": "network as Alg. 1 step 4's inner preconditioner (k_in 1)", "time_s": t_l, "its": st["its"],
           "final_relres": st["final_relres"], "train_pairs": info["pairs"], "train_grid": args.learn_n,
           "train_media": args.learn_media, "harvest_s": info["harvest_s"], "train_s": info["train_s"],
           "train_final_loss": info["final_loss"], "speedup_vs_mixed_fci": t_mixed / t_l,
           "net_apply_ms": t_net * 1e3,
           "net_roofline": {"bound": "mfma", "achieved": round(tflops, 1), "peak": 2500.0, "unit": "TFLOP/s",
                            "frac": round(tflops / 2500.0, 4)}}
    if fp64:
        out["speedup_vs_fp64"] = fp64["time_s"] / t_l
    # configuration 5's evaluation: an unseen 256^3 random-field medium, one point source
    g = L.compare(ctx, net, n=args.n, medium="grf", seed=901, tol=args.tol, max_it=args.max_it, mode="step4")
    out["unseen_grf"] = {"workload": g["workload"],
                         "fci": {"time_s": g["fci"]["time_s"], "its": g["fci"]["its"]},
                         "fci_net_step4": {"time_s": g["fci+net_step4"]["time_s"], "its": g["fci+net_step4"]["its"],
                                           "final_relres": g["fci+net_step4"]["final_relres"]}}
    net.close()
    return out


def inner_arm(args, ctx, op, cont, f_d, t_mixed, its_mixed):
    """Alg. 1 step 4 (Sec. 6.3) on the headline solve: the same mixed-precision solve with
    k_in GMRES steps on the remainder, right-preconditioned by the regularised Laplacian
    inverse (three FP64 complex GEMMs per sine transform), for each k_in of --k-in-list."""
    import torch
    from paper_1811_12378_amd import hfci
    out = {"baseline": {"k_in": 0, "time_s": round(t_mixed, 4), "its": its_mixed}, "runs": []}
    for k in args.k_in_list:
        hfci.solve(op, cont, f_d, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=1, k_in=k))  # workspace
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, st = hfci.solve(op, cont, f_d, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=args.max_it,
                                                                 k_in=k))
        torch.cuda.synchronize()
        t = time.perf_counter() - t0
        out["runs"].append({"k_in": k, "time_s": round(t, 4), "its": st["its"], "status": st["status"],
                            "final_relres": st["final_relres"], "speedup_vs_k0": round(t_mixed / t, 3)})
        log("step 4, k_in %d: %.3f s, its %d, relres %.3e" % (k, t, st["its"], st["final_relres"]))
    return out


def params_arm(args, ctx, op, f_d, t_mixed, its_mixed):
    """Contour choices on the headline solve: the degree q chosen by Sec. 4.2's rule (q = 0
    at creation) on the circle (t = 1) and on the paper's ellipse t = 0.1, against the
    headline's q, each a full mixed-precision solve to the headline tolerance."""
    import torch
    from paper_1811_12378_amd import hfci
    out = {"baseline": {"t": 1.0, "q": args.q_used, "time_s": round(t_mixed, 4), "its": its_mixed}, "runs": []}
    for t in (1.0, 0.1):
        c = hfci.Contour(op, args.poles, t, args.eps, 0)
        hfci.solve(op, c, f_d, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=1))
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, st = hfci.solve(op, c, f_d, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=args.max_it))
        torch.cuda.synchronize()
        ts = time.perf_counter() - t0
        nu = c.get()["nu"]
        out["runs"].append({"t": t, "q_chosen": c.q, "time_s": round(ts, 4), "its": st["its"], "status": st["status"],
                            "final_relres": st["final_relres"], "nu_max": round(float(nu.max()), 4)})
        log("contour t %.1f, chosen q %d: %.3f s, its %d" % (t, c.q, ts, st["its"]))
        c.close()
    return out


def spectral_arm(args, ctx):
    """The Fourier-spectral operator (Sec. 7.1) on the layered medium at 256^3 and the paper's
    2.25 points per wavelength (its spectral runs, Table 5(a)): contour J = 16, the headline
    eps, the degree chosen by Sec. 4.2's rule; the mixed-precision solve to the headline
    tolerance, with the oracle's FP64 residual of the returned u."""
    import numpy as np
    import torch
    import workloads as W
    from oracle import spectral as OS
    from paper_1811_12378_amd import hfci
    ppw = args.spectral_ppw
    wl = W.config_layered_256(n=args.n, nrhs=1, ppw=ppw)
    g = hfci.SpectralOperator(ctx, torch.from_numpy(wl.c).cuda(), wl.h, wl.omega, wl.damp_cells, wl.damp_rho2)
    c = hfci.Contour(g, args.poles, 1.0, args.eps, 0)
    f_d = torch.from_numpy(np.stack(wl.rhs)).cuda()
    hfci.solve(g, c, f_d, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=1))  # workspace, FFT plans
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    u, st = hfci.solve(g, c, f_d, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=args.max_it))
    torch.cuda.synchronize()
    t = time.perf_counter() - t0
    o = OS.SpectralOperator(wl.c, wl.omega, wl.damp_cells, wl.damp_rho2, h=wl.h)
    b = o.s * wl.rhs[0]
    ra = float(np.linalg.norm(b - o.apply(u[0].cpu().numpy())) / np.linalg.norm(b))
    info = g.info()
    out = {"ppw": ppw, "omega": wl.omega, "q_chosen": c.q, "box": [info["b1"], info["b2"], info["rho2"]],
           "time_s": round(t, 4), "its": st["its"], "status": st["status"], "stencil_products": st["matvecs"],
           "fp_steps": st["fp_steps"], "final_relres": st["final_relres"], "relres_oracle": ra}
    log("spectral %g ppw: q %d, %.3f s, its %d, products %d, relres %.3e (oracle %.3e)"
        % (ppw, c.q, t, st["its"], st["matvecs"], st["final_relres"], ra))
    c.close()
    g.close()
    return out


def case_two_arm(args, ctx, op, cont, wl, solve=True):
    """Case one versus case two (eq. mat-2x2) on the headline workload: the shifted solves of
    one FCI application, every pole of the same contour construction (eq. quad-points with
    the same J, q and eps for A, eps / 2 for B; delta searched on each operator's own box),
    reducing each residual
    by fp_reduce = 5 from y = 0 with the physical right-hand side (s f for A, [0; s f] for B).
    Reports steps and stencil products per pole, the time of each batch of shifted solves,
    and the case-two kernel's algorithmic bandwidth over its solve (wall clock); with `solve`,
    also the full mixed-precision FGMRES solve on B to the headline tolerance."""
    import numpy as np
    import torch
    from paper_1811_12378_amd import hfci
    info = op.info()
    n = wl.n
    f1 = (info["s"] * torch.from_numpy(wl.rhs[0]).cuda()).to(torch.complex64).reshape(1, n, n, n)
    g2 = op.case_two()
    # near the origin B's eigenvalues are about half of A's (mu = sqrt(a + 1) - 1, the map of
    # eq. shifted-2x2's equivalent shifts), so eps / 2 keeps the same modes inside the contour
    eps1 = cont.params()["eps"]
    eps2 = args.case_two_eps if args.case_two_eps > 0 else eps1 / 2
    c2 = hfci.Contour(g2, args.poles, 1.0, eps2, args.q_used)
    rhs2 = torch.zeros((1, 2, n, n, n), dtype=torch.complex64, device="cuda")
    rhs2[0, 1] = f1[0]
    out = {}
    for name, o_, c_, f_ in (("case_one", op, cont, f1), ("case_two", g2, c2, rhs2)):
        hfci.shifted_solve(o_, c_, f_, steps=1)  # untimed: workspace
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        y, st = hfci.shifted_solve(o_, c_, f_, reduce=5.0, max_steps=400)
        torch.cuda.synchronize()
        t = time.perf_counter() - t0
        steps = [int(v) for v in st[:, 0]]
        cg = c_.get()
        out[name] = {"time_s": round(t, 4), "eps": round(eps1 if name == "case_one" else eps2, 4),
                     "steps_per_pole": steps, "stencil_products": int(args.q_used * sum(steps)),
                     "nu_per_pole": [round(float(v), 4) for v in cg["nu"]],
                     "box": [round(o_.info()["b1"], 4), round(o_.info()["b2"], 4), o_.info()["rho2"]]}
        log("%s: %.3f s, steps per pole %s" % (name, t, steps))
        del y
    # algorithmic bytes of the case-two solve (complex64 blocks, float kappa): a launch of one
    # factor or of a pair reads x (2 x 8 B) and kappa (4 B) and writes 2 x 8 B per grid point;
    # step one runs its q - 1 factors as pairs after a single one when q - 1 is odd, the first
    # launch reading the right-hand side and the last also writing y; a later step runs
    # ceil(q / 2) launches (pairs, then a single for odd q), the first reading g for the
    # residual, the last reading y1
    q, nP = args.q_used, max(args.q_used - 1, 1)
    n1 = nP % 2 + nP // 2 if nP > 1 else 1
    nl = (q + 1) // 2
    per = 0.0
    for m in out["case_two"]["steps_per_pole"]:
        per += n1 * 36 + 16 + max(m - 1, 0) * (nl * 36 + 32) + (36 + 16)
    alg = per * n ** 3
    t2 = out["case_two"]["time_s"]
    out["case_two"]["alg_bytes"] = alg
    out["case_two"]["achieved_gbs_wall"] = round(alg / t2 / 1e9, 1)
    out["case_two"]["kernel"] = ("b2_zm_kernel<float, KIND, NF> (marching in z, no LDS staging; NF = 2 factors "
                                 "per pass, NF = 1 for a lone factor)")
    out["stencil_products_ratio_two_over_one"] = round(out["case_two"]["stencil_products"] /
                                                       max(out["case_one"]["stencil_products"], 1), 3)
    out["time_ratio_two_over_one"] = round(t2 / out["case_one"]["time_s"], 3)
    if solve:
        # end to end: FGMRES(30) with FCI(B) on eq. mat-2x2, mixed precision, to the headline
        # tolerance on the double-size system; u = x2, whose FP64 residual on A the oracle
        # recomputes on the host
        from oracle import operator as OO
        rhs = torch.zeros((1, 2, n, n, n), dtype=torch.complex128, device="cuda")
        rhs[0, 1] = torch.from_numpy(wl.rhs[0]).cuda()
        hfci.solve(g2, c2, rhs, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=1))  # workspace
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        x, st = hfci.solve(g2, c2, rhs, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=args.max_it))
        torch.cuda.synchronize()
        ts = time.perf_counter() - t0
        o = OO.Operator(wl.c, wl.omega, wl.damp_cells, wl.damp_rho2)
        b = o.s * wl.rhs[0]
        u = x[0, 1].cpu().numpy()
        ra = float(np.linalg.norm(b - o.apply(u)) / np.linalg.norm(b))
        out["solve"] = {"time_s": round(ts, 4), "its": st["its"], "status": st["status"],
                        "final_relres_double_size": st["final_relres"], "relres_on_A_oracle": ra,
                        "stencil_products": st["matvecs"]}
        log("case two solve: %.3f s, its %d, relres %.3e (double-size), %.3e on A (oracle)"
            % (ts, st["its"], st["final_relres"], ra))
        del x
    g2.close()
    c2.close()
    return out


class Budget:
    """Wall-clock budget of the whole run, counted from process start.  An arm runs only if
    its estimated duration fits in what is left; otherwise it is recorded as skipped."""

    def __init__(self, total_s):
        self.total = total_s if total_s > 0 else float("inf")

    def left(self):
        return self.total - (time.monotonic() - T_START)

    def fits(self, est_s):
        return est_s <= self.left()


def skipped(est_s, budget):
    return {"skipped": "budget", "estimate_s": round(est_s, 1), "left_s": round(budget.left(), 1)}


def guarded(fn):
    """Run one arm; an exception becomes an error record, so the JSON line is always printed."""
    try:
        return fn()
    except Exception as e:
        log("arm failed: %r" % (e,))
        return {"error": repr(e)}


def add_prof(acc, prof):
    """Sum two hfci_ctx_profile_read results class by class."""
    if acc is None:
        return prof
    return {k: {f: acc[k][f] + prof[k][f] for f in ("launches", "total_ms", "alg_bytes")} for k in acc}


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1, help="timed solves (a cap under --budget)")
    ap.add_argument("--warmup", type=int, default=0, help="untimed full solves first (a cap under --budget)")
    ap.add_argument("--budget", type=float, default=450.0,
                    help="wall-clock budget of the run in seconds from process start (0: none); arms and extra "
                         "steps whose estimate does not fit are skipped and recorded as such")
    ap.add_argument("--n", type=int, default=256)
    ap.add_argument("--nrhs", type=int, default=8)
    ap.add_argument("--poles", type=int, default=16)
    ap.add_argument("--eps", type=float, default=0.0,
                    help="contour eps (default 0: chosen by the library's rule for the operator's box and grid)")
    ap.add_argument("--q", type=int, default=0,
                    help="degree of the exponential-Taylor polynomial (default 0: chosen by the library, Sec. 4.2's "
                         "rule counted in passes of two factors)")
    ap.add_argument("--ppw", type=float, default=8.0)
    ap.add_argument("--tol", type=float, default=1e-6)
    ap.add_argument("--max-it", type=int, default=1000)
    ap.add_argument("--no-fp64", action="store_true", help="skip the plain FP64 comparison solve")
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle CPU baseline")
    ap.add_argument("--cpu-full", action="store_true",
                    help="also time a complete FP64 oracle solve at 32^3 (and the 96^3 per-product time)")
    ap.add_argument("--quiet", action="store_true", help="no per-cycle progress lines from the solver")
    ap.add_argument("--no-learned", action="store_true", help="skip the learned-preconditioner arm")
    ap.add_argument("--learn-n", type=int, default=128, help="training grid of the learned arm")
    ap.add_argument("--learn-media", type=int, default=42,
                    help="training media of the learned arm (48 remainders each)")
    ap.add_argument("--learn-steps", type=int, default=4000, help="Adam steps for the learned arm")
    ap.add_argument("--learn-est", type=float, default=110.0,
                    help="estimated seconds of the learned arm besides its headline solve (harvesting, "
                         "training, the unseen-medium comparison; budget check)")
    ap.add_argument("--uneven", type=int, default=0,
                    help="instances of the uneven-batch arm (64 = the full config; 0 skips it)")
    ap.add_argument("--uneven-only", action="store_true", help="run only the uneven-batch arm")
    ap.add_argument("--small", action="store_true", help="also run the 32^3 / 96^3 configurations")
    ap.add_argument("--case-two", action="store_true", help="also run the case-one versus case-two arm")
    ap.add_argument("--k-in-list", type=int, nargs="*", default=[],
                    help="k_in values of the Alg. 1 step 4 arm (none: the arm is skipped)")
    ap.add_argument("--inner-only", action="store_true",
                    help="run only the headline solve and the Alg. 1 step 4 arm")
    ap.add_argument("--spectral", action="store_true", help="also run the Fourier-spectral arm")
    ap.add_argument("--spectral-only", action="store_true", help="run only the Fourier-spectral arm")
    ap.add_argument("--spectral-ppw", type=float, default=2.25, help="points per wavelength of the spectral arm")
    ap.add_argument("--params", action="store_true",
                    help="also run the contour-choice arm (chosen q, ellipse t = 0.1)")
    ap.add_argument("--case-two-eps", type=float, default=0.0,
                    help="contour eps of the case-two arm (0: half the headline eps)")
    ap.add_argument("--case-two-only", action="store_true",
                    help="run only the case-one versus case-two shifted solves at the headline workload")
    ap.add_argument("--small-only", action="store_true", help="run only the 32^3 / 96^3 configurations")
    ap.add_argument("--profile-every", type=int, default=PROFILE_EVERY,
                    help="time every k-th launch of each kernel class in the timed solves")
    ap.add_argument("--shape", type=int, nargs="+", metavar="V",
                    help="pin the complex64 stencil launch shape instead of autotuning it")
    args = ap.parse_args()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py runs on exactly one GPU: the multi-GPU (pole-parallel) layout is not "
              "implemented; rerun with --gpus 1", file=sys.stderr)
        sys.exit(2)
    budget = Budget(args.budget)

    import numpy as np
    import torch

    import workloads as W
    from paper_1811_12378_amd import hfci

    if args.inner_only:
        args.no_fp64 = args.no_learned = args.no_cpu = True
        args.small = args.case_two = False
        args.uneven = 0
        if not args.k_in_list:
            args.k_in_list = [2, 4]
    hfci.load_library()
    assert torch.cuda.is_available(), "bench.py needs a GPU"
    verbose = 0 if args.quiet else 1
    if args.small_only:
        ctx = hfci.Context(0)
        r = small_configs_arm(args, ctx)
        print(json.dumps({"metric": "small configurations", "small_configs": r}), flush=True)
        return
    if args.spectral_only:
        ctx = hfci.Context(0)
        r = spectral_arm(args, ctx)
        print(json.dumps({"metric": "spectral time-to-%g (s)" % args.tol, "value": r["time_s"], "unit": "s",
                          "n_gpus": 1, "higher_is_better": False, "dtype": "f32+f64", "data": "synthetic",
                          "config": {"workload": "layered medium %d^3, Fourier-spectral, %g ppw" % (args.n, r["ppw"])},
                          "spectral": r}), flush=True)
        return
    if args.uneven_only:
        ctx = hfci.Context(0)
        r = uneven_arm(args, ctx, verbose)
        print(json.dumps({"metric": "uneven batch time-to-%g (s)" % args.tol, "value": r["time_batch_s"],
                          "unit": "s", "n_gpus": 1, "higher_is_better": False, "dtype": "f32+f64",
                          "data": "synthetic", "config": {"workload": "uneven GRF batch"}, "uneven": r}),
              flush=True)
        return
    wl = W.config_layered_256(n=args.n, nrhs=args.nrhs, ppw=args.ppw)
    log("workload %s: omega %.3f, c in [%.3f, %.3f] (%.1f s since start)"
        % (wl.name, wl.omega, wl.c.min(), wl.c.max(), time.monotonic() - T_START))
    ctx = hfci.Context(0)
    c_d = torch.from_numpy(wl.c).cuda()
    f_d = torch.from_numpy(np.stack(wl.rhs)).cuda()
    op = hfci.Operator(ctx, c_d, wl.h, wl.omega, wl.damp_cells, wl.damp_rho2)
    cont = hfci.Contour(op, args.poles, 1.0, args.eps, args.q)
    eps_used = cont.params()["eps"]  # the library's rule chooses it for --eps 0
    args.q_used = cont.q  # and the degree for --q 0 (Sec. 4.2's rule, in passes of two factors)
    info = op.info()
    log("operator:", info)

    # untimed setup: the library's autotuner picks the stencil launch shape per precision,
    # timed over about as many systems as a launch of the solve carries late in an FCI
    # application (about two per right-hand side: the slow poles)
    tune_sys = max(2, min(16, 2 * args.nrhs))
    if args.shape:
        op.set_tune(32, *args.shape)
        tune32 = op.get_tune(32)
        log("complex64 shape pinned to", tune32)
    else:
        tune32, rows32 = op.autotune(32, tune_sys)
        log("autotuned complex64 shape %s over %d systems (%.3f ms)" % (tune32, tune_sys,
                                                                      min(r[1] for r in rows32)))
    if args.case_two_only:
        r = case_two_arm(args, ctx, op, cont, wl)
        print(json.dumps({"metric": "shifted solves of one FCI application, case one vs case two (s)",
                          "value": r["case_two"]["time_s"], "unit": "s", "n_gpus": 1, "higher_is_better": False,
                          "dtype": "c64", "data": "synthetic", "config": {"workload": wl.name}, "case_two": r}),
              flush=True)
        return
    tune64, rows64 = op.autotune(64, tune_sys)
    log("autotuned complex128 shape %s (%.3f ms)" % (tune64, min(r[1] for r in rows64)))
    mixed = hfci.default_opts(precision=32, tol=args.tol, max_it=args.max_it, verbose=verbose)
    # untimed setup: one Arnoldi step launches every kernel of the solve and allocates every
    # workspace buffer, so the first timed solve pays no first-use cost
    hfci.solve(op, cont, f_d, opts=hfci.default_opts(precision=32, tol=args.tol, max_it=1))
    torch.cuda.synchronize()
    log("setup done at %.1f s" % (time.monotonic() - T_START))

    # roofline of the dominant kernel: HIP events on the library's stream bracket every k-th
    # launch of each kernel class inside the timed solves (k = 1 for the counter runs, whose
    # counters cover every dispatch)
    times, st, u, prof = [], None, None, None
    skip = {}

    def timed_solve():
        nonlocal st, u, prof
        ctx.profile(True, every=args.profile_every)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        u, st = hfci.solve(op, cont, f_d, opts=mixed)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
        prof = add_prof(prof, ctx.profile_read())
        ctx.profile(False)
        log("timed step %d: %.3f s, its %d, relres %.3e, matvecs %d (%.1f s since start)"
            % (len(times) - 1, times[-1], st["its"], st["final_relres"], st["matvecs"], time.monotonic() - T_START))

    # warm-up full solves are run only if, after them, the first timed solve and the
    # metric's other arms would still fit; the solve time is not known before the first
    # one, so a warm-up needs the budget to be unbounded
    warm_done = 0
    if args.warmup > 0 and budget.total == float("inf"):
        for w in range(args.warmup):
            hfci.solve(op, cont, f_d, opts=mixed)
            warm_done += 1
            log("warmup %d done" % w)
    elif args.warmup > 0:
        skip["warmup"] = ("%d warm-up solves not run: the untimed setup above (autotuning and one "
                          "Arnoldi step) already launched every kernel and allocated every buffer, and "
                          "a full warm-up solve would not leave room in the %.0f s budget" % (args.warmup,
                                                                                             budget.total))
    timed_solve()
    t1 = times[0]

    # independent residual check of the first solution with the FP64 oracle on the host
    from oracle import operator as OO
    o = OO.Operator(wl.c, wl.omega, wl.damp_cells, wl.damp_rho2)
    u0 = u[0].cpu().numpy()
    b = o.s * wl.rhs[0]
    relres_oracle = float(np.linalg.norm(b - o.apply(u0)) / np.linalg.norm(b))
    log("oracle FP64 relative residual of rhs 0: %.3e" % relres_oracle)
    st_first = dict(st)

    cpu = None
    if not args.no_cpu:
        est = 35.0
        if budget.fits(est):
            try:
                from oracle import fci as OF
                poles_o = OF.pole_parameters(o, args.poles, 1.0, eps_used, args.q_used)
                cpu = cpu_baseline(wl, poles_o, st_first["matvecs"])
                if args.cpu_full:
                    cpu["full_solves"] = cpu_full_solves(args)
                log("cpu baseline:", cpu["sample"])
            except Exception as e:  # the JSON line is printed whatever an arm does
                cpu = {"error": repr(e)}
        else:
            cpu = skipped(est, budget)

    fp64 = None
    if not args.no_fp64:
        est = 2.0 * t1 + 10.0
        if budget.fits(est):
            fp64 = guarded(lambda: fp64_arm(args, ctx, op, cont, f_d, wl, t1, verbose))
        else:
            fp64 = skipped(est, budget)

    learned = None
    if not args.no_learned:
        est = args.learn_est + 1.5 * t1
        if budget.fits(est):
            learned = guarded(lambda: learned_arm(args, ctx, op, cont, f_d, t1,
                                                  fp64 if fp64 and "time_s" in fp64 else None, verbose))
        else:
            learned = skipped(est, budget)

    optional = {}
    for name, flag, fn in (
            ("small_configs", args.small, lambda: small_configs_arm(args, ctx)),
            ("uneven_batch", args.uneven > 0, lambda: uneven_arm(args, ctx, verbose)),
            ("inner_step4", bool(args.k_in_list), lambda: inner_arm(args, ctx, op, cont, f_d, t1, st_first["its"])),
            ("spectral", args.spectral, lambda: spectral_arm(args, ctx)),
            ("contour_choice", args.params, lambda: params_arm(args, ctx, op, f_d, t1, st_first["its"])),
            ("case_two", args.case_two, lambda: case_two_arm(args, ctx, op, cont, wl))):
        if flag:
            optional[name] = guarded(fn)

    # further timed solves while the budget lasts (capped by --steps)
    while len(times) < args.steps:
        est = 1.15 * max(times) + 5.0
        if not budget.fits(est):
            skip["steps"] = ("%d of %d requested timed solves run: the next (about %.0f s) would not fit in "
                             "the %.0f s left of the budget" % (len(times), args.steps, est, budget.left()))
            break
        timed_solve()
    t_mixed = sum(times) / len(times)

    # the dominant middle kernel: the three-factor passes where they took more time than the
    # middle pairs (shapes with fuse 2), else the middle pairs
    triple = prof["fp_stage_triple"]["total_ms"] > prof["fp_stage"]["total_ms"]
    stage = prof["fp_stage_triple" if triple else "fp_stage"]
    avg_ms = stage["total_ms"] / max(stage["launches"], 1)
    bytes_per_launch = stage["alg_bytes"] / max(stage["launches"], 1)
    achieved = bytes_per_launch / (avg_ms * 1e-3) / 1e9 if avg_ms > 0 else 0.0
    traffic_ratio = measured_traffic(tune32, traffic_kernel(tune32, triple))
    # the counter runs are short solves: their launches cover a different mix of active
    # systems, so the measured bytes are carried over as a ratio to the algorithmic bytes
    traffic = round(traffic_ratio * bytes_per_launch, 0) if traffic_ratio else None

    def gbs(cls):
        p = prof[cls]
        return round(p["alg_bytes"] / (p["total_ms"] * 1e-3) / 1e9, 1) if p["total_ms"] > 0 else 0.0

    other_gbs = {k: gbs(k) for k in ("fp_stage", "fp_stage_triple", "fp_stage_first", "fp_stage_last",
                                      "fp_stage_init") if k != ("fp_stage_triple" if triple else "fp_stage")}
    launch_ms = {k: round(prof[k]["total_ms"], 1) for k in ("fp_stage", "fp_stage_triple", "fp_stage_first",
                                                             "fp_stage_last", "fp_stage_init")}
    if fp64 and "time_s" in fp64:
        fp64["speedup_mixed_vs_fp64"] = fp64["time_s"] / t_mixed

    out = {
        "metric": METRIC,
        "value": round(t_mixed, 4),
        "unit": "s",
        "n_gpus": 1,
        "steps": len(times),
        "warmup": warm_done,
        "steps_requested": args.steps,
        "warmup_requested": args.warmup,
        "ms_per_step": round(t_mixed * 1e3, 2),
        "step_times_s": [round(t, 3) for t in times],
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32+f64",
        "data": "synthetic",
        "config": {"workload": "layered medium %d^3, %d point sources, %d poles, q=%d, %g ppw, tol %g, "
                               "FP32 shifted sweeps + FP64 FGMRES(30)"
                               % (args.n, args.nrhs, args.poles, args.q_used, args.ppw, args.tol),
                   "grid": args.n, "rhs": args.nrhs, "poles": args.poles, "q": args.q_used, "eps": round(eps_used, 4),
                   "ppw": args.ppw, "tol": args.tol, "stencil_shape_c64": list(tune32),
                   "stencil_shape_c128": list(tune64)},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4),
                     "traffic": traffic, "traffic_over_alg": round(traffic_ratio, 4) if traffic_ratio else None,
                     "kernel": middle_kernel_name(tune32, triple),
                     "avg_launch_ms": round(avg_ms, 4), "alg_bytes_per_launch": bytes_per_launch,
                     "launches": stage["launches"], "timed_every": args.profile_every},
        "cpu_baseline": cpu,
        "its": st_first["its"],
        "matvecs": st_first["matvecs"],
        "matvecs_per_s": round(st_first["matvecs"] / t1, 1),
        "final_relres": st_first["final_relres"],
        "relres_oracle_rhs0": relres_oracle,
        "factor_kernels_gbs": other_gbs,
        "factor_kernels_timed_ms": launch_ms,
        "fp64": fp64,
        "learned": learned,
        "budget_s": args.budget,
        "run_s": round(time.monotonic() - T_START, 1),
        "not_run": skip or None,
    }
    out.update(optional)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
