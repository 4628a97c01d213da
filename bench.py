"""Benchmark of the hot path: wave-LB steps with per-step surface force.

Workload (one GPU): the 3D sphere, FP32 storage, 256 x 128 x 128 D3Q7,
lambda = 256, c0 = 0.5, c_p/c0 = 1.1, R = 12, 2048 surface points, with the
16 positions kh_j = j (pi/2)/15 run together in one handle (16 instances of
4.19 M cells).  A step advances all 16 boxes by one time step and measures
F(t) on every sphere.  The default K = 15360 steps is one full run (30 drive
periods, average over the last 10) and so yields the 16 time-averaged forces.

Prints one JSON line (see the keys below).  `roofline` reports the dominant
kernel (the fused step kernel): algorithmic bytes per launch, 2 Q s bytes per
cell update, divided by its average duration measured with HIP events on the
handle's stream; `cpu_baseline` times the FP64 oracle on the host cores on a
bounded sample of the same workload.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = ("wave-LB MLUPS & % HBM roofline; forces/s plain vs batched/surrogate at "
          "≤2% error")
HBM_PEAK_GBS = 8000.0
BF16_PEAK_TFLOPS = 2500.0  # dense MFMA
SHAPE = (256, 128, 128)
LAM, C0, CP_RATIO, RADIUS, NSURF = 256.0, 0.5, 1.1, 12.0, 2048
N_POS = 16


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=15360)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--storage", default="f32", choices=["f32", "f16", "bf16"])
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-surrogate", action="store_true",
                    help="skip training and timing the force surrogate")
    ap.add_argument("--surrogate-batch", type=int, default=1 << 20)
    ap.add_argument("--surrogate-steps", type=int, default=16000,
                    help="Adam steps of the surrogate's training (0: time the untrained network)")
    ap.add_argument("--cpu-steps", type=int, default=800)
    ap.add_argument("--variant", default=None,
                    help="kernel variant 'cells_per_lane,x_mode,nontemporal[,steps_per_launch]' "
                         "(skips autotune)")
    ap.add_argument("--workload", default="sphere",
                    choices=["sphere", "batch", "surrogate", "cylinder"],
                    help="sphere: the 16-position 3D sphere (default); batch: the seeded uneven "
                         "batch of boxes (forces/s batched vs plain); surrogate: the force "
                         "network alone (training, held-out error, inference rate); cylinder: "
                         "the 2D FP64 cylinder, alone and as a batch of positions")
    ap.add_argument("--batch-seed", type=int, default=2404)
    ap.add_argument("--batch-n", type=int, default=256,
                    help="boxes of the uneven batch (--workload batch)")
    ap.add_argument("--batch-subset", type=int, default=32,
                    help="boxes of the uneven batch (its first draws) timed in the default run")
    ap.add_argument("--no-batch", action="store_true",
                    help="skip the uneven-batch leg of the default run")
    ap.add_argument("--no-cylinder", action="store_true",
                    help="skip the 2D cylinder leg of the default run")
    ap.add_argument("--fallback-sample", type=int, default=4,
                    help="seeded queries outside the surrogate's box answered by the LB fallback "
                         "in this run, for the blended forces/s over the whole input box")
    ap.add_argument("--lb-sample", type=int, default=32,
                    help="draws of the surrogate's training generator run as one batched LB "
                         "handle in this run, for the surrogate's gain over the batched LB")
    ap.add_argument("--graph", type=int, default=64,
                    help="replay steady steps as captured HIP graphs of this many steps (0 = off)")
    ap.add_argument("--kernel-only", action="store_true",
                    help="time only the step kernel (no surface) and the copy reference; for "
                         "counter runs")
    return ap.parse_args()


def problems(x_mid, k, with_surface=True):
    import workloads
    out = []
    for kh in workloads.sphere_3d_positions(N_POS):
        p = workloads.sphere_3d(x_mid, k, kh, shape=SHAPE, lam=LAM, R=RADIUS,
                                cp_ratio=CP_RATIO, n_surf=NSURF, c0=C0)
        if not with_surface:
            for key in ("surf_xyz", "surf_normal", "surf_area"):
                p.pop(key)
        out.append(p)
    return out


def kernel_source_sha():
    h = hashlib.sha256()
    for f in ("lb_kernels.hpp",):
        with open(os.path.join(ROOT, "paper_2404_02346_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def set_variant(h, v):
    """Apply (cells_per_lane, x_mode, nontemporal, steps_per_launch) to a handle."""
    h.set_steps_per_launch(v[3])
    h.set_variant(*v[:3])


def get_variant(h):
    return tuple(h.variant()) + (h.steps_per_launch(),)


def kernel_name(storage, v, plan):
    if v[3] == 2:
        return "march_kernel<{},steps={},waves={},nt={}>".format(storage, *plan, min(v[2], 1))
    return "step_kernel<3,{},{},{},{}>".format(storage, *v[:3])


def measured_traffic(storage, variant, plan):
    """HBM bytes per launch from the committed counter summary, if current."""
    path = os.path.join(ROOT, "profiles", f"march_kernel_sphere16_{storage}_traffic.json")
    try:
        with open(path) as fh:
            d = json.load(fh)
    except OSError:
        return None
    if (d.get("kernel_source_sha") != kernel_source_sha()
            or tuple(d.get("variant", ())) != tuple(variant) or tuple(d.get("plan", ())) != tuple(plan)):
        return None
    return d.get("hbm_bytes_per_launch")


def cpu_baseline(x_mid, k, n_steps):
    """The FP64 oracle on the host cores, one position for n_steps steps."""
    import oracle
    p = problems(x_mid, k)[7]
    t0 = time.perf_counter()
    oracle.run(p, n_steps)
    dt = time.perf_counter() - t0
    cells = SHAPE[0] * SHAPE[1] * SHAPE[2]
    try:
        cores = len(os.sched_getaffinity(0))
    except AttributeError:
        cores = os.cpu_count()
    omp = os.environ.get("OMP_NUM_THREADS")
    if omp and omp.isdigit():
        cores = min(cores, int(omp))
    return {"value": cells * n_steps / dt / 1e6, "unit": "MLUPS", "cores": cores,
            "kind": "oracle",
            "sample": f"FP64 oracle, position kh_7 of 16, {n_steps} of 15360 steps on the full "
                      f"256x128x128 lattice with surface measurement ({dt:.1f} s)"}


def lb_sample_rate(n, graph):
    """Forces/s of the batched LB on the first n draws of the surrogate's training generator
    (seed 2405, k R <= 0.6), run to completion in one handle in this run.  The forces must
    equal the stored training forces of the same draws bit for bit."""
    from paper_2404_02346_amd import surrogate as S
    d = S.generate(2405, n, verbose=False)
    stored = S.load_sets(S.TRAIN_FILES[:1])[0]["rows"][:n]
    same = all(a["F"] == b["F"] for a, b in zip(d["rows"], stored))
    return {"forces_per_s": round(n / d["lb_seconds"], 3), "boxes": n,
            "seconds": round(d["lb_seconds"], 2), "updates": d["lb_updates"],
            "forces_equal_stored_training_data": bool(same),
            "boxes_by_edge": {str(e): sum(1 for r in d["rows"] if r["edge"] == e)
                              for e in (64, 96, 128, 192)}}


def fallback_rate(net, n, seed=2410):
    """n seeded queries just outside the trained box (c_p/c0 in (1.5, 1.6], the rest uniform over
    the box), answered by the surrogate's LB fallback in one batched handle (boxes lambda x 64 x
    64) in this run: forces/s."""
    import torch
    from paper_2404_02346_amd import surrogate as S
    q = np.random.Generator(np.random.PCG64(seed))
    kr, kh = q.uniform(*S.BOX["kR"], n), q.uniform(*S.BOX["kh"], n)
    ra, R = q.uniform(1.5, 1.6, n) + 1e-9, q.uniform(4.0, 16.0, n)
    sur = S.Surrogate(net)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    F, used = sur.predict(kr, kh, ra, R)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    lam = np.rint(2 * math.pi * R / kr)
    return {"queries": int(n), "seconds": round(dt, 2), "forces_per_s": round(n / dt, 4),
            "all_used_lb": bool(used.all()), "box_lengths": [int(v) for v in lam],
            "finite": bool(np.isfinite(F).all()),
            "sample": f"{n} seeded draws (seed {seed}): c_p/c0 in (1.5, 1.6], kR, kh, R uniform "
                      "over the box"}


def surrogate_leg(stream, batch, steps=16000, lb_sample=32, graph=64, fallback_sample=0):
    """Train the surrogate on the LB data, score it held out, time its fused inference, and
    time the batched LB on a sample of the same generator for the comparison."""
    import torch
    from paper_2404_02346_amd import surrogate as S
    if not all(os.path.exists(f) for f in S.data_paths(S.TRAIN_FILES + S.TEST_FILES)):
        return None
    train_sets = S.load_sets(S.TRAIN_FILES)
    if steps > 0:
        net, log, train_s = S.fit(train_sets, steps=steps)
    else:  # untrained network: the inference kernel's speed does not depend on the weights
        net, log, train_s = S.MLP(max_batch=1024, seed=0), [(0, float("nan"))], 0.0
    te = S.table(*S.load_sets(S.TEST_FILES))
    err = S.error_metric(net.predict(S.normalize(*te[:4])), te[4])
    # share of queries the network hands to the LB: seeded draws over the whole input box
    qrng = np.random.Generator(np.random.PCG64(2407))
    nq = 100000
    qkr = qrng.uniform(*S.BOX["kR"], nq)
    qkh = qrng.uniform(*S.BOX["kh"], nq)
    qra = qrng.uniform(*S.BOX["ratio"], nq)
    qR = qrng.uniform(4.0, 16.0, nq)
    fallback = float(1.0 - S.in_box(qkr, qkh, qra, qR).mean())
    fb = fallback_rate(net, fallback_sample) if fallback_sample > 0 else None
    x = torch.rand(batch, S.N_IN, device="cuda") * 2 - 1
    y = torch.empty(batch, device="cuda")
    for _ in range(3):
        net.forward_dev(x, y, batch)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    n = 20
    e0.record(stream)
    for _ in range(n):
        net.forward_dev(x, y, batch)
    e1.record(stream)
    e1.synchronize()
    ms = e0.elapsed_time(e1) / n
    net.close()
    d = S.DIMS
    flop = 2 * sum(d[i] * d[i + 1] for i in range(len(d) - 1))  # per sample
    tflops = flop * batch / (ms * 1e-3) / 1e12
    n_lb = sum(t["n"] for t in train_sets)
    lb_s = sum(t["lb_seconds"] for t in train_sets)
    lb_run = lb_sample_rate(lb_sample, graph) if lb_sample > 0 else None
    out = {
        "forces_per_s": round(batch / (ms * 1e-3), 1),
        "held_out_error": {k: (round(v, 5) if isinstance(v, float) else v)
                           for k, v in err.items()},
        "fallback_fraction": {
            "value": round(fallback, 4),
            "queries": f"{nq} seeded draws (seed 2407), uniform over kR [0.05, 0.6], kh [0, pi/2], "
                       "c_p/c0 [0.8, 1.5], R [4, 16] cells; those outside the trained box go to "
                       "the LB"},
        "test_samples": len(te[0]), "train_samples": n_lb,
        "train_seconds": round(train_s, 2), "train_final_loss": log[-1][1],
        "lb_seconds_for_training_data": round(lb_s, 1),
        "inference": {"kernel": "infer_kernel (fused 4-256-256-256-256-1, BF16 MFMA)",
                      "batch": batch, "ms": round(ms, 4), "flop_per_sample": flop,
                      "tflops": round(tflops, 1),
                      "frac_of_bf16_peak": round(tflops / BF16_PEAK_TFLOPS, 4)},
        # the training data's own generation time (an earlier run, stored with the data)
        "training_data_lb_forces_per_s": round(n_lb / lb_s, 3),
    }
    if lb_run is not None:
        out["batched_lb_this_run"] = lb_run
        out["gain_over_batched_lb"] = round(batch / (ms * 1e-3) / lb_run["forces_per_s"], 1)
    if fb is not None:
        # a query stream uniform over the whole input box: the fraction outside the trained box
        # costs the LB fallback's time per force, the rest the network's
        nn = batch / (ms * 1e-3)
        out["fallback_lb_this_run"] = fb
        out["blended_forces_per_s_whole_box"] = round(
            1.0 / (fallback / fb["forces_per_s"] + (1.0 - fallback) / nn), 1)
    return out


def batch_leg(args, n, stream):
    """The first n boxes of the seeded uneven batch: every box to its own length in one handle,
    against the same boxes one at a time (measured single-box step time per box edge)."""
    import torch
    import paper_2404_02346_amd as P
    import workloads
    from paper_2404_02346_amd import surrogate as S
    cal = S.calibrate_edges(workloads.BATCH_EDGES)
    probs, info = workloads.batch(args.batch_seed, n,
                                  {e: c["x_mid"] for e, c in cal.items()},
                                  {e: c["k"] for e, c in cal.items()}, return_draws=True)
    r = S.run_batch(probs, storage=args.storage, graph=args.graph)
    # plain: each instance alone on the GPU, step time measured per box edge
    plain_s, per_edge = 0.0, {}
    for e in sorted({int(p["nx"]) for p in probs}):
        group = [p for p in probs if int(p["nx"]) == e]
        h = P.LBWave([group[0]], storage=args.storage, stream=stream)
        h.autotune(4)
        h.set_graph(args.graph)
        h.step(2 * args.graph + 10)  # past the first graph capture
        torch.cuda.synchronize()
        n1 = 300
        t0 = time.perf_counter()
        h.step(n1)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) / n1 * 1e3
        h.close()
        per_edge[e] = ms
        plain_s += ms * 1e-3 * sum(int(p["n_steps"]) for p in group)
    return {
        "boxes": len(probs), "seed": args.batch_seed, "updates": r["updates"],
        "rejected_draws": info["rejected"], "kernel_variant": r["variant"],
        "boxes_by_edge": {str(e): sum(1 for p in probs if int(p["nx"]) == e)
                          for e in workloads.BATCH_EDGES},
        "batched_seconds": round(r["seconds"], 3), "plain_seconds_estimated": round(plain_s, 3),
        "mlups": round(r["updates"] / r["seconds"] / 1e6, 1),
        "forces_per_s": {"batched": round(len(probs) / r["seconds"], 3),
                         "plain_one_at_a_time": round(len(probs) / plain_s, 3),
                         "batched_over_plain": round(plain_s / r["seconds"], 3)},
        "plain_ms_per_step_by_edge": {str(k): round(v, 4) for k, v in per_edge.items()},
        "forces_x": [float(v) for v in r["F"][:, 0]],
    }


def batch_workload(args):
    """The uneven batch: every instance to its own length in one handle, vs one at a time."""
    import torch
    torch.cuda.set_device(0)
    leg = batch_leg(args, args.batch_n, torch.cuda.current_stream())
    n = leg["boxes"]
    steps = max(90 * int(e) for e, c in leg["boxes_by_edge"].items() if c)
    out = {
        "metric": METRIC, "value": leg["mlups"], "unit": "MLUPS",
        "n_gpus": 1, "steps": steps, "warmup": 0,
        "ms_per_step": round(leg["batched_seconds"] / steps * 1e3, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": args.storage, "data": "synthetic",
        "config": {"workload": f"uneven batch: {n} seeded cubic boxes (seed {args.batch_seed}), "
                               "edge in {64,96,128,192} = lambda, R~U[4,16], c_p/c0~U[0.8,1.5], "
                               "kh~U[0,pi/2], c0=1/3, 30 periods each (last 10 averaged), one "
                               "handle, graph-replayed steps",
                   "instances": n, "updates": leg["updates"],
                   "rejected_draws": leg["rejected_draws"],
                   "kernel_variant": leg["kernel_variant"], "graph_chunk": args.graph},
        "forces_per_s": leg["forces_per_s"],
        "batched_seconds": leg["batched_seconds"],
        "plain_seconds_estimated": leg["plain_seconds_estimated"],
        "plain_ms_per_step_by_edge": leg["plain_ms_per_step_by_edge"],
        "forces_x": leg["forces_x"],
    }
    print(json.dumps(out), flush=True)


def cylinder_leg(args, with_oracle):
    """The 2D FP64 cylinder (128 x 64 D2Q5, 5120 steps): one box alone, then 64 positions in one
    handle; the single box's force against the oracle's (the oracle runs on the host cores)."""
    import torch
    import paper_2404_02346_amd as P
    import workloads
    lam, c0 = 128.0, 0.5
    cal = P.cavity_calibrate(128, c0, 2 * math.pi * c0 / lam)
    p = workloads.cylinder_2d(cal["x_mid"], cal["k"])
    n_steps, cells = int(p["n_steps"]), 128 * 64
    out = {"dtype": "f64",
           "config": {"workload": "2D cylinder, D2Q5 128x64, lambda=128, c0=0.5, c_p/c0=1.2, R=8, "
                                  "64 surface points, kh=pi/4, 20 periods (5120 steps), average "
                                  "over the last 5"}}
    for n_inst in (1, 64):
        probs = [p] if n_inst == 1 else [
            workloads.cylinder_2d(cal["x_mid"], cal["k"], kh=j * (math.pi / 2) / (n_inst - 1))
            for j in range(n_inst)]
        h = P.LBWave(probs, storage="f64")
        h.autotune(4)
        h.set_graph(args.graph)
        h.step(2 * args.graph + 10)  # past the first graph capture
        h.reset()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        h.step(n_steps)
        F, _ = h.force()
        dt = time.perf_counter() - t0
        h.close()
        key = "single" if n_inst == 1 else f"batch_{n_inst}"
        out[key] = {"seconds": round(dt, 4), "ms_per_step": round(dt / n_steps * 1e3, 5),
                    "mlups": round(n_inst * cells * n_steps / dt / 1e6, 1),
                    "forces_per_s": round(n_inst / dt, 2)}
        if n_inst == 1:
            out["force_x"] = float(F[0, 0])
    if with_oracle:
        import oracle
        t0 = time.perf_counter()
        ref = oracle.run(p, n_steps)
        dt = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(cells * n_steps / dt / 1e6, 1), "unit": "MLUPS",
                               "kind": "oracle", "sample": "the whole 5120-step run",
                               "force_x": float(ref["F_avg"][0]),
                               "gpu_vs_oracle_rel": abs(out["force_x"] / ref["F_avg"][0] - 1)}
    return out


def cylinder_workload(args):
    import torch
    torch.cuda.set_device(0)
    print(json.dumps({"mode": "cylinder", **cylinder_leg(args, not args.no_cpu_baseline)}),
          flush=True)


def main():
    args = parse()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py runs on one GPU only: the library has no multi-GPU path "
              "(the batched instances would shard by instance; see the design notes)",
              file=sys.stderr)
        sys.exit(2)
    if args.workload == "batch":
        batch_workload(args)
        return
    if args.workload == "cylinder":
        cylinder_workload(args)
        return
    if args.workload == "surrogate":
        import torch
        torch.cuda.set_device(0)
        sur = surrogate_leg(torch.cuda.current_stream(), args.surrogate_batch, args.surrogate_steps,
                            args.lb_sample, args.graph, args.fallback_sample)
        print(json.dumps({"mode": "surrogate", **(sur or {})}), flush=True)
        return
    import torch
    import paper_2404_02346_amd as P
    import workloads  # noqa: F401

    torch.cuda.set_device(0)
    stream = torch.cuda.current_stream()
    omega = 2 * math.pi * C0 / LAM
    cal = P.cavity_calibrate(SHAPE[0], C0, omega)
    x_mid, k = cal["x_mid"], cal["k"]
    probs = problems(x_mid, k)
    cells = N_POS * SHAPE[0] * SHAPE[1] * SHAPE[2]
    Q, s = 7, {"f32": 4, "f16": 2, "bf16": 2}[args.storage]
    fixed = None
    if args.variant:
        fixed = tuple(int(v) for v in args.variant.split(","))
        fixed = fixed + (1,) * (4 - len(fixed))

    if args.kernel_only:
        # step kernel alone, then the copy of the same byte count, K launches each
        g = P.LBWave(problems(x_mid, k, with_surface=False), storage=args.storage, stream=stream)
        if fixed:
            set_variant(g, fixed)
        g.set_graph(args.graph)
        g.step(args.warmup)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        g.step(args.steps)
        e1.record(stream)
        e1.synchronize()
        kms = e0.elapsed_time(e1) / args.steps
        variant = get_variant(g)
        g.close()
        del g
        half = 2 * Q * s * cells // 2
        a_buf = torch.empty(half, dtype=torch.uint8, device="cuda")
        b_buf = torch.empty(half, dtype=torch.uint8, device="cuda")
        e0.record(stream)
        for _ in range(args.steps):
            P.stream_copy(a_buf, b_buf, half, stream)
        e1.record(stream)
        e1.synchronize()
        cms = e0.elapsed_time(e1) / args.steps
        print(json.dumps({"mode": "kernel-only", "variant": variant, "storage": args.storage,
                          "steps": args.steps, "ms_per_step": kms,
                          "one_step_equivalent_gbs": 2 * half / kms / 1e6, "copy_bytes": 2 * half,
                          "copy_ms": cms, "copy_gbs": 2 * half / cms / 1e6}), flush=True)
        return

    # --- whole hot path: step kernel + surface measurement, 16 instances ---
    h = P.LBWave(probs, storage=args.storage, stream=stream)
    if fixed:
        set_variant(h, fixed)
        tune_ms = None
    else:
        tune_ms = h.autotune(6)
    variant = get_variant(h)
    spl, plan = h.launch_steps(), h.launch_plan()
    h.set_graph(args.graph)
    h.step(args.warmup)
    if args.graph > 0 and args.steps > 2 * args.graph:
        # the replayed step sequence is captured and instantiated before the clock starts
        h.step(2 * args.graph + 6)
    h.reset()  # the timed steps start the run from rest
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    e0.record(stream)
    h.step(args.steps)
    e1.record(stream)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    # device time per launch over the timed region (one launch per spl steps,
    # the surface measurement fused in; the interval also holds the
    # graph-chunk counter updates and the launches that drain the measurement
    # pipeline at the end)
    launch_ms = e0.elapsed_time(e1) / args.steps * spl
    ms_per_step = elapsed / args.steps * 1e3
    mlups = cells * args.steps / elapsed / 1e6
    F, nacc = h.force(allow_empty=True)
    full_run = args.steps >= probs[0]["n_steps"]
    h.close()
    del h

    # --- the lattice stage alone (same instances and variant, no surface blocks) ---
    g = P.LBWave(problems(x_mid, k, with_surface=False), storage=args.storage, stream=stream)
    set_variant(g, variant)
    if plan[0] > 1:
        g.set_launch_plan(*plan)
    g.set_graph(args.graph)
    g.step(2 * args.graph + 10)  # past the first graph capture
    n_k = min(max(args.steps // 10, 50), 1000)
    e0.record(stream)
    g.step(n_k)
    e1.record(stream)
    e1.synchronize()
    lattice_ms = e0.elapsed_time(e1) / n_k * spl  # per launch
    g.close()
    del g
    # algorithmic HBM bytes of one launch: the state read once and written
    # once (2 Q s per cell), however many steps the launch advances
    bytes_per_launch = 2 * Q * s * cells
    achieved = bytes_per_launch / (launch_ms * 1e-3) / 1e9
    traffic = measured_traffic(args.storage, variant, plan)

    # --- copy reference: the same bytes through one read and one write stream ---
    half = bytes_per_launch // 2
    a_buf = torch.empty(half, dtype=torch.uint8, device="cuda")
    b_buf = torch.empty(half, dtype=torch.uint8, device="cuda")
    for _ in range(3):
        P.stream_copy(a_buf, b_buf, half, stream)
    e0.record(stream)
    n_c = 20
    for _ in range(n_c):
        P.stream_copy(a_buf, b_buf, half, stream)
    e1.record(stream)
    e1.synchronize()
    copy_gbs = 2 * half / (e0.elapsed_time(e1) / n_c * 1e-3) / 1e9
    del a_buf, b_buf

    # --- plain single-instance rate for the forces/s comparison ---
    one = P.LBWave([probs[7]], storage=args.storage, stream=stream)
    if fixed:
        set_variant(one, fixed)
    else:
        one.autotune(4)  # one box alone: its own best variant
    one.set_graph(args.graph)
    one.step(2 * args.graph + 10)  # past the first graph capture
    torch.cuda.synchronize()
    n1 = 400
    t1 = time.perf_counter()
    one.step(n1)
    torch.cuda.synchronize()
    single_ms = (time.perf_counter() - t1) / n1 * 1e3
    one.close()

    n_run = probs[0]["n_steps"]
    out = {
        "metric": METRIC,
        "value": round(mlups, 1),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": args.storage,
        "data": "synthetic",
        "config": {
            "workload": "3D sphere, D3Q7 256x128x128, lambda=256, c0=0.5, c_p/c0=1.1, R=12, "
                        "2048 Fibonacci surface points, 16 positions kh in [0, pi/2] batched "
                        "in one handle, 30 periods (15360 steps), average over the last 10",
            "instances": N_POS, "cells_per_step": cells, "storage": args.storage,
            "kernel_variant": {"cells_per_lane": variant[0], "x_mode": variant[1],
                               "nontemporal": variant[2], "steps_per_launch": spl},
            "graph_chunk": args.graph,
            "x_antinode": round(x_mid, 4), "Pa": cal["Pa"],
        },
        "roofline": {
            "bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
            "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4),
            "traffic": traffic,
            "kernel": kernel_name(args.storage, variant, plan),
            "kernel_ms": round(launch_ms, 5),
            "steps_per_launch": spl,
            "algorithmic_bytes_per_launch": bytes_per_launch,
            "one_step_equivalent_gbs": round(achieved * spl, 1),
            # the same rate counted at 2 Q s bytes per cell update (steps_per_launch updates per
            # cell per launch): above 1 when the launch keeps intermediate steps on chip
            "per_update_frac": round(achieved * spl / HBM_PEAK_GBS, 4),
            "lattice_stage_only_ms": round(lattice_ms, 5),
            "lattice_stage_only_gbs": round(bytes_per_launch / (lattice_ms * 1e-3) / 1e9, 1),
            "copy_reference_gbs": round(copy_gbs, 1),
            "frac_of_copy": round(achieved / copy_gbs, 4),
        },
        "forces_per_s": {
            "batched_16": round(N_POS / (n_run * ms_per_step * 1e-3), 3),
            "plain_single": round(1.0 / (n_run * single_ms * 1e-3), 3),
        },
        "autotune_ms_per_step": None if tune_ms is None else round(tune_ms, 4),
    }
    if full_run:
        out["forces_x"] = [float(v) for v in F[:, 0]]
        out["n_accum"] = int(nacc[0])
    if not args.no_batch and args.batch_subset > 0:
        b = batch_leg(args, args.batch_subset, stream)
        b.pop("forces_x")
        out["forces_per_s"]["uneven_batch_batched"] = b["forces_per_s"]["batched"]
        out["forces_per_s"]["uneven_batch_plain"] = b["forces_per_s"]["plain_one_at_a_time"]
        out["uneven_batch"] = b
    if not args.no_cylinder:
        c = cylinder_leg(args, not args.no_cpu_baseline)
        out["forces_per_s"]["cylinder_2d_single"] = c["single"]["forces_per_s"]
        out["forces_per_s"]["cylinder_2d_batch_64"] = c["batch_64"]["forces_per_s"]
        out["cylinder_2d"] = c
    if not args.no_surrogate:
        sur = surrogate_leg(stream, args.surrogate_batch, args.surrogate_steps, args.lb_sample,
                            args.graph, args.fallback_sample)
        if sur is not None:
            out["forces_per_s"]["surrogate"] = sur["forces_per_s"]
            out["surrogate"] = sur
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(x_mid, k, args.cpu_steps)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
