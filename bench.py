"""Benchmark: literal-gradient evaluations per second on one MI355X.

Headline workload: the large hybrid instance (n = 100000 variables; 420000
random 3-SAT clauses, 10000 XOR constraints of length 8..64, 2000
at-least-t constraints of length 128..512), 256 restarts, FP32 with FP64
root-of-unity products for constraints of 128 literals or more (the
library's default; at least those beyond 256 literals must be FP64), seeded
synthetic data.  One step is one pass of the whole per-batch hot path:
objective and gradient of every constraint at every restart, the
deterministic reduction into the gradient, the projected step, the exact
round-and-check and the adaptive-weight update, replayed from a captured
graph.

value = nnz * B / (seconds per step): one "literal-gradient evaluation" is
one (literal occurrence, restart) pair whose gradient contribution and the
objective are produced.

`roofline` describes the kernel with the most time per step, timed live
with HIP events on the stream it runs on.  One convention throughout:
FP32 root-of-unity kernels (running products) are priced at 10 k^2 FLOP per
(constraint, restart) against the published vector peak of their
arithmetic type (FP32 157.3, FP64 78.6 TFLOP/s) -- the kernels' own count,
about 7 k^2 (14 FLOP per literal and complex frequency over floor(k/2)
frequencies), is reported beside it as flop_exact_per_launch / frac_exact;
FP64 root-of-unity kernels (the polynomial form, about 2.25 k^2 + O(k) per
frequency-independent part) at that form's own FLOP count, from the
library's bin description (both figures then agree); transform-free chains and
the reduction move 8 B per (literal, restart) in the evaluation (a gathered
point, a slot written) plus 4 B per (literal, restart) and 8 B per
(variable, restart) in the reduction; the pulled gradient moves 4 B per
gathered other literal and per remaining slot, 8 B per (variable, restart)
and its entry lists; all against 8 TB/s.  A kernel is bound by whichever of
the two its work needs longer on.  Hardware counters of the
same kernel (VALU instructions, HBM bytes) come from the committed rocprofv3
summary in profiles/ while the kernel sources are unchanged.

Secondary workloads measured in the same run: the mixed n = 2000 instance
(1024 restarts), the 3-SAT part of the large instance alone, and random
3-SAT n = 50 with one restart in the persistent one-workgroup loop (a
latency line: its `roofline` names the loop and claims no fraction).  The time
to solve with learned against uniform initialisation (the metric's second
half) follows.  `cpu_baseline`: the FP64 oracle on the host cores, on a
leading subset of the headline's restarts.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import platform
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "literal-gradient evals/s at 1 GPU (vs FP64 oracle); time-to-solve learned vs random"
UNIT = "literal-gradient evals/s"
HBM_PEAK_GBS = 8000.0
PEAK_TFLOPS = {"f32": 157.3, "f64": 78.6}     # published vector peaks
CLOCK_GHZ, SIMDS = 2.4, 1024                  # 256 CUs x 4 SIMDs
FLOP_PER_K2 = 10.0                             # root-of-unity work per (constraint, restart), in FLOP
FP64_FAMILY = "k_eval<float, double, *, *, true>"  # per-bin FP64 root-of-unity kernels, as one family


WORKLOADS = {
    "large": {"gen": "config3", "seed": 3000, "B": 256, "steps": 30, "warmup": 3,
              "desc": "large hybrid SAT n=100000: 420000 3-SAT, 10000 XOR (len 8-64), 2000 at-least-t "
                      "(len 128-512, t ~ U{{1..len/2}}; FP64 root-of-unity products from 128 literals), "
                      "{B} restarts, FP32"},
    "mixed2000": {"gen": "config2", "seed": 2000, "B": 1024, "steps": 200, "warmup": 20,
                  "desc": "mixed hybrid SAT n=2000: 8000 OR (len 3-7), 500 XOR (len 3-20), "
                          "200 at-least-t (len 10-100), {B} restarts, FP32"},
    "large3sat": {"gen": "config3a", "seed": 3000, "B": 256, "steps": 100, "warmup": 10,
                  "desc": "random 3-SAT n=100000, m=420000 (the 3-SAT part of the large instance), "
                          "{B} restarts, FP32"},
    "uf50": {"gen": "config1", "seed": 1000, "B": 1, "steps": 200, "warmup": 20, "persistent": True,
             "desc": "random 3-SAT n=50, m=213 (latency: one restart; all iterations of a graph replay in one "
                     "persistent launch), {B} restart(s), FP32"},
}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=0, help="timed steps (0: the workload's default)")
    ap.add_argument("--warmup", type=int, default=-1, help="untimed warm-up steps (-1: the workload's default)")
    ap.add_argument("--restarts", type=int, default=0, help="restarts (0: the workload's own)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-tts", action="store_true",
                    help="skip the time-to-solve comparison (learned vs uniform initialisation)")
    ap.add_argument("--no-secondary", action="store_true",
                    help="measure the headline workload only")
    ap.add_argument("--no-autotune", action="store_true")
    ap.add_argument("--fp64-min-len", type=int, default=0,
                    help="root-of-unity constraints at least this long run in FP64 (0: the library's default)")
    ap.add_argument("--eta", type=float, default=0.05)
    ap.add_argument("--workload", default="large", choices=sorted(WORKLOADS),
                    help="headline instance family (default: the large instance)")
    ap.add_argument("--chunk", type=int, default=10, help="iterations per graph replay in the timed loop")
    ap.add_argument("--mode", default="auto", choices=["auto", "per_bin", "group_all", "group_dft"],
                    help="launch structure of the evaluation (auto: chosen by the autotuner)")
    ap.add_argument("--serial", action="store_true",
                    help="launch every bin on the caller's stream (no concurrent bins)")
    ap.add_argument("--tune-cache", default=None,
                    help="JSON file of tuned tile shapes (read if present, written after tuning)")
    ap.add_argument("--rq1", action="store_true",
                    help="instead of the step benchmark: the paper's RQ1 gradient timing (seven formulas, "
                         "10000 random points, time per point in FP32 and FP64, the FP64 oracle beside it)")
    ap.add_argument("--copy-mib", type=int, default=0,
                    help="also run a plain device copy of this many MiB (counter calibration)")
    ap.add_argument("--cpu-budget", type=float, default=15.0, help="seconds of oracle work for cpu_baseline")
    return ap.parse_args()


# ----------------------------------------------------------------------------- roofline

def bin_work(bd, B):
    """Algorithmic work of one evaluation bin per launch: (flop, bytes, dtype).
    Root-of-unity bins: the library's per-restart figure (10 k^2 per
    constraint for the running-product form, the polynomial form's own count
    for FP64 bins), else 10 k^2."""
    per = bd.get("alg_flops_per_restart")
    flop = (per if per is not None else FLOP_PER_K2 * bd.get("k2_per_restart", 0.0)) * B
    nbytes = 8.0 * bd["lits"] * B
    return flop, nbytes, bd["ct"]


def bin_flop_exact(bd, B):
    """The kernels' own FLOP count of a bin per launch: 14 per (literal,
    complex frequency) over the floor(k/2) frequencies conjugate symmetry
    leaves, 4 per frequency, 8 per literal of a real chain (about 7 k^2 per
    root-of-unity constraint and restart)."""
    return bd.get("flops_per_restart", 0.0) * B


def bound_of(flop, nbytes, dt):
    t_alu = flop / (PEAK_TFLOPS[dt] * 1e12)
    t_hbm = nbytes / (HBM_PEAK_GBS * 1e9)
    return "alu" if t_alu >= t_hbm else "hbm"


def roofline_entry(label, flop, nbytes, dt, avg_s, launches_per_step):
    bound = bound_of(flop, nbytes, dt)
    ent = {"kernel": label, "avg_launch_ms": avg_s * 1e3, "launches_per_step": launches_per_step,
           "flop_per_launch": flop, "bytes_per_launch": nbytes, "arith": dt}
    if bound == "alu":
        ach = flop / avg_s / 1e12
        ent.update({"bound": "alu", "achieved": ach, "peak": PEAK_TFLOPS[dt],
                    "unit": "TFLOP/s", "frac": ach / PEAK_TFLOPS[dt]})
    else:
        ach = nbytes / avg_s / 1e9
        ent.update({"bound": "hbm", "achieved": ach, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                    "frac": ach / HBM_PEAK_GBS})
    return ent


def kernel_card(workload, kernel_name):
    """Counters of one kernel from the committed rocprofv3 summary
    (profiles/eval_step_<workload>_counters.txt, its `card:` lines), if the
    library sources hash to the value recorded with them; else None."""
    from paper_2308_15020_amd.profsum import kernel_source_hash
    path = os.path.join(ROOT, "profiles", f"eval_step_{workload}_counters.txt")
    if not os.path.exists(path):
        return None
    for line in open(path):
        if line.startswith("card: "):
            c = json.loads(line[len("card: "):])
            if c.get("kernel_name") == kernel_name and c.get("source_sha256") == kernel_source_hash():
                return c
    return None


def measure(name, args, dev, headline):
    """Runs one workload: an eager loop with library events (per-kernel
    launch times), then the timed loop of graph-replayed fused iterations."""
    import numpy as np
    import torch

    import workloads
    from paper_2308_15020_amd import Plan, Problem
    wl = WORKLOADS[name]
    steps = args.steps if (headline and args.steps > 0) else wl["steps"]
    warmup = args.warmup if (headline and args.warmup >= 0) else wl["warmup"]
    inst = getattr(workloads, wl["gen"])(wl["seed"])
    B = args.restarts if (headline and args.restarts) else wl["B"]
    x_np = workloads.points(inst.n_vars, B, workloads.point_seed(wl["seed"]))
    t_setup = time.perf_counter()
    prob = Problem(inst, device=0, fp64_min_len=args.fp64_min_len)
    plan = Plan(prob, B, autotune=not args.no_autotune, tune_cache=args.tune_cache, side_streams=not args.serial,
                mode=args.mode, persistent=wl.get("persistent", False))
    torch.cuda.synchronize()
    setup_s = time.perf_counter() - t_setup
    x0 = torch.from_numpy(x_np).to(dev)
    x = x0.clone()
    outs = {"F": torch.empty(B, device=dev), "n_sat": torch.empty(B, dtype=torch.int32, device=dev),
            "U": torch.empty(inst.m, dtype=torch.int32, device=dev)}

    # eager loop: objective, gradient, exact check of x_t and the projected
    # step in one pass, then the adaptive weights; library events per kernel.
    # With one launch per bin (many launches overlapping on the side
    # streams) each kernel's own launch time comes from the same tuned plan
    # with every launch on one stream (the per-bin shapes come from the
    # tuner's cache, a fixed per-bin structure times nothing more), so that
    # concurrent launches do not stretch each other's events; a grouped
    # structure is timed as it runs.
    d0 = plan.describe()
    split = not args.serial and d0["mode"] == "per_bin"
    tplan = plan if not split else Plan(prob, B, autotune=not args.no_autotune, tune_cache=args.tune_cache,
                                        side_streams=False, mode="per_bin",
                                        pull={0: "off", 3: "le3", 7: "le7"}.get(d0["pull"], "auto"),
                                        persistent=wl.get("persistent", False))

    def eager_step():
        o = tplan.eval_step(x, args.eta)
        tplan.erwa_update(o["U"], 0.4)

    prof_steps = max(1, min(steps, 10))
    for _ in range(max(1, warmup // 2)):
        eager_step()
    torch.cuda.synchronize()
    tplan.profile(True)
    tplan.profile_read(reset=True)
    for _ in range(prof_steps):
        eager_step()
    torch.cuda.synchronize()
    prof = tplan.profile_read(reset=True)
    tplan.profile(False)
    tdesc = tplan.describe()   # its bins are the profile's bin indices
    if tplan is not plan:
        tplan.close()

    # timed loop: chunk fused iterations per graph replay
    # the persistent loop runs every timed iteration in one launch
    chunk = steps if wl.get("persistent") else max(1, min(args.chunk, steps))
    while steps % chunk:
        chunk -= 1
    x.copy_(x0)
    prob.set_weights(inst.weights_or_ones())
    for _ in range(max(1, warmup // chunk)):
        plan.run_iters(x, chunk, args.eta, 0.4, out=outs)     # capture and warm-up, outside the timed region
    x.copy_(x0)
    prob.set_weights(inst.weights_or_ones())
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    for _ in range(steps // chunk):
        plan.run_iters(x, chunk, args.eta, 0.4, out=outs)
    torch.cuda.synchronize()
    t3 = time.perf_counter()
    ms_per_step = (t3 - t2) * 1e3 / steps
    value = inst.nnz * B / (ms_per_step / 1e3)
    n_sat_last = int(outs["n_sat"].max().item())

    desc = plan.describe()
    bins = tdesc["bins"]["f32"]
    assert tdesc["mode"] == desc["mode"] and len(tdesc["bins"]["f32"]) == len(desc["bins"]["f32"])
    kern = [k for k in prof["kernels"] if k["io"] == "f32"]
    entries = []
    for k in kern:
        avg_s = k["avg_ms"] / 1e3
        per_step = k["launches"] / prof_steps
        if k["bin"] == -2:
            grp = [b for b in bins if b["in_group"]]
            flop = sum(bin_work(b, B)[0] for b in grp)
            nbytes = sum(bin_work(b, B)[1] for b in grp)
            label = (f"grouped FP32 evaluation launch ({len(grp)} bins, "
                     f"{sum(1 for b in grp if b['class'] == 'dft')} root-of-unity, "
                     f"{sum(b['count'] for b in grp)} constraints)")
            ent = roofline_entry(label, flop, nbytes, "f32", avg_s, per_step)
            ent["flop_exact_per_launch"] = sum(bin_flop_exact(b, B) for b in grp)
            ent["kernel_name"] = "k_eval_group"
        elif k["bin"] == -4:
            grp = [b for b in bins if b.get("in_group64")]
            flop = sum(bin_work(b, B)[0] for b in grp)
            nbytes = sum(bin_work(b, B)[1] for b in grp)
            label = (f"grouped FP64 root-of-unity launch ({len(grp)} bins, {sum(b['count'] for b in grp)} constraints, "
                     f"len <= {max(b['maxk'] for b in grp)})")
            ent = roofline_entry(label, flop, nbytes, "f64", avg_s, per_step)
            ent["flop_exact_per_launch"] = sum(bin_flop_exact(b, B) for b in grp)
            ent["flop_10k2_per_launch"] = sum(FLOP_PER_K2 * b["k2_per_restart"] * B for b in grp)
            ent["kernel_name"] = "k_eval_group64"
        elif k["bin"] >= 0:
            bd = bins[k["bin"]]
            flop, nbytes, dt = bin_work(bd, B)
            label = (f"eval bin {k['bin']} ({bd['class']}, {bd['ct']} arithmetic, seg {bd['seg']}, L {bd['L']}, "
                     f"{bd['count']} constraints, len <= {bd['maxk']})")
            ent = roofline_entry(label, flop, nbytes, dt, avg_s, per_step)
            ent["flop_exact_per_launch"] = bin_flop_exact(bd, B)
            if bd["ct"] == "f64" and bd["class"] == "dft":
                ent["flop_10k2_per_launch"] = FLOP_PER_K2 * bd["k2_per_restart"] * B
            ent["kernel_name"] = (f"k_eval<float, {'double' if bd['ct'] == 'f64' else 'float'}, {bd['seg']}, "
                                  f"{bd['L']}, {'true' if bd['class'] == 'dft' else 'false'}>")
        elif k["bin"] == -3:
            # pulled gradient: the other literals of every pulled occurrence
            # gathered, the remaining slots read, the entry lists read once per
            # 64 * rpl restarts, x read and the stepped x written, one objective
            # and one count row per block written
            rpl = desc["pull_rpl"]
            nbytes = (4.0 * desc["pull_gathers_per_restart"] * B + 4.0 * desc["pull_other_slots"] * B
                      + desc["pull_entries"] * desc["pull_entry_bytes"] * math.ceil(B / (64 * rpl))
                      + 8.0 * inst.n_vars * B + 8.0 * desc["pull_rows"] * B)
            ent = roofline_entry(f"pulled gradient + projected step (transform-free constraints of length <= "
                                 f"{desc['pull']}: {desc['pull_entries']} occurrences, "
                                 f"{desc['pull_gathers_per_restart']} gathers per restart; "
                                 f"{desc['pull_other_slots']} other slots)", 0.0, nbytes, "f32", avg_s, per_step)
            ent["kernel_name"] = f"k_pull<{desc['pull_entry_bytes'] // 4}, {rpl}, true>"
        elif desc["pull"]:
            nbytes = 8.0 * desc["objective_rows"] * B
            ent = roofline_entry("objective and count row sums", 0.0, nbytes, "f32", avg_s, per_step)
            ent["kernel_name"] = f"k_reduce<float, false, {4 if B % 4 == 0 else 2 if B % 2 == 0 else 1}>"
        else:
            nbytes = (4.0 * inst.nnz + 8.0 * inst.n_vars) * B
            ent = roofline_entry("gradient reduction + projected step", 0.0, nbytes, "f32", avg_s, per_step)
            ent["kernel_name"] = f"k_reduce<float, true, {4 if B % 4 == 0 else 2 if B % 2 == 0 else 1}>"
        ent["ms_per_step"] = avg_s * 1e3 * per_step
        entries.append(ent)
    # kernels of one template are reported together (split bins of one shape)
    merged = {}
    for e in entries:
        m = merged.get(e["kernel_name"])
        if m is None:
            merged[e["kernel_name"]] = dict(e, _t=e["avg_launch_ms"] * e["launches_per_step"], _f=e["flop_per_launch"]
                                            * e["launches_per_step"], _b=e["bytes_per_launch"] * e["launches_per_step"],
                                            _x=e.get("flop_exact_per_launch", 0.0) * e["launches_per_step"],
                                            _k=e.get("flop_10k2_per_launch", 0.0) * e["launches_per_step"],
                                            _n=e["launches_per_step"], parts=1)
        else:
            m["_t"] += e["avg_launch_ms"] * e["launches_per_step"]
            m["_f"] += e["flop_per_launch"] * e["launches_per_step"]
            m["_x"] += e.get("flop_exact_per_launch", 0.0) * e["launches_per_step"]
            m["_k"] += e.get("flop_10k2_per_launch", 0.0) * e["launches_per_step"]
            m["_b"] += e["bytes_per_launch"] * e["launches_per_step"]
            m["_n"] += e["launches_per_step"]
            m["parts"] += 1
    kernels = []
    for kname, m in merged.items():
        n = m["_n"]
        ent = roofline_entry(m["kernel"] if m["parts"] == 1 else f"{kname} ({m['parts']} bin ranges)",
                             m["_f"] / n, m["_b"] / n, m["arith"], m["_t"] / n / 1e3, n)
        ent["kernel_name"] = kname
        ent["ms_per_step"] = m["_t"]
        if m["_x"] > 0 and ent["bound"] == "alu":
            ent["flop_exact_per_launch"] = m["_x"] / n
            ent["frac_exact"] = m["_x"] / n / (m["_t"] / n / 1e3) / 1e12 / PEAK_TFLOPS[m["arith"]]
        if m["_k"] > 0:
            ent["flop_10k2_per_launch"] = m["_k"] / n
        kernels.append(ent)
    # the FP64 root-of-unity bins launched one per segment shape (per-bin
    # launch structure) run one kernel template in several instances: they
    # are reported as one family, whose launches share the per-launch
    # average (total work / total time)
    fam = [e for e in kernels if e["kernel_name"].startswith("k_eval<float, double,")
           and e["kernel_name"].endswith("true>")]
    if len(fam) > 1:
        n = sum(e["launches_per_step"] for e in fam)
        t = sum(e["ms_per_step"] for e in fam)
        f = sum(e["flop_per_launch"] * e["launches_per_step"] for e in fam)
        nb = sum(e["bytes_per_launch"] * e["launches_per_step"] for e in fam)
        ent = roofline_entry(f"FP64 root-of-unity launches, polynomial form ({n:g} launches over "
                             f"{len(fam)} segment shapes)", f / n, nb / n, "f64", t / n / 1e3, n)
        ent["kernel_name"] = FP64_FAMILY
        ent["ms_per_step"] = t
        k10 = sum(e.get("flop_10k2_per_launch", 0.0) * e["launches_per_step"] for e in fam)
        if k10 > 0:
            ent["flop_10k2_per_launch"] = k10 / n
        ent["members"] = [e["kernel_name"] for e in fam]
        kernels = [e for e in kernels if e not in fam] + [ent] + fam
    kernels.sort(key=lambda e: -e["ms_per_step"])
    top = [e for e in kernels if not any(e["kernel_name"] in k.get("members", ()) for k in kernels)]
    dom = dict(top[0])
    if "flop_10k2_per_launch" in dom:
        # the same work at the 10 k^2 pricing of the running products: a rate
        # above the FP64 peak shows how much less the polynomial form computes
        dom["tflops_at_10k2"] = dom["flop_10k2_per_launch"] / (dom["avg_launch_ms"] / 1e3) / 1e12
    dom["traffic"] = None
    card = kernel_card(name, dom["kernel_name"])
    if card is not None:
        if "traffic_bytes_per_launch" in card:
            dom["traffic"] = float(card["traffic_bytes_per_launch"])
            dom["traffic_to_algorithmic_bytes"] = dom["traffic"] / max(dom["bytes_per_launch"], 1.0)
        if "rocprof_avg_us" in card:
            dom["rocprof_avg_launch_ms"] = float(card["rocprof_avg_us"]) / 1e3
        if "valu_insts_per_launch" in card:
            vi = float(card["valu_insts_per_launch"])
            # wave64 VALU instructions issue one per 4 cycles per SIMD
            dom["valu_insts_per_launch"] = vi
            dom["valu_issue"] = vi * 4.0 / (SIMDS * CLOCK_GHZ * 1e9 * dom["avg_launch_ms"] / 1e3)
    if wl.get("persistent") and desc.get("persistent_steps"):
        # the timed loop runs in the persistent kernel, not in the eager
        # loop's kernels listed under `kernels`: a latency line
        dom = {"kernel": "persistent fused-iteration loop (one workgroup runs every iteration of a replay)",
               "kernel_name": "k_iters_small", "bound": "latency", "achieved": None, "peak": None, "unit": None,
               "frac": None, "traffic": None, "us_per_iteration": ms_per_step * 1e3}
    for e in kernels:
        for key in ("flop_per_launch", "flop_exact_per_launch", "bytes_per_launch", "achieved", "frac", "frac_exact",
                    "avg_launch_ms", "ms_per_step"):
            if key in e and isinstance(e[key], float):
                e[key] = float(f"{e[key]:.5g}")
    res = {"workload": wl["desc"].format(B=B), "n_vars": inst.n_vars, "n_cons": inst.m, "nnz": inst.nnz,
           "restarts": B, "steps": steps, "warmup": warmup, "ms_per_step": ms_per_step, "value": value,
           "iterations_per_graph_replay": chunk, "setup_s_incl_autotune": setup_s,
           "best_n_sat_last_step": n_sat_last,
           "plan": {"launch_structure": desc["mode"], "pull_max_len": desc["pull"],
                    "tuned_candidates_ms": desc.get("tuned_modes")},
           "roofline": dom, "kernels": kernels[:12]}
    out = (res, inst, x_np)
    plan.close()
    prob.close()
    return out


# ----------------------------------------------------------------------------- host baseline

def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or "unknown"


def cpu_baseline(inst, x_np, budget_s=15.0):
    """FP64 oracle on the host: the same instance and points.  A probe on as
    many restarts as threads sizes a leading subset that takes about a third
    of the budget per pass; passes repeat until the budget is spent; the
    median pass gives evals/s (the oracle's cost is linear in the restarts,
    which are independent)."""
    import numpy as np

    import oracle
    n, B = x_np.shape
    threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    Bp = max(1, min(B, threads))
    probe = np.ascontiguousarray(x_np[:, :Bp].astype(np.float64))
    t0 = time.perf_counter()
    r = oracle.eval_batch(inst, probe, want_g=True, nthreads=threads)
    t_probe = max(time.perf_counter() - t0, 1e-6)
    used = r["threads"]
    Bs = min(B, Bp * max(1, int(budget_s / 3.0 / t_probe)))
    times = [t_probe] if Bs == Bp else []
    sub = np.ascontiguousarray(x_np[:, :Bs].astype(np.float64))
    t_start = time.perf_counter()
    while len(times) < 3 and (time.perf_counter() - t_start < budget_s or not times):
        t0 = time.perf_counter()
        r = oracle.eval_batch(inst, sub, want_g=True, nthreads=threads)
        times.append(time.perf_counter() - t0)
        used = r["threads"]
    t = float(np.median(times))
    return {"value": inst.nnz * Bs / t, "unit": UNIT, "cores": int(used), "kind": "oracle",
            "nproc": os.cpu_count(), "cpu_model": cpu_model(),
            "sample": f"the first {Bs} of {B} restarts of the same instance and points (restarts are "
                      f"independent, so evals/s = nnz * {Bs} / pass time), F and gradient in FP64 "
                      f"(count-lattice recursion for at-least-t, closed forms for OR/XOR); median of "
                      f"{len(times)} passes of {t:.2f} s, {int(used)} OpenMP threads"}


# ----------------------------------------------------------------------------- time to solve

def time_to_solve():
    """The second half of the metric: learned initialisation against uniform
    restarts (test instances disjoint from the training ones) on the
    leak-free hidden-assignment family shaped like the mixed n = 2000
    workload, with 300 XOR constraints (the most at which uniform restarts
    still solve nearly every instance within 60 rounds); the harness's log
    goes to stderr."""
    import contextlib
    from paper_2308_15020_amd import tts
    argv = ["--train", "50", "--test", "100", "--family", "hidden2", "--n-xor", "300", "--rounds", "60", "--T", "40",
            "--eta", "0.3"]
    t0 = time.perf_counter()
    with contextlib.redirect_stdout(sys.stderr):
        s = tts.main(argv)
    ms = lambda v: None if v is None else v * 1e3  # noqa: E731
    return {"instances": s["instances"], "family": s["family"], "n_xor": s["n_xor"], "B": s["B"],
            "rounds": s["rounds"], "T": s["T"],
            "reuse_proposal": s["reuse_proposal"],
            "solve_rate": s["solve_rate"], "both_solved": s["both_solved"],
            "median_ms": {k: ms(v) for k, v in s["median_s"].items()},
            "mean_ms": {k: ms(v) for k, v in s["mean_s"].items()},
            "median_rounds": s["median_rounds"],
            "cactus_at_lower_solve_rate": {
                (k[:-2] + "_ms" if k.endswith("_s") else k): (ms(v) if k.endswith("_s") else v)
                for k, v in s["cactus_at_lower_solve_rate"].items()},
            "learned_vs_polarity_median_ms": [ms(v) for v in s["learned_vs_polarity_median_s"]],
            "learned_first_round_only_median_ms": ms(s.get("learned_once_median_s")),
            "learned_first_round_only_solve_rate": s.get("learned_once_solve_rate"),
            "median_rounds_all_instances": s.get("median_rounds_all"),
            "harness_seconds": time.perf_counter() - t0}


# ----------------------------------------------------------------------------- RQ1

def rq1(args, dev, points=10000, reps=20):
    """Average time of one objective + gradient evaluation per random point
    for the paper's seven RQ1 formulas (its Benchmark Details lists their
    counts and lengths; n = 1000 and t = len/2 are not given there): all
    points as restarts of one batch, FP32 and FP64 evaluation, HIP events over
    `reps` evaluations; the FP64 oracle on the host beside it (a subset of the
    points, all threads and one thread)."""
    import numpy as np
    import torch

    import oracle
    import workloads
    from paper_2308_15020_amd import Plan, Problem
    threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    rows = []
    for name in workloads.RQ1_SHAPES:
        inst = workloads.rq1(name)
        x_np = workloads.points(inst.n_vars, points, workloads.point_seed(6000))
        prob = Problem(inst, device=0)
        plan = Plan(prob, points, autotune=not args.no_autotune, tune_cache=args.tune_cache)
        row = {"formula": name, "n": inst.n_vars, "m": inst.m, "nnz": inst.nnz, "points": points}
        for dt, key in ((torch.float32, "gpu_f32_us_per_point"), (torch.float64, "gpu_f64_us_per_point")):
            x = torch.from_numpy(x_np).to(dev, dt)
            out = plan.eval(x)
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(reps):
                plan.eval(x, out=out)
            e1.record()
            torch.cuda.synchronize()
            row[key] = e0.elapsed_time(e1) * 1e3 / reps / points
        sub = np.ascontiguousarray(x_np[:, :256].astype(np.float64))
        for nt, key in ((threads, "oracle_us_per_point"), (1, "oracle_1thread_us_per_point")):
            times = []
            for _ in range(3):
                t0 = time.perf_counter()
                oracle.eval_batch(inst, sub, want_g=True, nthreads=nt)
                times.append(time.perf_counter() - t0)
            row[key] = float(np.median(times)) * 1e6 / sub.shape[1]
        row["oracle_threads"] = threads
        rows.append(row)
        plan.close()
        prob.close()
    print(json.dumps({"metric": "RQ1 gradient computation time per random point", "unit": "us",
                      "data": "synthetic", "rows": rows}))


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU only; the multi-GPU path "
                                   "(sharding over restarts) is not built", "n_gpus": args.gpus}))
        sys.exit(2)
    import torch

    dev = torch.device("cuda:0")
    if args.rq1:
        return rq1(args, dev)
    if args.copy_mib > 0:
        # a plain elementwise kernel of known size: reads and writes copy_mib MiB
        src = torch.ones(args.copy_mib * 262144, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.neg(src, out=dst)
        torch.cuda.synchronize()
        del src, dst

    t_run = time.perf_counter()
    head, inst, x_np = measure(args.workload, args, dev, True)
    print(f"[bench] {args.workload}: {head['ms_per_step']:.3f} ms/step", file=sys.stderr, flush=True)
    secondary = {}
    if not args.no_secondary:
        for name in ("mixed2000", "large3sat", "uf50"):
            if name == args.workload:
                continue
            r, _, _ = measure(name, args, dev, False)
            secondary[name] = r
            print(f"[bench] {name}: {r['ms_per_step']:.3f} ms/step", file=sys.stderr, flush=True)

    res = {
        "metric": METRIC, "value": head["value"], "unit": UNIT, "n_gpus": 1, "steps": head["steps"],
        "warmup": head["warmup"], "ms_per_step": head["ms_per_step"], "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32+f64", "data": "synthetic",
        "config": {"workload": head["workload"], "n_vars": head["n_vars"], "n_cons": head["n_cons"],
                   "nnz": head["nnz"], "restarts": head["restarts"],
                   "step": "objective + gradient + exact round-and-check of x_t (one pass), projected step, "
                           "ERWA weight update; graph-replayed",
                   "iterations_per_graph_replay": head["iterations_per_graph_replay"],
                   "plan": head["plan"],
                   "setup_s_incl_autotune": round(head["setup_s_incl_autotune"], 2)},
        "roofline": head["roofline"],
        "kernels": head["kernels"],
    }
    if secondary:
        res["secondary"] = {k: {"workload": v["workload"], "value": v["value"], "ms_per_step": v["ms_per_step"],
                                "steps": v["steps"], "roofline": v["roofline"], "kernels": v["kernels"][:6]}
                            for k, v in secondary.items()}
    if not args.no_cpu_baseline:
        res["cpu_baseline"] = cpu_baseline(inst, x_np, args.cpu_budget)
        print(f"[bench] cpu baseline done", file=sys.stderr, flush=True)
    if not args.no_tts:
        res["time_to_solve"] = time_to_solve()
    res["bench_seconds"] = round(time.perf_counter() - t_run, 1)
    print(json.dumps(res))


if __name__ == "__main__":
    main()
