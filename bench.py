#!/usr/bin/env python3
"""Benchmark of the grouped Barnes-Hut tree force on one MI355X.

One step = the whole hot path over one synthetic particle set already
resident in HBM: root cube, Morton keys, radix sort, tree topology and
moments, groups, the group walk writing the interaction lists, and the FP32
force sum.  Default workload: clustered box, N = 4,194,304 (30% uniform + 70%
in 2048 Plummer halos), eps = 1e-4, n_crit = 256: the learned-vs-fixed theta
configuration.

Before timing, theta is bisected until the RMS relative force error against
FP64 direct summation on a seeded sample of 4096 particles is 1e-3 (+-0.3%),
and the network's output shift likewise for the learned mode (fixed theta is
the fallback when the network's output is not finite or misses the target).
Prints one JSON line.  value = tree-force interactions per second of whole
fixed-theta steps at that theta (sum over members of list length - 1,
divided by the step time), each step one HIP graph replay.  Beside it:
particles/s; the learned per-group theta at the same error, its step
(features, probe walk and inference included) replayed as a graph the same
way and timed in alternation with the fixed step; interactions of both modes
interpolated to exactly 1e-3; both modes' RMS on a held-out judge sample; the
2M clustered box in the same two modes; 20 leapfrog steps of the 8M box with
learned theta (energy drift); the quadrupole option and Peano-Hilbert order
at the same error; the neighbour search with SPH densities at 64 neighbours
per particle; the per-particle walk at the same error; the 64-system batch;
the roofline of the dominant kernel (the force sum, FP32 VALU); and the FP64
CPU oracle: its throughput, its own RMS against direct summation, and the
GPU's deviation from it.
"""
from __future__ import annotations

import argparse
import dataclasses
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "tree-force interactions/s and particles/s at 1e-3 RMS force error, learned vs fixed θ"
FP32_VALU_PEAK_TFLOPS = 157.3   # MI355X published FP32 vector peak
FLOPS_PER_INTERACTION = 20      # 3 sub, 3 FMA (r^2), rsqrt, 3 mul, 3 FMA (acc), 1 add (pot)
HBM_PEAK_GBPS = 8000.0          # MI355X published HBM3E bandwidth
NODE_BYTES = 56                 # node record bytes a walk visit reads (centre of mass, mass, side, offset, children)
FAR_BYTES, NEAR_BYTES = 16, 32  # list bytes written per far / near entry
HELDOUT_SEED = 54321            # a second judge sample, not used by any calibration


# HBM traffic of the force kernel from rocprofv3 FETCH_SIZE / WRITE_SIZE runs
# of this script (bytes per launch, scaled by the counters' reading of a
# device copy of known size), valid only for the kernel source and theta it
# was taken on.
TRAFFIC = {
    # clustered box, 4,194,304 particles, theta 0.3328125 (the 1e-3 RMS theta):
    # FETCH_SIZE 5491322.9 KiB x 1.99986 (a 512 MiB device copy reads as
    # 262162.06 KiB) + WRITE_SIZE 284525.4 KiB x 1.0 (the copy writes 524288 KiB)
    "clustered_4m": {"theta": 0.3328125, "bytes_per_launch": 11536796073,
                     "k_force_sha256": "2fc5575c90f30892c16d579095380bf51558e0739e558dad6c85852d823274dc"},
    # clustered box, 2,097,152 particles, theta 0.41997070312499996:
    # FETCH_SIZE 1658197.5 KiB x 1.99986 + WRITE_SIZE 146784.9 KiB x 1.0
    "clustered_2m": {"theta": 0.41997070312499996, "bytes_per_launch": 3546058498,
                     "k_force_sha256": "2fc5575c90f30892c16d579095380bf51558e0739e558dad6c85852d823274dc"},
}


def traffic_for(workload, theta):
    rec = TRAFFIC.get(workload)
    if rec is None or abs(rec["theta"] - theta) > 1e-12:
        return None
    src = os.path.join(ROOT, "paper_0909_0541_amd", "csrc", "k_force.hip")
    with open(src, "rb") as f:
        if hashlib.sha256(f.read()).hexdigest() != rec["k_force_sha256"]:
            return None
    return rec["bytes_per_launch"]


def parse():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="clustered_4m")
    ap.add_argument("--n", type=int, default=None, help="override the particle count")
    ap.add_argument("--judge-sample", type=int, default=4096)
    ap.add_argument("--cpu-seconds", type=float, default=12.0, help="target CPU time of the oracle's tree sample")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--waves-per-cu", type=int, default=None)
    ap.add_argument("--theta", type=float, default=None,
                    help="time this fixed theta (no calibration, no learned leg)")
    ap.add_argument("--target-rms", type=float, default=1e-3,
                    help="calibrate theta by bisection to this RMS force error before timing "
                         "(0: time the workload's own theta)")
    ap.add_argument("--theta-lo", type=float, default=0.3,
                    help="lower end of the theta bisections (tighter targets need smaller theta)")
    ap.add_argument("--theta-net", default=os.path.join(ROOT, "paper_0909_0541_amd", "theta_net.npz"),
                    help="trained per-group theta network (the learned leg is skipped when missing)")
    ap.add_argument("--rounds", type=int, default=3,
                    help="alternating rounds of fixed and learned graph replays for their time ratio")
    ap.add_argument("--no-learned", action="store_true")
    ap.add_argument("--no-particle", action="store_true", help="skip the per-particle walk A/B leg")
    ap.add_argument("--no-quadrupole", action="store_true", help="skip the quadrupole A/B leg")
    ap.add_argument("--no-neighbors", action="store_true", help="skip the neighbour-search leg")
    ap.add_argument("--no-hilbert", action="store_true", help="skip the Peano-Hilbert order A/B leg")
    ap.add_argument("--no-batch", action="store_true", help="skip the batched-systems leg")
    ap.add_argument("--no-2m", action="store_true", help="skip the 2M clustered leg")
    ap.add_argument("--no-leapfrog", action="store_true", help="skip the 8M leapfrog leg")
    ap.add_argument("--leapfrog-steps", type=int, default=20)
    ap.add_argument("--curve", type=int, default=0, choices=(0, 1),
                    help="key order of the headline step: 0 Morton (default), 1 Peano-Hilbert (for counter runs)")
    ap.add_argument("--copy-check-mib", type=int, default=0,
                    help="run one device-to-device copy of this many MiB before the timed steps, "
                         "as the reference kernel that scales HBM byte counters")
    return ap.parse_args()


_T0 = time.perf_counter()


def progress(msg):
    """One line on stderr as each part of the run ends (stdout keeps the one JSON line)."""
    print(f"bench: {msg} ({time.perf_counter() - _T0:.1f} s)", file=sys.stderr, flush=True)


def _cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _rel_rms(a, ref):
    import numpy as np
    n = np.linalg.norm(ref, axis=1)
    n = np.where(n > 0, n, np.inf)
    return float(np.sqrt(np.mean((np.linalg.norm(a - ref, axis=1) / n) ** 2)))


def _deviation(gpu_acc, gpu_pot, ref, sel):
    """GPU against the oracle on the particles sel: relative vector deviation
    |a_gpu - a_orc| / |a_orc| (max, 99.9th percentile), and the fraction of
    particles inside the per-component parity bound (1e-5 of |a_orc|, or of
    the sum of term magnitudes where the resultant cancels)."""
    import numpy as np
    a = gpu_acc[sel]
    r = ref["acc"][sel]
    an = np.linalg.norm(r, axis=1)
    rel = np.linalg.norm(a - r, axis=1) / np.where(an > 0, an, np.inf)
    comp = np.abs(a - r).max(axis=1)
    prel = np.abs(gpu_pot[sel] - ref["pot"][sel]) / np.abs(ref["pot"][sel])
    return {"particles": int(sel.shape[0]), "max_rel": float(rel.max()),
            "p999_rel": float(np.quantile(rel, 0.999)),
            "within_bar": float(np.mean(comp <= 1e-5 * np.maximum(an, ref["acc_abs"][sel]))),
            "pot_max_rel": float(prel.max())}


def cpu_baseline(pos, mass, w, theta, total_interactions, target_s, judge_idx, gpu, learned_run=None):
    """The FP64 oracle on the host.

    Timed: the full tree build and grouping, the walk + force sum for the
    groups that hold the judge's particles plus further groups drawn at
    random until the sample is about target_s seconds of work (whole-job
    throughput extrapolated by interaction count), and FP64 direct summation
    for the judge's particles.  Reported with it: the oracle tree's own RMS
    error against that direct summation, and the GPU's deviation from the
    oracle on every member of the sampled groups (fixed theta; with
    learned_run = (theta_g, acc, pot) also the learned step against the
    oracle with the same per-group theta)."""
    import numpy as np

    import oracle

    gpu_acc, gpu_pot = gpu
    t0 = time.perf_counter()
    tree = oracle.Tree(pos, mass)
    G = tree.groups(w.n_crit)
    t_build = time.perf_counter() - t0
    first, count, _, _ = tree.group_info()
    _, perm = tree.sorted()
    inv = np.empty_like(perm)
    inv[perm] = np.arange(perm.shape[0])
    jg = np.unique(np.searchsorted(first, inv[judge_idx], side="right") - 1)
    t0 = time.perf_counter()
    out = tree.forces(w.eps, theta, groups=jg)
    t_judge = time.perf_counter() - t0
    rate = max(out["interactions"], 1) / max(t_judge, 1e-6)
    rest = np.setdiff1d(np.arange(G), jg)
    extra = np.random.default_rng(0).permutation(rest)
    want = max(0.0, target_s - t_judge - t_build) * rate
    mean_per_group = max(out["interactions"], 1) / max(jg.shape[0], 1)
    k = int(min(extra.shape[0], want / mean_per_group))
    t_extra, inter_extra = 0.0, 0
    if k > 0:
        t0 = time.perf_counter()
        o2 = tree.forces(w.eps, theta, groups=extra[:k])
        t_extra = time.perf_counter() - t0
        inter_extra = o2["interactions"]
        m = ~np.isnan(o2["acc"][:, 0])
        out["acc"][m], out["pot"][m], out["acc_abs"][m] = o2["acc"][m], o2["pot"][m], o2["acc_abs"][m]
    sample_inter = max(out["interactions"] + inter_extra, 1)
    t_force = t_judge + t_extra
    t_job = t_build + t_force * total_interactions / sample_inter
    t0 = time.perf_counter()
    a_dir, _ = oracle.direct(pos, mass, w.eps, idx=judge_idx)
    t_direct = time.perf_counter() - t0
    sel = np.flatnonzero(~np.isnan(out["acc"][:, 0]))
    res = {
        "value": total_interactions / t_job,
        "unit": "interactions/s",
        "cores": oracle.num_threads(),
        "kind": "oracle",
        "sample": (f"FP64 oracle: full tree build + grouping of all {pos.shape[0]} particles ({t_build:.2f} s); "
                   f"walk + force for the {jg.shape[0]} groups holding the {judge_idx.shape[0]} judge particles "
                   f"and {k} more of the {G} groups chosen at random ({sample_inter} interactions, "
                   f"{t_force:.2f} s); whole job extrapolated by interaction count"),
        "cpu_model": _cpu_model(),
        "oracle_rms_force_error": _rel_rms(out["acc"][judge_idx], a_dir),
        "gpu_rms_vs_oracle_direct": _rel_rms(gpu_acc[judge_idx], a_dir),
        "gpu_vs_oracle": _deviation(gpu_acc, gpu_pot, out, sel),
        "sampled_direct": {"particles": int(judge_idx.shape[0]), "seconds": t_direct,
                           "pairs_per_s": judge_idx.shape[0] * pos.shape[0] / t_direct},
    }
    if learned_run is not None:
        tg, lacc, lpot = learned_run
        t0 = time.perf_counter()
        ol = tree.forces(w.eps, theta, theta_g=tg, groups=jg)
        res["learned"] = {"oracle_rms_force_error": _rel_rms(ol["acc"][judge_idx], a_dir),
                          "gpu_rms_vs_oracle_direct": _rel_rms(lacc[judge_idx], a_dir),
                          "gpu_vs_oracle": _deviation(lacc, lpot, ol, np.flatnonzero(~np.isnan(ol["acc"][:, 0]))),
                          "seconds": time.perf_counter() - t0}
    # full direct summation at the small Plummer configuration (8192 particles)
    from paper_0909_0541_amd import inputs
    p8, m8, _ = inputs.plummer(8192, 1, with_vel=False)
    t0 = time.perf_counter()
    oracle.direct(p8, m8, 1.0 / 256.0)
    res["direct_plummer_8k_s"] = time.perf_counter() - t0
    return res


def batch_leg(args):
    """64 independent systems of uneven size (Plummer spheres and clustered
    boxes, N log-uniform in [1024, 262144], theta = 0.7, eps = N^(-1/3)/20) as
    one captured HIP graph per step, n_crit, waves per CU and the list tile
    length autotuned."""
    import torch

    from paper_0909_0541_amd import autotune, inputs

    pos, mass, off, eps = inputs.batch_systems()
    dpos = torch.as_tensor(pos, device="cuda")
    dmass = torch.as_tensor(mass, device="cuda")
    theta = 0.7
    best, trials, ctx = autotune.autotune(off, dpos, dmass, eps, theta)
    ms = autotune.time_graph(ctx, args.steps, args.warmup)
    st = ctx.get_stats()
    acc = ctx._graph_io[2]
    n = int(off[-1])
    return {"workload": "batch_64", "systems": int(len(off) - 1), "n": n, "theta": theta,
            "n_crit": best.n_crit, "waves_per_cu": best.waves_per_cu, "list_tile": best.list_tile, "ms_per_step": ms,
            "interactions_per_step": st.interactions, "interactions_per_s": st.interactions / (ms * 1e-3),
            "particles_per_s": n / (ms * 1e-3),
            "rms_force_error": autotune.batch_rms(ctx, off, dpos, dmass, eps, acc, sample=args.judge_sample),
            "step": "one HIP graph replay: build of all 64 trees, groups, list walk, force sum",
            "autotune": [{"n_crit": t.n_crit, "waves_per_cu": t.waves_per_cu, "list_tile": t.list_tile,
                          "ms": t.ms_per_step} for t in trials]}


def particle_leg(args, ctx, judge, dpos, dmass, w, line):
    """The paper's own GPU form as an A/B: every particle walks the tree by
    itself and sums on the way (no groups, no lists); theta bisected to the
    same RMS error (within 3%); the step is the tree build plus that walk."""
    import torch

    from paper_0909_0541_amd import learned

    n = dpos.shape[0]

    def step(th):
        ctx.build_tree(dpos, dmass)
        return ctx.compute_forces_particle(w.eps, th)

    def rms_of(th):
        acc, _ = step(th)
        return judge.rms(acc)

    theta, r = learned.bisect(rms_of, 0.2, 1.0, args.target_rms, rel_tol=0.03, iters=12)
    for _ in range(max(args.warmup, 1)):
        step(theta)
    torch.cuda.synchronize()
    ctx.get_stats()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    steps = max(1, min(args.steps, 3))
    e0.record()
    for _ in range(steps):
        step(theta)
    e1.record()
    torch.cuda.synchronize()
    st = ctx.get_stats()
    if st.error_flags:
        raise RuntimeError(f"device error flags {st.error_flags}")
    ms = e0.elapsed_time(e1) / steps
    return {"theta": theta, "rms_force_error": r, "ms_per_step": ms, "interactions_per_step": st.interactions,
            "interactions_per_s": st.interactions / (ms * 1e-3), "particles_per_s": n / (ms * 1e-3),
            "walk_ms": st.t_particle_ms / max(st.n_particle_calls, 1), "max_list": st.max_list,
            "grouped_speedup": ms / line["ms_per_step"],
            "interactions_vs_grouped": st.interactions / line["interactions_per_step"],
            "step": "tree build + per-particle walk and sum (each particle opens nodes by itself, as in the "
                    "paper's threaded-tree kernel; a wave shares the node reads of 16 or 32 neighbours)"}


def variant_leg(args, judge, dpos, dmass, w, line, inter_ref, step, **opts):
    """An option of the same step as an A/B at the same RMS force error:
    theta bisected to the target error with the option set, timed as a graph
    replay checked bit for bit against its eager step."""
    import numpy as np
    import torch

    from paper_0909_0541_amd import autotune, bh, learned

    n = dpos.shape[0]
    vctx = bh.Context(timing=True, waves_per_cu=args.waves_per_cu, **opts)
    v = learned.Stepper(vctx, dpos, dmass, w.eps, w.n_crit)

    def rms_of(th):
        v(theta=th)
        return judge.rms(v.acc)

    theta, r = learned.bisect(rms_of, args.theta_lo, 1.0, args.target_rms)
    ms_eager, st = learned.timed_steps(v, args.steps, args.warmup, theta=theta)
    per = lambda t, k: t / max(k, 1)
    stage = {"build": per(st.t_build_ms, st.n_build_calls), "groups": per(st.t_groups_ms, st.n_groups_calls),
             "walk": per(st.t_walk_ms, st.n_walk_calls), "force": per(st.t_force_ms, st.n_force_calls)}
    ms, mode = ms_eager, "eager"
    try:
        g = bh.Context(waves_per_cu=args.waves_per_cu, **opts)
        g.graph_capture(np.array([0, n], dtype=np.int64), dpos, dmass, w.n_crit, [w.eps], [theta])
        ms_g = autotune.time_graph(g, args.steps, args.warmup)
        gst = g.get_stats()
        if not gst.error_flags and gst.interactions == st.interactions and torch.equal(g._graph_io[2], v.acc):
            ms, mode = ms_g, "graph"
        g.close()
    except (RuntimeError, bh.BHError):
        pass
    res = {"options": opts, "theta": theta, "rms_force_error": judge.rms(v.acc), "ms_per_step": ms,
           "step_mode": mode, "eager_ms_per_step": ms_eager, "interactions_per_step": st.interactions,
           "interactions_per_s": st.interactions / (ms * 1e-3), "particles_per_s": n / (ms * 1e-3),
           "stage_ms": stage, "max_list": st.max_list, "groups": st.n_groups,
           "interactions_vs_default": st.interactions / inter_ref,
           "particles_per_s_vs_default": (n / (ms * 1e-3)) / line["particles_per_s"],
           "step": step}
    vctx.close()
    return res


FP64_VALU_PEAK_TFLOPS = 78.6    # MI355X published FP64 vector peak
NEIGHBOR_NCRIT = 64             # group size of the neighbour search
FLOPS_PER_NEIGHBOR_TEST = 8      # FP64: 3 sub, 3 mul, 2 add for r^2 (the compare is not counted)


def neighbor_leg(args, dpos, dmass, w):
    """Neighbour search and SPH density (the general treewalk for a short-
    range interaction) on the same particles: radii for 64 neighbours (set-up,
    a few count passes), then the search with counts and densities timed."""
    import torch

    from paper_0909_0541_amd import bh, sph

    n = dpos.shape[0]
    c = bh.Context(timing=True, waves_per_cu=args.waves_per_cu)
    c.build_tree(dpos, dmass)
    c.make_groups(w.n_crit)
    h = sph.smoothing_lengths(c, dpos, n_target=64)
    # the search's own groups: smaller groups test fewer candidate pairs per
    # member (64 measured best on this machine; 256 tests 2.2x as many pairs)
    c.make_groups(NEIGHBOR_NCRIT)
    for _ in range(max(args.warmup, 1)):
        c.neighbors(h, count=True, rho=True)
    torch.cuda.synchronize()
    c.get_stats()
    steps = max(1, args.steps)
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        c.neighbors(h, count=True, rho=True)
    e1.record()
    torch.cuda.synchronize()
    st = c.get_stats()
    if st.error_flags:
        raise RuntimeError(f"device error flags {st.error_flags}")
    ms = e0.elapsed_time(e1) / steps
    kms = st.t_neighbor_ms / max(st.n_neighbor_calls, 1)
    achieved = FLOPS_PER_NEIGHBOR_TEST * st.neighbor_tests / (kms * 1e-3) / 1e12
    cn = c.neighbors(h, count=True)[0].cpu()
    c.close()
    return {"workload": w.name, "n": n, "n_target": 64, "n_crit": NEIGHBOR_NCRIT, "ms_per_call": ms, "kernel_ms": kms,
            "neighbor_pairs": st.neighbor_pairs, "pair_tests": st.neighbor_tests,
            "pairs_per_s": st.neighbor_pairs / (ms * 1e-3), "tests_per_s": st.neighbor_tests / (ms * 1e-3),
            "particles_per_s": n / (ms * 1e-3),
            "median_neighbors": float(cn.median().item()), "max_neighbors": int(cn.max().item()),
            "roofline": {"bound": "issue", "achieved": achieved, "peak": FP64_VALU_PEAK_TFLOPS, "unit": "TFLOP/s",
                         "frac": achieved / FP64_VALU_PEAK_TFLOPS, "kernel": "k_neighbors",
                         "flops_per_test": FLOPS_PER_NEIGHBOR_TEST,
                         "note": "bound by vector issue (scan, pair bookkeeping, FP64 decisions and kernel), 62 to 69 % "
                                 "of the cycles at three waves a SIMD; the FP64 rate is given for scale, not "
                                 "as the bound"},
            "step": "neighbour counts and SPH densities of every particle on a built tree and groups"}


def _stages(st, theta=False):
    per = lambda t, k: t / max(k, 1)
    out = {"build": per(st.t_build_ms, st.n_build_calls), "groups": per(st.t_groups_ms, st.n_groups_calls),
           "walk": per(st.t_walk_ms, st.n_walk_calls), "force": per(st.t_force_ms, st.n_force_calls)}
    if theta:
        out["theta"] = per(st.t_theta_ms, st.n_theta_calls)
    return out


def equal_error(args, w, dpos, dmass, net, headline: bool):
    """Fixed and learned theta on one particle set at the same RMS error.

    Both are calibrated on the judge sample (bisection to within 0.3%, plus
    interactions interpolated to exactly the target from the bisections);
    each mode's whole step is captured as a HIP graph, its replay checked bit
    for bit against the eager step, and the two replays are timed in
    alternating rounds.  Returns (report, objects the caller may reuse)."""
    import numpy as np
    import torch

    from paper_0909_0541_amd import autotune, bh, learned

    n = dpos.shape[0]
    ctx = bh.Context(timing=True, waves_per_cu=args.waves_per_cu, curve=args.curve)
    judge = learned.Judge(ctx, dpos, dmass, w.eps, args.judge_sample)
    heldout = learned.Judge(ctx, dpos, dmass, w.eps, args.judge_sample, seed=HELDOUT_SEED)
    fixed = learned.Stepper(ctx, dpos, dmass, w.eps, w.n_crit)
    cal = None
    if args.target_rms > 0 and args.theta is None:
        cal = learned.calibrate(ctx, dpos, dmass, w.eps, w.n_crit, None if args.no_learned else net, judge,
                                args.target_rms, theta_lo=args.theta_lo)
        theta = cal.theta
    else:
        theta = w.theta if args.theta is None else args.theta
    ms_eager, st = learned.timed_steps(fixed, args.steps, args.warmup, theta=theta)
    inter = st.interactions
    t_walk = _stages(st)["walk"]
    walk_bytes = (NODE_BYTES * st.node_visits + FAR_BYTES * (st.list_entries - st.near_entries)
                  + NEAR_BYTES * st.near_entries)
    walk = {"bound": "latency", "achieved": walk_bytes / (t_walk * 1e-3) / 1e9, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
            "node_visits": st.node_visits, "list_entries": st.list_entries, "near_entries": st.near_entries,
            "bytes_per_step": walk_bytes,
            "note": "algorithmic bytes (56 B per node visit read, 16/32 B per far/near list entry written) over "
                    "the walk kernel's time; the node reads mostly hit the XCD's L2, so HBM is not its bound"}
    walk["frac"] = walk["achieved"] / HBM_PEAK_GBPS
    rep = {"n": n, "theta": theta, "rms_force_error": judge.rms(fixed.acc),
           "heldout_rms_force_error": heldout.rms(fixed.acc), "interactions_per_step": inter,
           "stage_ms": _stages(st), "eager_ms_per_step": ms_eager, "groups": st.n_groups, "cells": st.n_cells,
           "max_list": st.max_list, "walk_roofline": walk}
    off = np.array([0, n], dtype=np.int64)
    gf = bh.Context(waves_per_cu=args.waves_per_cu, curve=args.curve)
    gf.graph_capture(off, dpos, dmass, w.n_crit, [w.eps], [theta])
    graph_error = None
    ms_fixed = autotune.time_graph(gf, args.steps, args.warmup)
    gst = gf.get_stats()
    if gst.error_flags or gst.interactions != inter or not torch.equal(gf._graph_io[2], fixed.acc):
        graph_error = (f"replay differs from the eager step (flags {gst.error_flags}, "
                       f"interactions {gst.interactions} vs {inter})")
        ms_fixed = ms_eager
    rep["ms_per_step"] = ms_fixed
    rep["step_mode"] = "graph" if graph_error is None else f"eager ({graph_error})"
    rep["interactions_per_s"] = inter / (ms_fixed * 1e-3)
    rep["particles_per_s"] = n / (ms_fixed * 1e-3)
    if cal is not None:
        rep["calibration"] = {"target_rms": args.target_rms, "theta": theta, "rms": cal.fixed_rms,
                              "band": 0.003, "evaluations": len(cal.fixed_history),
                              "search": f"bisection over theta in [{args.theta_lo}, 1.0]",
                              "interactions_at_target": learned.at_target(cal.fixed_history, args.target_rms)}
    keep = {"ctx": ctx, "judge": judge, "fixed": fixed, "theta": theta, "stats": st, "learned": None}
    if cal is not None and net is not None and not args.no_learned:
        lr = {"mode": cal.mode, "fallback_reason": cal.reason, "shift": cal.shift,
              "calibration_rms": cal.learned_rms, "evaluations": len(cal.learned_history),
              "interactions_at_target": learned.at_target(cal.learned_history, args.target_rms)}
        if cal.mode == "learned":
            lstep = learned.Stepper(ctx, dpos, dmass, w.eps, w.n_crit, net)
            ms_le, st_l = learned.timed_steps(lstep, args.steps, args.warmup, theta=theta, shift=cal.shift)
            gl = bh.Context(waves_per_cu=args.waves_per_cu, curve=args.curve)
            gl.graph_capture_learned(off, dpos, dmass, w.n_crit, [w.eps], [theta], net.params, net.mu, net.sigma,
                                     shift=cal.shift)
            ms_l = autotune.time_graph(gl, args.steps, args.warmup)
            lst = gl.get_stats()
            lmode = "graph"
            if lst.error_flags or lst.interactions != st_l.interactions or not torch.equal(gl._graph_io[2], lstep.acc):
                lmode, ms_l = "eager (replay differs from the eager step)", ms_le
            # alternating rounds: fixed replay, learned replay, ... (drifts of
            # clock or temperature then hit both modes alike)
            rounds_f, rounds_l = [], []
            if lmode == "graph" and graph_error is None:
                for _ in range(max(args.rounds, 1)):
                    rounds_f.append(autotune.time_graph(gf, args.steps, 1))
                    rounds_l.append(autotune.time_graph(gl, args.steps, 1))
            ratio = (float(np.median(np.array(rounds_f) / np.array(rounds_l))) if rounds_f
                     else ms_fixed / ms_l)
            tg = lstep.theta_g[:st_l.n_groups].cpu().numpy()
            lr.update({
                "rms_force_error": judge.rms(lstep.acc), "heldout_rms_force_error": heldout.rms(lstep.acc),
                "ms_per_step": ms_l, "step_mode": lmode, "eager_ms_per_step": ms_le,
                "interactions_per_step": st_l.interactions,
                "interactions_per_s": st_l.interactions / (ms_l * 1e-3), "particles_per_s": n / (ms_l * 1e-3),
                "stage_ms": _stages(st_l, theta=True), "theta_fallback_groups": st_l.n_theta_fallback,
                "theta_mean": float(tg.mean()), "theta_min": float(tg.min()), "theta_max": float(tg.max()),
                "interactions_saved": 1.0 - st_l.interactions / inter,
                "alternating_ms": {"fixed": rounds_f, "learned": rounds_l},
                "particles_per_s_vs_fixed": ratio,
                "step": "one HIP graph replay: tree build, groups, features + probe walk + inference, "
                        "list walk, force sum"})
            fa, la = rep["calibration"]["interactions_at_target"], lr["interactions_at_target"]
            if fa and la:
                lr["interactions_at_target_vs_fixed"] = la / fa
            keep["learned"] = (lstep, gl)
        rep["learned"] = lr
    keep["graph"] = gf
    return rep, keep


def leapfrog_leg(args):
    """Time integration of the 8M clustered box (halo velocities): learned
    theta calibrated to the target RMS at t = 0 (fixed theta as fallback),
    then kick-drift-kick steps with the tree rebuilt every step."""
    from paper_0909_0541_amd import simulate
    out = simulate.run("clustered_8m", steps=args.leapfrog_steps, dt=1e-4, target_rms=args.target_rms,
                       learned_theta=os.path.exists(args.theta_net) and not args.no_learned,
                       theta_net=args.theta_net, judge_sample=args.judge_sample, every=10)
    out.pop("energy", None)
    return out


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only: --gpus {args.gpus} is not supported "
              f"(the method runs on a single MI355X here)", file=sys.stderr)
        sys.exit(2)
    import numpy as np
    import torch

    from paper_0909_0541_amd import inputs, learned

    torch.cuda.set_device(0)
    net = None
    if os.path.exists(args.theta_net) and not args.no_learned:
        net = learned.ThetaNet.load(args.theta_net)
    pos, mass, _, w = inputs.make_workload(args.workload, n=args.n)
    n = pos.shape[0]
    dpos = torch.as_tensor(pos, device="cuda")
    dmass = torch.as_tensor(mass, device="cuda")

    if args.copy_check_mib > 0:
        nb = args.copy_check_mib << 20
        src = torch.ones(nb, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    progress(f"{w.name}: inputs on the device")
    rep, keep = equal_error(args, w, dpos, dmass, net, headline=True)
    progress(f"{w.name}: fixed and learned calibrated and timed")
    ctx, judge, theta, st = keep["ctx"], keep["judge"], keep["theta"], keep["stats"]
    inter = rep["interactions_per_step"]
    ms_per_step = rep["ms_per_step"]
    t_force = rep["stage_ms"]["force"]
    achieved = FLOPS_PER_INTERACTION * inter / (t_force * 1e-3) / 1e12
    line = {
        "metric": METRIC,
        "value": inter / (ms_per_step * 1e-3),
        "unit": "interactions/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": w.name, "description": w.description, "n": n, "eps": w.eps, "theta": theta,
                   "workload_theta": w.theta, "n_crit": w.n_crit,
                   "theta_mode": ("fixed, bisected to the target RMS force error" if "calibration" in rep
                                  else "fixed"),
                   "key_order": "Peano-Hilbert" if args.curve else "Morton"},
        "particles_per_s": rep["particles_per_s"],
        "step": ("one HIP graph replay: tree build, groups, list walk, force sum" if rep["step_mode"] == "graph"
                 else rep["step_mode"]),
        "eager": {"ms_per_step": rep["eager_ms_per_step"], "interactions_per_s": inter / (rep["eager_ms_per_step"] * 1e-3),
                  "step": "the same calls issued one by one (the force call waits for the walk to check its "
                          "list pools)"},
        "interactions_per_step": inter,
        "interactions_per_particle": inter / n,
        "rms_force_error": rep["rms_force_error"],
        "heldout_rms_force_error": rep["heldout_rms_force_error"],
        "judge_sample": int(judge.idx.shape[0]),
        "theta_calibration": rep.get("calibration"),
        "groups": rep["groups"],
        "cells": rep["cells"],
        "max_list": rep["max_list"],
        "stage_ms": rep["stage_ms"],
        "roofline": {"bound": "alu", "achieved": achieved, "peak": FP32_VALU_PEAK_TFLOPS, "unit": "TFLOP/s",
                     "frac": achieved / FP32_VALU_PEAK_TFLOPS, "traffic": traffic_for(w.name, theta),
                     "kernel": "k_force_lists", "flops_per_interaction": FLOPS_PER_INTERACTION},
        "walk_roofline": rep["walk_roofline"],
        "force_kernel_interactions_per_s": inter / (t_force * 1e-3),
        "walk_plus_force_interactions_per_s": inter / ((rep["stage_ms"]["walk"] + t_force) * 1e-3),
    }
    if "learned" in rep:
        line["learned"] = rep["learned"]
    fixed_acc = keep["fixed"].acc
    gpu_fixed = (fixed_acc.double().cpu().numpy(), keep["fixed"].pot.double().cpu().numpy())
    learned_run = None
    if keep["learned"] is not None:
        lstep, _ = keep["learned"]
        G = st.n_groups
        learned_run = (lstep.theta_g[:G].double().cpu().numpy(), lstep.acc.double().cpu().numpy(),
                       lstep.pot.double().cpu().numpy())
    if "calibration" in rep and abs(theta - w.theta) > 1e-12:
        fixed = keep["fixed"]
        ms2, st2 = learned.timed_steps(fixed, args.steps, args.warmup, theta=w.theta)
        s2 = _stages(st2)
        line["at_workload_theta"] = {
            "theta": w.theta, "rms_force_error": judge.rms(fixed.acc), "ms_per_step": ms2,
            "interactions_per_s": st2.interactions / (ms2 * 1e-3), "particles_per_s": n / (ms2 * 1e-3),
            "interactions_per_step": st2.interactions, "stage_ms": s2,
            "force_kernel_tflops": FLOPS_PER_INTERACTION * st2.interactions / (s2["force"] * 1e-3) / 1e12}
    keep["graph"].close()
    if keep["learned"] is not None:
        keep["learned"][1].close()
    if "calibration" in rep and not args.no_quadrupole:
        line["quadrupole"] = variant_leg(
            args, judge, dpos, dmass, w, line, inter,
            "tree build with second moments, groups, list walk, force sum with quadrupole terms", quadrupole=True)
        progress("quadrupole leg done")
    if "calibration" in rep and not args.no_hilbert:
        line["hilbert"] = variant_leg(
            args, judge, dpos, dmass, w, line, inter,
            "the same step with Peano-Hilbert keys (particles, children and groups in curve order)", curve=1)
        progress("Peano-Hilbert leg done")
    if not args.no_neighbors:
        line["neighbors"] = neighbor_leg(args, dpos, dmass, w)
        progress("neighbour leg done")
    if "calibration" in rep and not args.no_particle:
        line["per_particle"] = particle_leg(args, ctx, judge, dpos, dmass, w, line)
        progress("per-particle leg done")
    ctx.close()
    del keep
    if not args.no_2m and w.name != "clustered_2m" and args.n is None and args.theta is None:
        p2, m2, _, w2 = inputs.make_workload("clustered_2m")
        d2p, d2m = torch.as_tensor(p2, device="cuda"), torch.as_tensor(m2, device="cuda")
        r2, k2 = equal_error(args, w2, d2p, d2m, net, headline=False)
        for k in ("graph",):
            k2[k].close()
        if k2["learned"] is not None:
            k2["learned"][1].close()
        k2["ctx"].close()
        r2["workload"] = w2.name
        line["clustered_2m"] = r2
        progress("2M leg done")
        del d2p, d2m, k2
    if not args.no_batch:
        line["batch"] = batch_leg(args)
        progress("batch leg done")
    if not args.no_leapfrog and args.n is None:
        torch.cuda.empty_cache()
        line["leapfrog_8m"] = leapfrog_leg(args)
        progress("8M leapfrog leg done")
    if not args.no_cpu_baseline:
        w_cpu = dataclasses.replace(w, theta=theta)
        line["cpu_baseline"] = cpu_baseline(pos, mass, w_cpu, theta, inter, args.cpu_seconds, judge.idx,
                                            gpu_fixed, learned_run)
        progress("CPU oracle baseline done")
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
