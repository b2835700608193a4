#!/usr/bin/env python3
"""Benchmark of the multi-hypothesis criticality hot path on one MI355X.

Workload: the 11-object scene (6 vehicles with 15x15 acceleration x yaw-rate
grids, 5 pedestrians with 15x15 speed x heading grids, 30 steps of 0.1 s),
83,531,250 pose-pair checks per pass. One step = one pass of the whole device
path on inputs resident in HBM: probability normalisation and trajectory
generation, collision recognition of every trajectory pair of every object
pair at every step, risk reduction to per-trajectory and per-object
criticality. A check is the decision of one pose pair; the rate counts every
check decided (sum of T_a * T_b * H over the object pairs). The collision
kernel decides most of them together, from bounds of groups of trajectories
that lie apart at a step, and tests the rest one by one, so the rate is an
effective one; results are those of testing every pose pair.

Prints one JSON line on stdout; progress goes to stderr.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# HBM rate of the MI355X, TB/s.
PEAK_HBM_TB_S = 8.0


def log(*a):
    print(*a, file=sys.stderr, flush=True)


# The paper's execution-time table (Sec. VI-B, Table I): scenario, COs,
# acceleration profiles, median ms of the whole algorithm on the Drive PX 2's
# GP106 (another machine and another overlap implementation: context only).
TABLE_ONE = [("S1", 3, 6, 10.0), ("S1", 3, 5, 8.0), ("S2", 10, 6, 21.0), ("S2", 10, 5, 14.0)]


def table_one(mhc, ctx, sg, torch, steps=50):
    """Each Table I configuration in both overlap modes: the whole path on
    inputs resident in HBM (as the headline), the collision kernel alone
    (HIP events on the launch stream), and host scene in -> host criticality
    out (the comparable quantity to the paper's timings)."""
    rows = []
    stream = torch.cuda.current_stream()
    for name, n_co, n_acc, paper_ms in TABLE_ONE:
        for overlap in (sg.OVERLAP_EXACT, sg.OVERLAP_PIP):
            cs_scene = sg.paper_scene(5, n_co=n_co, n_acc=n_acc, overlap=overlap)
            cs = mhc.CScene(cs_scene)
            checks = mhc.mhc_query_sizes(cs)["n_checks"]
            best, us = mhc.mhc_autotune(ctx, cs, reps=10)
            plan = mhc.mhc_plan_create(ctx, cs)
            out, r = mhc.device_result(cs, first_hit=True, q=True)
            for _ in range(5):
                mhc.mhc_plan_execute(plan, r, stream)
            torch.cuda.synchronize()
            a = time.perf_counter()
            for _ in range(steps):
                mhc.mhc_plan_execute(plan, r, stream)
            torch.cuda.synchronize()
            step_ms = (time.perf_counter() - a) * 1e3 / steps
            ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
            for k in range(steps):
                mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_TRAJ, r, stream)
                ev[k][0].record(stream)
                mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_COLLIDE, r, stream)
                ev[k][1].record(stream)
                mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_RISK, r, stream)
            torch.cuda.synchronize()
            k2_ms = sum(x.elapsed_time(y) for x, y in ev) / steps
            plan.close()
            lat = []
            for k in range(25):
                a = time.perf_counter()
                mhc.mhc_evaluate(ctx, cs, first_hit=False, q=False)
                if k >= 5:
                    lat.append((time.perf_counter() - a) * 1e3)
            row = {"scenario": name, "cos": n_co, "accel_profiles": n_acc,
                   "overlap": "pip" if overlap == sg.OVERLAP_PIP else "exact", "checks": checks,
                   "step_ms": step_ms, "checks_per_s": checks / (step_ms * 1e-3),
                   "collide_us": k2_ms * 1e3,
                   "e2e_p50_ms": pct(lat, 50), "tile_variant": best,
                   "paper_gp106_ms": paper_ms}
            rows.append(row)
            log(f"Table I {name} {n_co} COs x {n_acc} profiles, {row['overlap']:5s}: {checks:,} checks, "
                f"step {step_ms * 1e3:.1f} us ({row['checks_per_s']:.3g} checks/s), collide {k2_ms * 1e3:.1f} us "
                f"host-to-host p50 {row['e2e_p50_ms']:.3f} ms "
                f"[paper, GP106: {paper_ms:.0f} ms]")
    return rows


def timeline_extra(mhc, ctx, sg, torch, steps=50):
    """The risk over time (criticality per slot and its attribution) against
    the plain path, per risk reading, on the 11-object and the Table I S2
    scenes: whole-path step and each module's time (HIP events on the launch
    stream); the risk module then reads the per-slot sums once. Then the
    approach sequence (an EGO driving at a stopped vehicle, a frame every
    100 ms until contact) as one batch, and the anticipation times read from
    its criticality series."""
    stream = torch.cuda.current_stream()
    T, C, R = mhc.MHC_STAGE_TRAJ, mhc.MHC_STAGE_COLLIDE, mhc.MHC_STAGE_RISK
    rows = []
    for wname, make in (("eleven_object", lambda: sg.eleven_object_scene(1)),
                        ("table_one_s2", lambda: sg.paper_scene(5, n_co=10))):
        for risk in (sg.RISK_EXCLUSIVE, sg.RISK_INDEPENDENT):
            row = {"workload": wname, "risk": "exclusive" if risk == sg.RISK_EXCLUSIVE else "independent"}
            for tl in (0, 1):
                s = make()
                s.risk, s.timeline = risk, tl
                cs = mhc.CScene(s)
                plan = mhc.mhc_plan_create(ctx, cs)
                out, r = mhc.device_result(cs, first_hit=True, q=True)
                for _ in range(5):
                    mhc.mhc_plan_execute(plan, r, stream)
                torch.cuda.synchronize()
                a = time.perf_counter()
                for _ in range(steps):
                    mhc.mhc_plan_execute(plan, r, stream)
                torch.cuda.synchronize()
                step_us = (time.perf_counter() - a) * 1e6 / steps
                ev = [[torch.cuda.Event(enable_timing=True) for _ in range(4)] for _ in range(steps)]
                for k in range(steps):
                    ev[k][0].record(stream)
                    mhc.mhc_plan_execute_stages(plan, T, r, stream)
                    ev[k][1].record(stream)
                    mhc.mhc_plan_execute_stages(plan, C, r, stream)
                    ev[k][2].record(stream)
                    mhc.mhc_plan_execute_stages(plan, R, r, stream)
                    ev[k][3].record(stream)
                torch.cuda.synchronize()
                mods = [sum(e[m].elapsed_time(e[m + 1]) for e in ev) * 1e3 / steps for m in range(3)]
                plan.close()
                key = "timeline" if tl else "plain"
                row[key] = {"step_us": step_us, "traj_us": mods[0], "collide_us": mods[1], "risk_us": mods[2]}
                if tl:
                    n, H, nt = s.n_objects, s.horizon, sum(s.traj_counts())
                    # bytes the risk module must move: the per-slot sums in,
                    # criticality over time out (scratch + output), the
                    # attribution and the plain outputs
                    row["timeline"]["risk_bytes"] = 8 * (nt * n * H + 2 * nt * H + 4 * nt * n + n * H + n * n + 3 * nt)
                    row["timeline"]["risk_gb_s"] = row["timeline"]["risk_bytes"] / (mods[2] * 1e-6) / 1e9
            rows.append(row)
            p_, t_ = row["plain"], row["timeline"]
            log(f"timeline {wname} {row['risk']}: step {p_['step_us']:.1f} -> {t_['step_us']:.1f} us, collide "
                f"{p_['collide_us']:.1f} -> {t_['collide_us']:.1f} us, risk {p_['risk_us']:.1f} -> "
                f"{t_['risk_us']:.1f} us ({t_['risk_gb_s']:.0f} GB/s)")
    frames, event = sg.approach_sequence(8)
    cframes = [mhc.CScene(f) for f in frames]
    mhc.mhc_evaluate_batch(ctx, cframes, first_hit=False, q=False)
    lat = []
    for _ in range(10):
        a = time.perf_counter()
        outs = mhc.mhc_evaluate_batch(ctx, cframes, first_hit=False, q=False)
        lat.append((time.perf_counter() - a) * 1e3)
    crit = [float(o["object_crit"][0]) for o in outs]
    ant = {str(th): mhc.mhc_anticipation_time(crit, 0.1, th, event) for th in (0.5, 0.9, 0.99)}
    appr = {"frames": len(frames), "event_frame": event, "frame_dt_s": 0.1, "batch_ms_p50": pct(lat, 50),
            "ego_crit_last_frames": [round(c, 4) for c in crit[-6:]], "anticipation_s": ant}
    log(f"approach sequence: {len(frames)} frames in one batch, p50 {appr['batch_ms_p50']:.2f} ms; "
        f"anticipation time {ant} s")
    return {"rows": rows, "approach": appr}


def streams_extra(mhc, ctx, cs, checks, ref_out, steps, torch):
    """Whole-path steps of the timed scene issued round-robin on S streams,
    each with a plan (workspace) and outputs of its own, S = 1 .. 4: the
    steps of one stream run in order, those of different streams overlap, so
    one step's trajectory and risk stages and its collision kernel's tail
    share the GPU with the others' collision kernels. Every stream's results
    are checked bit for bit against the headline run's. Reported beside the
    headline value, which issues one step at a time."""
    import numpy as np
    ref = {k: (None if v is None else v.cpu().numpy()) for k, v in ref_out.items()}
    K = max(steps, 60)
    rows = []
    for S in (1, 2, 3, 4):
        plans = [mhc.mhc_plan_create(ctx, cs) for _ in range(S)]
        outs = [mhc.device_result(cs, first_hit=True, q=True) for _ in range(S)]
        streams = [torch.cuda.current_stream()] if S == 1 else [torch.cuda.Stream() for _ in range(S)]
        for k in range(4 * S):
            mhc.mhc_plan_execute(plans[k % S], outs[k % S][1], streams[k % S])
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for k in range(K):
            mhc.mhc_plan_execute(plans[k % S], outs[k % S][1], streams[k % S])
        torch.cuda.synchronize()
        us = (time.perf_counter() - t0) * 1e6 / K
        for o, _ in outs:
            for key in ("first_hit", "object_crit", "traj_crit", "traj_prob", "q"):
                if ref.get(key) is not None:
                    assert np.array_equal(o[key].cpu().numpy(), ref[key]), f"stream results differ: {key}"
        for pl in plans:
            pl.close()
        rows.append({"streams": S, "us_per_step": us, "checks_per_s": checks / (us * 1e-6), "steps": K})
        log(f"{S} stream(s), a plan each: {us:.1f} us per step -> {checks / (us * 1e-6):.4g} checks/s "
            f"(results identical)")
    return {"rows": rows, "note": "steps issued round-robin on S streams, one plan and output set per "
                                  "stream; every step a whole pass; results bitwise equal to the headline's"}


def polygon_extra(mhc, ctx, sg, torch, steps=50):
    """General convex outlines: every vehicle an octagonal car (corners
    chamfered 0.35 m). The 11-object scene (vehicle pairs 8 x 8 polygons,
    vehicle-pedestrian pairs polygon-circle) and the Table I S2 scene in both
    overlap modes: whole-path step and collision kernel alone (HIP events on
    the launch stream), against the same scene with rectangles."""
    stream = torch.cuda.current_stream()
    rows = []

    def octagons(s):
        for o in s.objects:
            if o.kind == sg.VEHICLE:
                o.outline = sg.car_outline(o.length, o.width)
        return s
    cases = [("eleven_object", lambda: sg.eleven_object_scene(1)),
             ("table_one_s2", lambda: sg.paper_scene(5, n_co=10)),
             ("table_one_s2_pip", lambda: sg.paper_scene(5, n_co=10, overlap=sg.OVERLAP_PIP))]
    for name, make in cases:
        row = {"workload": name}
        for shape in ("rectangles", "octagons"):
            s = make() if shape == "rectangles" else octagons(make())
            cs = mhc.CScene(s)
            checks = mhc.mhc_query_sizes(cs)["n_checks"]
            best, _ = mhc.mhc_autotune(ctx, cs, reps=10)
            plan = mhc.mhc_plan_create(ctx, cs)
            out, r = mhc.device_result(cs, first_hit=True, q=True)
            for _ in range(5):
                mhc.mhc_plan_execute(plan, r, stream)
            torch.cuda.synchronize()
            a = time.perf_counter()
            for _ in range(steps):
                mhc.mhc_plan_execute(plan, r, stream)
            torch.cuda.synchronize()
            step_us = (time.perf_counter() - a) * 1e6 / steps
            ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
            for k in range(steps):
                mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_TRAJ, r, stream)
                ev[k][0].record(stream)
                mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_COLLIDE, r, stream)
                ev[k][1].record(stream)
                mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_RISK, r, stream)
            torch.cuda.synchronize()
            k2_us = sum(x.elapsed_time(y) for x, y in ev) * 1e3 / steps
            plan.close()
            row[shape] = {"checks": checks, "step_us": step_us, "checks_per_s": checks / (step_us * 1e-6),
                          "collide_us": k2_us, "tile_variant": best}
        rows.append(row)
        r_, o_ = row["rectangles"], row["octagons"]
        log(f"polygons {name}: rectangles step {r_['step_us']:.1f} us collide {r_['collide_us']:.1f} us; octagons step "
            f"{o_['step_us']:.1f} us ({o_['checks_per_s']:.3g} checks/s), collide {o_['collide_us']:.1f} us")
    return rows


def models_extra(mhc, ctx, sg, torch, steps=50):
    """The paper's other motion models against the kinematic grids: the
    11-object scene with one-track vehicles and accelerating pedestrians
    (same grid sizes), and the Table I S2 scene with one-track vehicles:
    whole-path step and each module's time (HIP events on the launch
    stream). Both run a lane per step: the kinematic trajectories as prefix
    sums of closed-form increments, the one-track ones as a scan of the
    per-step affine maps of their lateral state."""
    stream = torch.cuda.current_stream()
    T, C, R = mhc.MHC_STAGE_TRAJ, mhc.MHC_STAGE_COLLIDE, mhc.MHC_STAGE_RISK

    def one_track_table_one():
        s = sg.paper_scene(5, n_co=10)
        for o in s.objects:
            o.model = sg.MODEL_ONE_TRACK
            o.params = sg.one_track_params(o.length)
            o.u = sg.accel_grid(6, -9.7, 9.7)
            o.w = sg.steer_grid(len(o.w))
            o.score = sg.vehicle_scores(o.u, o.w)
        return s
    rows = []
    for name, kin, mod in (("eleven_object", lambda: sg.eleven_object_scene(10), lambda: sg.models_scene(10)),
                           ("table_one_s2", lambda: sg.paper_scene(5, n_co=10), one_track_table_one)):
        row = {"workload": name}
        for label, make in (("kinematic", kin), ("paper_models", mod)):
            cs = mhc.CScene(make())
            plan = mhc.mhc_plan_create(ctx, cs)
            out, r = mhc.device_result(cs, first_hit=True, q=True)
            for _ in range(5):
                mhc.mhc_plan_execute(plan, r, stream)
            torch.cuda.synchronize()
            a = time.perf_counter()
            for _ in range(steps):
                mhc.mhc_plan_execute(plan, r, stream)
            torch.cuda.synchronize()
            step_us = (time.perf_counter() - a) * 1e6 / steps
            ev = [[torch.cuda.Event(enable_timing=True) for _ in range(4)] for _ in range(steps)]
            for k in range(steps):
                ev[k][0].record(stream)
                mhc.mhc_plan_execute_stages(plan, T, r, stream)
                ev[k][1].record(stream)
                mhc.mhc_plan_execute_stages(plan, C, r, stream)
                ev[k][2].record(stream)
                mhc.mhc_plan_execute_stages(plan, R, r, stream)
                ev[k][3].record(stream)
            torch.cuda.synchronize()
            mods = [sum(e[m].elapsed_time(e[m + 1]) for e in ev) * 1e3 / steps for m in range(3)]
            plan.close()
            row[label] = {"step_us": step_us, "traj_us": mods[0], "collide_us": mods[1], "risk_us": mods[2]}
        rows.append(row)
        k_, m_ = row["kinematic"], row["paper_models"]
        log(f"models {name}: kinematic step {k_['step_us']:.1f} us (trajectories {k_['traj_us']:.1f} us); "
            f"one-track / pedestrian acceleration step {m_['step_us']:.1f} us (trajectories {m_['traj_us']:.1f} us, "
            f"collide {m_['collide_us']:.1f} us)")
    return rows


# Measurements after the timed workload, in this order (--extras).
EXTRAS = ("latency", "streams", "batched", "served", "table_one", "timeline", "polygons", "models", "stress")

# Timed workloads: the 11-object scene is the headline; the Table I S2
# configuration (Sec. VI-B) can be timed the same way in either overlap mode.
WORKLOADS = ("eleven_object", "two_vehicle", "table_one_s2", "table_one_s2_pip", "table_one_s2_timeline", "table_one_s2_5",
             "table_one_s1", "table_one_s1_5", "eleven_object_octagons", "eleven_object_timeline",
             "eleven_object_models", "stress")


def make_workload(name, seed, sg):
    """(scene, metric label, config, description) of a timed workload."""
    if name.startswith("eleven_object"):
        variant = name[len("eleven_object"):].lstrip("_") or "plain"
        scene = {"plain": sg.eleven_object_scene, "octagons": sg.polygon_scene,
                 "models": sg.models_scene, "timeline": sg.eleven_object_scene}[variant](seed)
        if variant == "timeline":
            scene.timeline = 1
        cfg = {"workload": "eleven_object_scene", "objects": 11, "vehicles": 6, "pedestrians": 5,
               "trajectories_per_object": 225, "horizon": 30, "dt": 0.1, "seed": seed, "pairs": "all",
               "overlap": "exact"}
        label = "11-object scene"
        if variant == "octagons":
            cfg["vehicle_shape"] = "octagonal outline (corners cut 0.35 m)"
            label += ", octagonal cars"
        elif variant == "timeline":
            cfg["risk_over_time"] = True
            label += ", risk over time"
        elif variant == "models":
            cfg["motion_models"] = "one-track vehicles, accelerating pedestrians capped at 2.7 m/s"
            label += ", one-track / pedestrian acceleration models"
        return scene, label, cfg, f"{label} seed {seed}"
    if name == "two_vehicle":
        scene = sg.two_vehicle_scene(seed)
        cfg = {"workload": "two_vehicle_scene", "objects": 2, "vehicles": 2, "pedestrians": 0,
               "trajectories_per_object": 25, "horizon": 30, "dt": 0.1, "seed": seed, "pairs": "all",
               "overlap": "exact"}
        return scene, "two-vehicle scene", cfg, f"two-vehicle scene seed {seed}"
    if name == "stress":
        scene = sg.stress_scene(seed)
        cfg = {"workload": "stress_scene", "objects": 40, "vehicles": 24, "pedestrians": 16,
               "trajectories_per_object": 1024, "horizon": 50, "dt": 0.1, "seed": seed, "pairs": "all",
               "overlap": "exact"}
        return scene, "40-object stress scene", cfg, f"40-object stress scene seed {seed}"
    pip = name.endswith("_pip")
    tl = name.endswith("_timeline")
    s1 = name.startswith("table_one_s1")
    n_acc = 5 if name.endswith("_5") else 6
    n_co = 3 if s1 else 10
    scene = sg.paper_scene(seed, n_co=n_co, n_acc=n_acc, overlap=sg.OVERLAP_PIP if pip else sg.OVERLAP_EXACT)
    scene.timeline = 1 if tl else 0
    cfg = {"workload": f"table_one_{'s1' if s1 else 's2'}_scene", "objects": n_co + 1, "vehicles": n_co + 1,
           "pedestrians": 0, "trajectories": {"ego": n_acc * 343, "co": n_acc * 7}, "horizon": 100, "dt": 0.02,
           "seed": seed, "pairs": "ego", "overlap": "pip" if pip else "exact"}
    label = (f"Table I {'S1' if s1 else 'S2'} scene" + (", 5 profiles" if n_acc == 5 else "")
             + (", point-in-polygon" if pip else "") + (", risk over time" if tl else ""))
    if tl:
        cfg["risk_over_time"] = True
    return scene, label, cfg, f"{label} seed {seed}"


def recorded_traffic(variant, workload):
    """HBM bytes per collision stage from the committed counter runs
    (profiles/k2_collide_eleven_object_traffic.txt, one FETCH_SIZE and one
    WRITE_SIZE figure per tile variant), each counter scaled by what it reads
    for a plain copy kernel of known size; None when the kernel sources differ
    from those the counters were taken on or the variant has no record."""
    import hashlib
    path = os.path.join(ROOT, "profiles", "k2_collide_eleven_object_traffic.txt")
    if workload != "eleven_object" or not os.path.exists(path):
        return None
    rec = {}
    for line in open(path):
        if "=" in line and not line.lstrip().startswith("#"):
            k, v = line.split("=", 1)
            rec[k.strip()] = v.strip()
    h = hashlib.sha256()
    for f in ("paper_2005_06773_amd/csrc/kernels.hip", "paper_2005_06773_amd/csrc/mhc_internal.h"):
        h.update(open(os.path.join(ROOT, f), "rb").read())
    fkey, wkey = f"fetch_kib_per_dispatch[{variant}]", f"write_kib_per_dispatch[{variant}]"
    if rec.get("kernel_source_sha256") != h.hexdigest() or fkey not in rec or wkey not in rec:
        return None
    copy_kib = float(rec["copy_mib"]) * 1024.0
    fetch = float(rec[fkey]) * copy_kib / float(rec["copy_fetch_kib"])
    write = float(rec[wkey]) * copy_kib / float(rec["copy_write_kib"])
    return (fetch + write) * 1024.0


def pct(xs, q):
    xs = sorted(xs)
    k = min(len(xs) - 1, max(0, int(math.ceil(q / 100.0 * len(xs))) - 1))
    return xs[k]


def cpu_baseline(scene, checks, seconds, described, pair_list=None):
    """The FP64 oracle as it stands, on the host cores (rank 0, N=1 only).
    ``pair_list`` restricts it to a sample of object pairs (the stress scene,
    whose full pass takes the oracle minutes); the rate is then the sample's
    checks per second."""
    import oracle
    oracle.lib()
    nproc = os.cpu_count() or 1
    cores = min(16, nproc)
    if pair_list is not None:
        T = scene.traj_counts()
        checks = sum(T[a] * T[b] for a, b in pair_list) * scene.horizon

    def timed(threads, budget):
        t0 = time.perf_counter()
        runs = 0
        while True:
            oracle.evaluate(scene, pair_list=pair_list, threads=threads, masks=False)
            runs += 1
            if time.perf_counter() - t0 >= budget:
                break
        return runs, time.perf_counter() - t0

    runs, dt = timed(cores, seconds)
    value = checks * runs / dt
    log(f"cpu baseline: {runs} oracle runs in {dt:.2f} s on {cores} threads -> {value:.4g} checks/s")
    # the same oracle on every thread the host reports, and on one thread
    runs_n, dt_n = timed(nproc, seconds / 3) if nproc != cores else (runs, dt)
    log(f"cpu baseline, {nproc} threads (nproc): {runs_n} oracle runs in {dt_n:.2f} s -> "
        f"{checks * runs_n / dt_n:.4g} checks/s")
    runs_1, dt1 = timed(1, 0.0)
    log(f"cpu baseline, one thread: one oracle run in {dt1:.2f} s -> {checks / dt1:.4g} checks/s")
    what = "the full timed scene" if pair_list is None else f"{len(pair_list)} sampled object pairs of"
    return {"value": value, "unit": "checks/s", "cores": cores, "kind": "oracle",
            "sample": f"{what} ({described}), {runs} complete oracle passes "
                      f"(trajectories, {checks:,} checks, risk) in {dt:.1f} s",
            "cpu_model": cpu_model(), "nproc": nproc,
            "value_nproc": checks * runs_n / dt_n, "value_one_thread": checks / dt1}


def cpu_model():
    """The host CPU's model name (first 'model name' of /proc/cpuinfo)."""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def serve(mhc, ctx, sg, seconds):
    """Serving workload: 32 streams, each a Poisson process at 10 Hz with a
    start offset in U(0, 100 ms), frames drawn as in the batched workload
    (seed 3), replayed in real time; then the same arrivals through a plain
    per-frame mhc_evaluate loop. Latency = scheduled arrival -> results in
    host memory, for both."""
    import threading
    warm = 1.0
    events = [e for e in sg.serving_schedule(3, 32, 10.0, seconds, warm)]
    frames = [(t, sid, mhc.CScene(sc)) for t, sid, sc in events]
    checks = [mhc.mhc_query_sizes(c)["n_checks"] for _, _, c in frames]
    srv = mhc.Server(ctx, budget=4 << 30, inflight=2)
    tickets = []
    done = {}

    def waiter():
        k = 0
        while k < len(frames):
            while len(tickets) <= k:
                time.sleep(0.0002)
            t_ticket = tickets[k]
            _, timing = srv.wait(t_ticket)
            done[k] = timing
            k += 1

    w = threading.Thread(target=waiter)
    w.start()
    # the server stamps completion on the monotonic clock, the one
    # time.monotonic_ns reads: latency runs from each frame's scheduled
    # arrival, so time spent submitting counts against the server
    t0 = time.monotonic_ns()
    for t, sid, cs in frames:
        at = t0 + int(t * 1e9)
        while time.monotonic_ns() < at:
            time.sleep(0.0001)
        tickets.append(srv.submit(sid, cs))
    w.join()
    srv.stop()
    lat = [(done[k]["done_ns"] - (t0 + int(frames[k][0] * 1e9))) * 1e-6
           for k in range(len(frames)) if frames[k][0] >= warm]
    busy_checks = sum(c for (t, _, _), c in zip(frames, checks) if t >= warm)
    out = {"streams": 32, "rate_hz_per_stream": 10, "seconds": seconds, "frames": len(lat),
           "p50_ms": pct(lat, 50), "p99_ms": pct(lat, 99), "max_ms": max(lat),
           "deadline_ms": 50.0, "within_deadline": sum(x <= 50.0 for x in lat) / len(lat),
           "sustained_checks_per_s": busy_checks / seconds}
    # the same arrivals through the plain per-frame loop, timed the same way
    lat2 = []
    t0 = time.monotonic_ns()
    for (t, sid, cs) in frames:
        at = t0 + int(t * 1e9)
        while time.monotonic_ns() < at:
            time.sleep(0.0001)
        mhc.mhc_evaluate(ctx, cs, first_hit=False, q=False)
        if t >= warm:
            lat2.append((time.monotonic_ns() - at) * 1e-6)
    out["plain_loop"] = {"p50_ms": pct(lat2, 50), "p99_ms": pct(lat2, 99), "max_ms": max(lat2),
                         "within_deadline": sum(x <= 50.0 for x in lat2) / len(lat2)}
    log(f"served: {len(lat)} frames, p50 {out['p50_ms']:.2f} ms p99 {out['p99_ms']:.2f} ms "
        f"({out['sustained_checks_per_s']:.3g} checks/s offered); plain loop p50 {out['plain_loop']['p50_ms']:.2f} "
        f"ms p99 {out['plain_loop']['p99_ms']:.2f} ms")
    out["with_stress_frames"] = serve_mixed(mhc, ctx, sg, frames, warm, seconds)
    return out


def serve_mixed(mhc, ctx, sg, frames, warm, seconds, period_s=0.25):
    """The same served arrivals with a 40-object stress frame (4.09e10
    checks, above the per-tick check cap, so it rides in a tick of its own)
    arriving every period_s: latency of the small frames from their
    scheduled arrival, beside that of the stress frames."""
    import threading
    big = mhc.CScene(sg.stress_scene(4))
    events = [(t, sid, cs, False) for t, sid, cs in frames]
    t = 0.05
    while t < warm + seconds:
        events.append((t, 99, big, True))
        t += period_s
    events.sort(key=lambda e: e[0])
    srv = mhc.Server(ctx, budget=4 << 30, inflight=2)
    tickets, done = [], {}

    def waiter():
        k = 0
        while k < len(events):
            while len(tickets) <= k:
                time.sleep(0.0002)
            _, timing = srv.wait(tickets[k])
            done[k] = timing
            k += 1

    w = threading.Thread(target=waiter)
    w.start()
    t0 = time.monotonic_ns()
    for at_s, sid, cs, _ in events:
        at = t0 + int(at_s * 1e9)
        while time.monotonic_ns() < at:
            time.sleep(0.0001)
        tickets.append(srv.submit(sid, cs))
    w.join()
    srv.stop()
    small = [(done[k]["done_ns"] - (t0 + int(events[k][0] * 1e9))) * 1e-6
             for k in range(len(events)) if events[k][0] >= warm and not events[k][3]]
    large = [(done[k]["done_ns"] - (t0 + int(events[k][0] * 1e9))) * 1e-6
             for k in range(len(events)) if events[k][0] >= warm and events[k][3]]
    out = {"stress_frame_period_s": period_s, "small_frames": len(small), "stress_frames": len(large),
           "small_p50_ms": pct(small, 50), "small_p99_ms": pct(small, 99), "small_max_ms": max(small),
           "small_within_deadline": sum(x <= 50.0 for x in small) / len(small),
           "stress_p50_ms": pct(large, 50), "stress_max_ms": max(large)}
    log(f"served with a stress frame every {period_s} s: small frames p50 {out['small_p50_ms']:.2f} ms "
        f"p99 {out['small_p99_ms']:.2f} ms; stress frames p50 {out['stress_p50_ms']:.1f} ms")
    return out


def stress_extra(mhc, ctx, sg, torch, steps=10):
    """The 40-object stress scene (24 vehicles + 16 pedestrians, 32 x 32
    grids, 50 steps, 40,894,464,000 checks): whole-path step and collision
    kernel alone, with and without the 1.64 GB first-hit output."""
    stream = torch.cuda.current_stream()
    s = sg.stress_scene(4)
    cs = mhc.CScene(s)
    checks = mhc.mhc_query_sizes(cs)["n_checks"]
    best, us = mhc.mhc_autotune(ctx, cs, reps=3)
    out = {"workload": "stress_scene", "objects": 40, "trajectories_per_object": 1024, "horizon": 50,
           "checks": checks, "tile_variant": best}
    for fh in (False, True):
        plan = mhc.mhc_plan_create(ctx, cs)
        outs, r = mhc.device_result(cs, first_hit=fh, q=True)
        for _ in range(2):
            mhc.mhc_plan_execute(plan, r, stream)
        torch.cuda.synchronize()
        a = time.perf_counter()
        for _ in range(steps):
            mhc.mhc_plan_execute(plan, r, stream)
        torch.cuda.synchronize()
        step_ms = (time.perf_counter() - a) * 1e3 / steps
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
        for k in range(steps):
            mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_TRAJ, r, stream)
            ev[k][0].record(stream)
            mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_COLLIDE, r, stream)
            ev[k][1].record(stream)
            mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_RISK, r, stream)
        torch.cuda.synchronize()
        k2_ms = sum(x.elapsed_time(y) for x, y in ev) / steps
        plan.close()
        del outs, r
        key = "with_first_hit" if fh else "criticality_only"
        out[key] = {"step_ms": step_ms, "checks_per_s": checks / (step_ms * 1e-3), "collide_ms": k2_ms}
        log(f"stress scene ({key}): step {step_ms:.2f} ms ({checks / (step_ms * 1e-3):.4g} checks/s), "
            f"collide {k2_ms:.2f} ms")
    torch.cuda.empty_cache()
    return out


def sweep_arrivals(streams, seconds, warm, rate, n_pool):
    """Poisson arrivals of `streams` streams at `rate` Hz over warm + seconds
    (start offsets U(0, 100 ms)), with the stream of each arrival and the
    pool frame it carries; the same draws for the served and the plain
    sweep at a given load."""
    import numpy as np
    rng = np.random.default_rng(1000 + streams)
    arr, sid = [], []
    for s in range(streams):
        t = float(rng.uniform(0.0, 0.1))
        gaps = rng.exponential(1.0 / rate, int((warm + seconds) * rate * 3) + 20)
        ts = t + np.concatenate([[0.0], np.cumsum(gaps)])
        arr.append(ts[ts < warm + seconds])
        sid.append(np.full(arr[-1].size, s))
    order = np.argsort(np.concatenate(arr), kind="stable")
    arrivals = np.concatenate(arr)[order]
    stream_of = np.concatenate(sid)[order]
    which = rng.integers(0, n_pool, arrivals.size)
    return arrivals, stream_of, which


def plain_sweep(mhc, ctx, sg, seconds, streams_list=(32, 128, 256, 384, 512, 640, 768, 1024)):
    """The served load sweep's arrivals (same streams, draws and frame pool)
    through the plain per-frame loop: each frame evaluated by mhc_evaluate
    when the loop reaches it, latency from its scheduled arrival to its
    results in host memory. Stops at the first load whose p99 passes 50 ms
    and reports the largest sustained rate within the deadline, the
    comparison point of the served sweep."""
    scenes = sg.batch_scenes(3, 512)
    pool = [mhc.CScene(s) for s in scenes]
    pool_checks = [mhc.mhc_query_sizes(c)["n_checks"] for c in pool]
    warm, rate, deadline = 0.5, 10.0, 50.0
    points, best = [], None
    for c in pool[:16]:
        mhc.mhc_evaluate(ctx, c, first_hit=False, q=False)
    for streams in streams_list:
        arrivals, _, which = sweep_arrivals(streams, seconds, warm, rate, len(pool))
        lat, chk = [], 0
        t0 = time.monotonic_ns()
        end = t0
        for k in range(arrivals.size):
            at = t0 + int(arrivals[k] * 1e9)
            while time.monotonic_ns() < at:
                time.sleep(0.00005)
            mhc.mhc_evaluate(ctx, pool[which[k]], first_hit=False, q=False)
            end = time.monotonic_ns()
            if arrivals[k] >= warm:
                lat.append((end - at) * 1e-6)
                chk += pool_checks[which[k]]
        span = (end - (t0 + int(warm * 1e9))) * 1e-9
        pt = {"streams": streams, "frames": len(lat), "p50_ms": pct(lat, 50), "p99_ms": pct(lat, 99),
              "max_ms": max(lat), "completed_checks_per_s": chk / span,
              "within_deadline": sum(x <= deadline for x in lat) / len(lat)}
        points.append(pt)
        log(f"plain loop sweep: {streams} streams, {len(lat)} frames, p50 {pt['p50_ms']:.2f} ms p99 "
            f"{pt['p99_ms']:.2f} ms, {pt['completed_checks_per_s']:.4g} checks/s")
        if pt["p99_ms"] > deadline:
            break
        best = pt
    return {"rate_hz_per_stream": rate, "seconds_per_point": seconds, "deadline_ms": deadline, "points": points,
            "max_sustained_checks_per_s_within_deadline": None if best is None else best["completed_checks_per_s"],
            "at_streams": None if best is None else best["streams"]}


def serve_sweep(mhc, ctx, sg, seconds,
                streams_list=(32, 256, 512, 768, 1024, 1280, 1536, 1792, 2048, 2304, 2560, 3072, 3584, 4096)):
    """Served load sweep: the serving workload with more and more 10 Hz
    Poisson streams until the p99 latency passes the 50 ms deadline. Frames
    come from a pool of 512 drawn as in the batched workload (seed 3) and are
    submitted in real time; latency runs from each frame's scheduled arrival
    (the server's own monotonic clock) to its results in host memory, so a
    submitter that falls behind counts against the server. Reports, per load,
    p50/p99 and the completed checks per second, and the largest sustained
    rate whose p99 meets the deadline."""
    import ctypes
    import threading
    import numpy as np
    scenes = sg.batch_scenes(3, 512)
    pool = [mhc.CScene(s) for s in scenes]
    pool_checks = [mhc.mhc_query_sizes(c)["n_checks"] for c in pool]
    n_max = max(s.n_objects for s in scenes)
    t_max = max(mhc.mhc_query_sizes(c)["n_traj"] for c in pool)
    ring = 4096
    bufs = [(np.empty(n_max), np.empty(t_max)) for _ in range(ring)]
    dsts = [mhc.mhc_result(oc.ctypes.data, tc.ctypes.data, *([None] * (len(mhc.RESULT_FIELDS) - 2)))
            for oc, tc in bufs]
    warm, rate, deadline = 0.5, 10.0, 50.0
    points, best = [], None
    for streams in streams_list:
        arrivals, stream_of, which = sweep_arrivals(streams, seconds, warm, rate, len(pool))
        srv = mhc.Server(ctx, budget=4 << 30, inflight=2)
        n = arrivals.size
        tickets = [0] * n
        done_ns = [0] * n
        submitted = [0]
        completed = [0]
        busy = [0]

        def waiter():
            tm = mhc.mhc_timing()
            for k in range(n):
                while submitted[0] <= k:
                    time.sleep(0.0002)
                if tickets[k] < 0:
                    completed[0] = k + 1
                    continue
                st = mhc.lib.mhc_wait(srv.h, tickets[k], -1, ctypes.byref(tm))
                if st != mhc.MHC_OK:
                    raise RuntimeError(f"mhc_wait: {st}")
                done_ns[k] = tm.done_ns
                completed[0] = k + 1

        w = threading.Thread(target=waiter)
        w.start()
        t0 = time.monotonic_ns()
        tk = ctypes.c_uint64()
        for k in range(n):
            at = t0 + int(arrivals[k] * 1e9)
            while time.monotonic_ns() < at:
                time.sleep(0.00005)
            while completed[0] <= k - ring:          # the ring slot is still in flight
                if not w.is_alive():
                    raise RuntimeError("served sweep: waiter thread ended early")
                time.sleep(0.0002)
            st = mhc.lib.mhc_submit(srv.h, int(stream_of[k]), ctypes.byref(pool[which[k]].c),
                                    ctypes.byref(dsts[k % ring]), ctypes.byref(tk))
            if st == mhc.MHC_E_BUSY:
                tickets[k] = -1
                busy[0] += 1
            elif st != mhc.MHC_OK:
                raise mhc.MhcError(st, mhc.mhc_last_error(ctx))
            else:
                tickets[k] = tk.value
            submitted[0] = k + 1
        w.join()
        srv.stop()
        sel = [k for k in range(n) if arrivals[k] >= warm]
        lat = [(done_ns[k] - (t0 + int(arrivals[k] * 1e9))) * 1e-6 if tickets[k] >= 0 else float("inf")
               for k in sel]
        span = max(done_ns[k] for k in sel if tickets[k] >= 0) - (t0 + int(warm * 1e9))
        chk = sum(pool_checks[which[k]] for k in sel if tickets[k] >= 0)
        pt = {"streams": streams, "frames": len(sel), "rejected_busy": busy[0],
              "offered_checks_per_s": sum(pool_checks[which[k]] for k in sel) / seconds,
              "completed_checks_per_s": chk / (span * 1e-9),
              "p50_ms": pct(lat, 50), "p99_ms": pct(lat, 99), "max_ms": max(lat),
              "within_deadline": sum(x <= deadline for x in lat) / len(lat)}
        points.append(pt)
        log(f"served sweep: {streams} streams, {len(sel)} frames, p50 {pt['p50_ms']:.2f} ms p99 "
            f"{pt['p99_ms']:.2f} ms, {pt['completed_checks_per_s']:.4g} checks/s")
        if pt["p99_ms"] > deadline:
            break
        best = pt
    return {"rate_hz_per_stream": rate, "seconds_per_point": seconds, "deadline_ms": deadline,
            "pool_frames": len(pool), "points": points,
            "max_sustained_checks_per_s_within_deadline": None if best is None else best["completed_checks_per_s"],
            "at_streams": None if best is None else best["streams"]}


def main():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=300)
    ap.add_argument("--warmup", type=int, default=30)
    ap.add_argument("--workload", choices=WORKLOADS, default="eleven_object",
                    help="timed workload (default: the 11-object scene)")
    ap.add_argument("--seed", type=int, default=None, help="scene seed (default 1; 5 for the Table I scenes)")
    ap.add_argument("--cpu-seconds", type=float, default=12.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true", help="skip the latency and batched measurements")
    ap.add_argument("--extras", default=",".join(EXTRAS),
                    help="comma-separated extras to run (default: all of " + ", ".join(EXTRAS) + ")")
    ap.add_argument("--serve-seconds", type=float, default=4.0,
                    help="length of the served-load measurement (after 1 s of warm-up)")
    ap.add_argument("--serve-sweep-seconds", type=float, default=1.5,
                    help="length of each point of the served load sweep (0: no sweep)")
    ap.add_argument("--variant", type=int, default=-1,
                    help="force a collision micro-tile variant (default: autotune on the workload)")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="MIB",
                    help="also run one plain device copy of MIB MiB (reference for HBM byte counters)")
    args = ap.parse_args()
    extras = set() if args.no_extras else {e for e in args.extras.split(",") if e}
    if extras - set(EXTRAS):
        sys.exit(f"bench.py: unknown extras {sorted(extras - set(EXTRAS))}; choose from {', '.join(EXTRAS)}")
    if args.gpus != 1:
        print(f"bench.py measures one GPU only; --gpus {args.gpus} is not supported "
              "(the path would shard object pairs across GPUs)", file=sys.stderr)
        sys.exit(2)
    if args.seed is None:
        args.seed = {"eleven_object": 1, "eleven_object_octagons": 1, "eleven_object_timeline": 1,
                     "eleven_object_models": 10, "stress": 4, "two_vehicle": 0}.get(args.workload, 5)

    import torch
    from paper_2005_06773_amd import mhc, scenegen as sg

    scene, label, config, described = make_workload(args.workload, args.seed, sg)
    cs = mhc.CScene(scene)
    sizes = mhc.mhc_query_sizes(cs)
    checks = sizes["n_checks"]

    # Set-up that leaves the GPU idle (torch's first allocations and kernels)
    # comes before the autotune, so that the warm-up steps follow the
    # autotune's launches directly: after tens of milliseconds of idling the
    # collision kernel takes ~15 ms of continuous launches to come back to
    # its steady duration (38.5 -> 34.4 us on the 11-object scene).
    out, r = mhc.device_result(cs, first_hit=True, q=True)
    stream = torch.cuda.current_stream()
    torch.cuda.synchronize()
    ctx = mhc.mhc_create(0)
    if args.variant >= 0:
        mhc.mhc_set_variant(ctx, args.variant)
        tune = {"forced": args.variant}
        variant = args.variant
    else:
        best, us = mhc.mhc_autotune(ctx, cs, reps=20)
        tune = {"chosen": best, "us_per_variant": [round(u, 2) for u in us]}
        variant = best
    plan = mhc.mhc_plan_create(ctx, cs)
    if args.variant < 0:
        log(f"autotune: collision kernel us per variant {[round(u, 1) for u in us]} -> variant {best}")
    T, C, R = mhc.MHC_STAGE_TRAJ, mhc.MHC_STAGE_COLLIDE, mhc.MHC_STAGE_RISK

    if args.calibrate_copy:
        # one plain elementwise kernel that reads MIB MiB and writes MIB MiB
        src = torch.ones(args.calibrate_copy * (1 << 20) // 4, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        torch.mul(src, 1.0, out=dst)
        torch.cuda.synchronize()
        log(f"calibration copy: {args.calibrate_copy} MiB read, {args.calibrate_copy} MiB written")
        del src, dst
    log(f"workload: {described}, {checks:,} checks/pass; warmup {args.warmup}, steps {args.steps}")
    for _ in range(args.warmup):
        mhc.mhc_plan_execute(plan, r, stream)
    torch.cuda.synchronize()

    # Timed region: K whole-path steps on the launch stream.
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        mhc.mhc_plan_execute(plan, r, stream)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_step = (t1 - t0) * 1e3 / args.steps
    value = checks / (ms_step / 1e3)

    # Collision-kernel duration, live, on the launch stream. (a) The way a
    # kernel trace sees it: K collision launches back to back between two HIP
    # events (the trajectory stage runs once before them; the repeated
    # launches add to the same q sums, which only the timing uses, and a whole
    # step afterwards restores the results). (b) Every collision launch of K
    # whole steps bracketed by its own pair of events, which adds each
    # launch's start-up to its time (reported beside it).
    mhc.mhc_plan_execute_stages(plan, T, r, stream)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(args.steps):
        mhc.mhc_plan_execute_stages(plan, C, r, stream)
    e1.record(stream)
    torch.cuda.synchronize()
    k2_ms = e0.elapsed_time(e1) / args.steps
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    for k in range(args.steps):
        mhc.mhc_plan_execute_stages(plan, T, r, stream)
        ev[k][0].record(stream)
        mhc.mhc_plan_execute_stages(plan, C, r, stream)
        ev[k][1].record(stream)
        mhc.mhc_plan_execute_stages(plan, R, r, stream)
    torch.cuda.synchronize()
    k2_bracketed_ms = sum(a.elapsed_time(b) for a, b in ev) / args.steps

    # The same steps replayed as one captured HIP graph per step (reported only).
    mhc.mhc_plan_set_graph(plan, True)
    for _ in range(5):
        mhc.mhc_plan_execute(plan, r, stream)
    torch.cuda.synchronize()
    a = time.perf_counter()
    for _ in range(args.steps):
        mhc.mhc_plan_execute(plan, r, stream)
    torch.cuda.synchronize()
    graph_step_us = (time.perf_counter() - a) * 1e6 / args.steps
    mhc.mhc_plan_set_graph(plan, False)
    traffic = recorded_traffic(variant, args.workload)
    achieved = None if traffic is None else traffic / (k2_ms * 1e-3) / 1e12
    log(f"step {ms_step * 1e3:.1f} us -> {value:.4g} checks/s; collision kernel {k2_ms * 1e3:.1f} us back to back "
        f"({k2_bracketed_ms * 1e3:.1f} us bracketed per launch)")

    result = {
        "metric": f"pose-pair checks/sec ({label})",
        "value": value,
        "unit": "checks/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": dict(config, checks=checks, inputs="resident in HBM"),
        "tile_variant": tune,
        "graph_step_us": graph_step_us,
        "counting": "checks decided; most of them together, by bounds of groups of trajectories",
        # The collision stage (clearing the first hits and the collision
        # kernel) by the HBM bytes it moves: with the bounds it is limited by
        # the latency of its dependent reads, far from any rate.
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_TB_S, "unit": "TB/s",
                     "frac": None if achieved is None else achieved / PEAK_HBM_TB_S, "traffic": traffic,
                     "kernel": "k2_collide", "kernel_us": k2_ms * 1e3,
                     "kernel_us_timing": "mean of K back-to-back collision stages between two HIP events on the "
                                         "launch stream",
                     "kernel_us_bracketed": k2_bracketed_ms * 1e3},
    }

    # Sanity: the results of a whole step are finite and in range.
    mhc.mhc_plan_execute(plan, r, stream)
    torch.cuda.synchronize()
    oc = out["object_crit"].cpu()
    assert torch.isfinite(oc).all() and (oc >= 0).all() and (oc <= 1).all(), "bad criticality"

    if "latency" in extras:
        # Plain end-to-end latency: host scene in -> host criticality out.
        lat = []
        for _ in range(10):
            mhc.mhc_evaluate(ctx, cs, first_hit=False, q=False)
        for _ in range(200):
            a = time.perf_counter()
            mhc.mhc_evaluate(ctx, cs, first_hit=False, q=False)
            lat.append((time.perf_counter() - a) * 1e3)
        result["plain_latency_ms"] = {"p50": pct(lat, 50), "p99": pct(lat, 99), "max": max(lat),
                                      "note": "mhc_evaluate, host scene in, host criticality out (PCIe included)"}
        log(f"plain end-to-end latency p50 {pct(lat, 50):.3f} ms p99 {pct(lat, 99):.3f} ms")
    if "streams" in extras:
        result["streams"] = streams_extra(mhc, ctx, cs, checks, out, args.steps, torch)
    if "batched" in extras:
        # Batched vs plain loop over the same 64 scenes; the batch's tile
        # variant is autotuned on the batch itself first.
        scenes = [mhc.CScene(s) for s in sg.batch_scenes(2, 64)]
        bchecks = sum(mhc.mhc_query_sizes(s)["n_checks"] for s in scenes)
        bbest, bus = mhc.mhc_autotune_batch(ctx, scenes, reps=5)
        log(f"batch autotune: collision kernel us per variant {[round(u, 1) for u in bus]} -> variant {bbest}")
        mhc.mhc_evaluate_batch(ctx, scenes, first_hit=False, q=False)
        for s in scenes[:4]:
            mhc.mhc_evaluate(ctx, s, first_hit=False, q=False)
        reps = 10
        a = time.perf_counter()
        for _ in range(reps):
            mhc.mhc_evaluate_batch(ctx, scenes, first_hit=False, q=False)
        tb = (time.perf_counter() - a) / reps
        a = time.perf_counter()
        for _ in range(reps):
            for s in scenes:
                mhc.mhc_evaluate(ctx, s, first_hit=False, q=False)
        tp = (time.perf_counter() - a) / reps
        result["batched"] = {"scenes": 64, "checks": bchecks, "batch_ms": tb * 1e3, "plain_loop_ms": tp * 1e3,
                             "batch_checks_per_s": bchecks / tb, "plain_loop_checks_per_s": bchecks / tp,
                             "speedup": tp / tb,
                             "tile_variant": {"chosen": bbest, "collide_us_per_variant": [round(u, 2) for u in bus],
                                              "gain_over_default": bus[0] / bus[bbest]}}
        log(f"batched 64 scenes: {tb * 1e3:.2f} ms ({bchecks / tb:.4g} checks/s) vs plain loop "
            f"{tp * 1e3:.2f} ms ({bchecks / tp:.4g} checks/s)")

    if "served" in extras:
        result["served"] = serve(mhc, ctx, sg, args.serve_seconds)
        if args.serve_sweep_seconds > 0:
            result["served_sweep"] = serve_sweep(mhc, ctx, sg, args.serve_sweep_seconds)
            result["plain_loop_sweep"] = plain_sweep(mhc, ctx, sg, args.serve_sweep_seconds)
    for name, fn in (("table_one", table_one), ("timeline", timeline_extra), ("polygons", polygon_extra),
                     ("models", models_extra), ("stress", stress_extra)):
        if name in extras:
            result[name] = fn(mhc, ctx, sg, torch)

    plan.close()
    mhc.mhc_destroy(ctx)

    if not args.no_cpu_baseline:
        sample = sg.stress_sample_pairs(scene.n_objects, 20, 1004) if args.workload == "stress" else None
        result["cpu_baseline"] = cpu_baseline(scene, checks, args.cpu_seconds, described, sample)
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
