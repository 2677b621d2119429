#!/usr/bin/env python3
"""Multi-tenant throughput benchmark on one MI355X.

A step is one round: every tenant of the workload runs once (inputs, weights and activations
resident in HBM).  Three executions of the same kernels are timed: sequential (one stream, unsplit),
stream-parallel (one stream per tenant, unsplit, no ordering) and regulated (the chosen plan:
operator chunks + pointer edges).  ``value`` is the regulated aggregate items/s of the headline
workload (configs[1]); ``per_config`` carries the same measurements for configs[2..4], ``paper_mixes`` for three tenant
mixes of the paper's own evaluation (its Table 2) that need no dataset.

Prints ONE JSON line, short enough for readers that keep only the end of a program's output; the full record of every
workload (kernel tables, percentiles, plan selection) goes to stderr.  Plan selection (profile, search, short trials) happens before the timed
region, as in offline deployment (Section 4.4, "Search Cost Analysis").
"""
import argparse
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK = {"f32": 157.3e12, "bf16": 2.5e15}        # dense MFMA FLOP/s, MI355X
HBM_PEAK = 8.0e12


# HBM-side traffic of the dominant kernel per launch, from two rocprofv3 counter passes (FETCH_SIZE, WRITE_SIZE, KiB per
# dispatch, scaled by what the same counters read for a plain copy of known size).  Valid only for the kernel sources the
# counters were taken with (the digest below covers them: any change resets `traffic` to null) and for the plan they were
# taken on: per-launch bytes change when the chosen plan decomposes operators of this kernel, so `traffic` is reported only
# when the kernel's launches per round equal the profiled count; the profiled figure itself is always given beside it.
TRAFFIC = {
    2: {"kernel": "igemm_dma_taps_f32_64x64x32s3", "fetch_bytes": 12.39e6, "write_bytes": 5.47e6, "plan": "unsplit",
        "launches_per_round": 11, "algorithmic_bytes": 12.45e6,
        "sources_sha256": "80f07e3788111b24679abb2a698cf770ec2ee00bf57e95854c05bbc3bfd62952"},
}
TRAFFIC_SOURCES = ["igemm.hip", "slices.hip", "rows.hip", "stream_ops.hip", "gemm_util.h", "slices_geom.h", "device_util.h", "kernels.h"]


def sources_digest():
    import hashlib
    h = hashlib.sha256()
    for f in TRAFFIC_SOURCES:
        with open(os.path.join(ROOT, "paper_2304_11745_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def measured_traffic(config, kernel, launches_per_round):
    """(traffic, profiled): bytes per launch for the roofline object (None unless kernel, sources and launch count match
    what the counters were taken on) and the profiled record itself (None unless kernel and sources match)."""
    t = TRAFFIC.get(config)
    if not t or t["kernel"] != kernel or t["fetch_bytes"] is None or t["sources_sha256"] != sources_digest():
        return None, None
    profiled = {"bytes_per_launch": t["fetch_bytes"] + t["write_bytes"], "fetch_bytes": t["fetch_bytes"],
                "write_bytes": t["write_bytes"], "algorithmic_bytes_per_launch": t["algorithmic_bytes"],
                "plan": t["plan"], "launches_per_round": t["launches_per_round"]}
    return (profiled["bytes_per_launch"] if launches_per_round == t["launches_per_round"] else None), profiled


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def rounded(v):
    """Floats to six significant digits, all the way down."""
    if isinstance(v, dict):
        return {k: rounded(x) for k, x in v.items()}
    if isinstance(v, (list, tuple)):
        return [rounded(x) for x in v]
    return float(f"{v:.6g}") if isinstance(v, float) else v


def summary(r):
    """What the line says about a workload other than the headline one."""
    s = {k: r[k] for k in ("workload", "dtype", "plan", "plan_kind", "launches_per_round", "ms_per_step", "regulated_images_per_s",
                           "sequential_images_per_s", "stream_parallel_images_per_s", "speedup_vs_sequential",
                           "speedup_vs_stream_parallel", "issue_threads")}
    s["mfma_frac_of_peak"] = r["mfma_frac_of_peak"]["regulated"]
    if r.get("roofline"):
        s["roofline"] = {k: r["roofline"].get(k) for k in ("kernel", "bound", "achieved", "peak", "frac", "share_of_kernel_time")}
    if r.get("cpu_baseline"):
        s["cpu_images_per_s"] = r["cpu_baseline"].get("value")
    return s


def pct(v):
    v = sorted(v)
    return [v[int(0.1 * (len(v) - 1))], v[int(0.9 * (len(v) - 1))]]


def timed_rounds(sess, mode, steps, warmup):
    import torch
    sess.run(mode, max(1, warmup))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    per_round = sess.run(mode, steps)
    torch.cuda.synchronize()
    wall_ms = (time.perf_counter() - t0) * 1e3 / steps
    return wall_ms, per_round


def model_makespan(sess, B, rows, splits, P):
    """Completion time and residue the regulation model (Eq. 1, Eq. 8) predicts for a plan, from the lookup table."""
    import ctypes as C
    from paper_2304_11745_amd import harness
    keep, sp_rows = [], []
    for row in splits:
        t, o, a, f = row[:4]
        if isinstance(f, (list, tuple)):
            arr = (C.c_int * len(f))(*f)
            keep.append(arr)
            sp_rows.append(B.gacer_split(t, o, harness.AXIS[a], len(f), arr))
        else:
            sp_rows.append(B.gacer_split(t, o, harness.AXIS[a], f, None))
    sp = (B.gacer_split * max(1, len(sp_rows)))(*sp_rows)
    n_ptr = len(P[0]) if P else 0
    flat = (C.c_int * max(1, len(sess.tenants) * n_ptr))(*[p for row in P for p in row])
    R, mk = C.c_double(), C.c_double()
    st = B.gacer_model_residue(sess.ctx, rows, len(rows), sp, len(sp_rows), flat, n_ptr, C.byref(R), C.byref(mk))
    if st != B.GACER_OK:
        return None
    return {"makespan_ms": round(mk.value, 4), "residue": round(R.value, 4)}


def calibrated_table(sess, B, rows, measured_unsplit_ms):
    """The lookup table with every W scaled by one factor, chosen so that the model's completion time of the unsplit plan
    equals the measured one.  W from launch geometry says how full a launch makes the chip by its own limiter; how much
    two launches really slow each other is a property of the chip that one measured round can supply."""
    import ctypes as C
    n = len(rows)
    none_P = [[] for _ in sess.tenants]

    def scaled(gamma):
        out = (B.gacer_prof * n)()
        C.memmove(out, rows, C.sizeof(B.gacer_prof) * n)
        for r in out:
            if r.tenant >= 0:
                r.cu_share = min(1.0, max(r.cu_share * gamma, 1.0 / 2048))
        return out

    def makespan(gamma):
        m = model_makespan(sess, B, scaled(gamma), [], none_P)
        return m["makespan_ms"] if m else None

    lo, hi = 1.0 / 64, 64.0
    m_lo, m_hi = makespan(lo), makespan(hi)
    if m_lo is None or m_hi is None:
        return None, None
    if measured_unsplit_ms <= m_lo:
        gamma = lo
    elif measured_unsplit_ms >= m_hi:
        gamma = hi
    else:
        for _ in range(40):                     # bisection in log space; the model's makespan grows with gamma
            mid = (lo * hi) ** 0.5
            if makespan(mid) < measured_unsplit_ms:
                lo = mid
            else:
                hi = mid
        gamma = (lo * hi) ** 0.5
    return scaled(gamma), gamma


def choose_plan(sess, B, trial_rounds):
    """Candidates: the searched plan (Algorithm 1 + spatial regulation on the profiled table), its decompositions alone and its
    pointers alone, plain stream-parallel, and uniform sweeps; each is measured for a few rounds next to what the model predicts for it; the fastest is refined
    (gacer_refine) and installed.  Because the unsplit plan is a candidate, the regulated run is never slower than
    stream-parallel by more than measurement noise."""
    t0 = time.perf_counter()
    rows = sess.profile()
    t_prof = time.perf_counter() - t0
    t0 = time.perf_counter()
    splits, syncs, P, R = sess.search(rows, 100)
    t_search = time.perf_counter() - t0
    none_P = [[] for _ in sess.tenants]
    cands = {"searched": (splits, syncs, P), "unsplit": ([], [], none_P)}
    # the two halves of the searched plan on their own (the Spatial / Temporal / GACER decomposition of Section 5.2, Fig. 7)
    if splits and syncs:
        cands["searched-spatial-only"] = (splits, [], none_P)
        cands["searched-temporal-only"] = ([], syncs, P)
    for axis in ("batch", "cout"):
        for f in (2, 4):
            sp = sess.uniform_splits(axis, f)
            if sp:
                cands[f"sweep-{axis}x{f}"] = (sp, [], none_P)
    results, model = {}, {}
    for name, (sp, sy, Pm) in cands.items():
        sess.set_plan(sp, sy)
        sess.run(B.GACER_MODE_PLAN, 3)
        ms = sess.run(B.GACER_MODE_PLAN, trial_rounds)
        results[name] = statistics.median(ms)
        model[name] = model_makespan(sess, B, rows, sp, Pm)
    # the search again, on the table calibrated against the measured unsplit round
    cal_rows, gamma = calibrated_table(sess, B, rows, results["unsplit"])
    cal_info = None
    if cal_rows is not None:
        c_splits, c_syncs, c_P, c_R = sess.search(cal_rows, 100)
        cands["searched-calibrated"] = (c_splits, c_syncs, c_P)
        sess.set_plan(c_splits, c_syncs)
        sess.run(B.GACER_MODE_PLAN, 3)
        results["searched-calibrated"] = statistics.median(sess.run(B.GACER_MODE_PLAN, trial_rounds))
        model["searched-calibrated"] = model_makespan(sess, B, cal_rows, c_splits, c_P)
        cal_info = {"w_scale": round(gamma, 4), "pointers": c_P, "splits": len(c_splits), "model_residue": c_R,
                    "model_unsplit": model_makespan(sess, B, cal_rows, [], none_P)}
    best = min(results, key=results.get)
    sp, sy, _ = cands[best]
    t0 = time.perf_counter()
    sess.set_plan(sp, sy)
    sp2, sy2, ms2 = sess.refine_plan(rows, rounds=trial_rounds)
    t_refine = time.perf_counter() - t0
    results["refined"] = ms2
    chosen = best
    if ms2 < results[best] and len(sp2) > len(sp):
        chosen, sp, sy = f"{best}+refined({len(sp2) - len(sp)} ops decomposed)", sp2, sy2
    kind = "regulated (decomposition and/or pointers)" if (sp or sy) else "stream-parallel (the plan holds no decomposition and no pointers)"
    info = {"profile_s": round(t_prof, 3), "search_s": round(t_search, 4), "refine_s": round(t_refine, 3), "searched_pointers": P,
            "searched_splits": len(splits), "model_residue": R,
            "trial_ms": {k: round(v, 4) for k, v in results.items()},
            "model_vs_measured": {k: {"model": model[k], "measured_ms": round(results[k], 4)} for k in cands},
            "calibrated_search": cal_info, "chosen": chosen, "chosen_kind": kind}
    sess.set_plan(sp, sy)
    return info


def cpu_baseline(tenants, data, budget_s=25.0, floor_s=10.0):
    """The oracle as it stands, timed on the host cores: whole rounds of the workload (tenants in order) until about
    `floor_s` seconds of work are done; a round that alone exceeds `budget_s` is cut after the tenant that crosses it."""
    from oracle import forward as F
    F.lib()
    items, t_total, rounds, partial = 0, 0.0, 0, None
    while t_total < floor_s and rounds < 64:
        done = []
        for t, (x, p) in zip(tenants, data):
            t0 = time.perf_counter()
            F.run_tenant(t, x, p)
            t_total += time.perf_counter() - t0
            done.append(t)
            items += t.batch
            if t_total > budget_s:
                break
        if len(done) < len(tenants):
            partial = done
            break
        rounds += 1
    cores = int(os.environ.get("OMP_NUM_THREADS", 0)) or len(os.sched_getaffinity(0))
    if partial is not None and rounds == 0:
        what = "the first %d of %d tenants of a round (%s)" % (len(partial), len(tenants), "+".join(f"{t.name}({t.batch})" for t in partial))
    elif partial is not None:
        what = "%d full rounds of the workload and part of another" % rounds
    else:
        what = "%d full round%s of the workload" % (rounds, "" if rounds == 1 else "s")
    return {"value": items / t_total, "unit": "images/s", "cores": cores, "kind": "oracle",
            "sample": f"{what}: {items} items, {t_total:.2f} s wall"}


def dominant_roofline(trace, dtype, config):
    per_kernel = {}
    for r in trace:
        k = per_kernel.setdefault(r["kernel"], {"ms": 0.0, "flops": 0.0, "bytes": 0.0, "launches": 0})
        k["ms"] += r["ms"]; k["flops"] += r["flops"]; k["bytes"] += r["bytes"]; k["launches"] += 1
    dom = max(per_kernel, key=lambda n: per_kernel[n]["ms"])
    d = per_kernel[dom]
    avg_ms = d["ms"] / d["launches"]
    traffic, profiled = measured_traffic(config, dom, d["launches"])
    # which roof bounds the kernel: the one its algorithmic work would take longer under (a contraction whose arithmetic
    # intensity lies below the ridge of its dtype is a bandwidth-bound kernel, e.g. bf16 pointwise products with short K)
    if d["flops"] / PEAK[dtype] >= d["bytes"] / HBM_PEAK and d["flops"] > 0:
        achieved = d["flops"] / d["launches"] / (avg_ms * 1e-3) / 1e12
        roof = {"bound": "mfma", "achieved": achieved, "peak": PEAK[dtype] / 1e12, "unit": "TFLOP/s",
                "frac": achieved / (PEAK[dtype] / 1e12), "traffic": traffic}
    else:
        achieved = d["bytes"] / d["launches"] / (avg_ms * 1e-3) / 1e9
        roof = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK / 1e9, "unit": "GB/s",
                "frac": achieved / (HBM_PEAK / 1e9), "traffic": traffic}
    if profiled:
        roof["traffic_profiled"] = profiled
    roof["algorithmic_bytes_per_launch"] = d["bytes"] / d["launches"]
    roof.update({"kernel": dom, "launches_per_round": d["launches"], "avg_launch_us": avg_ms * 1e3,
                 "share_of_kernel_time": d["ms"] / sum(k["ms"] for k in per_kernel.values()),
                 "duration_basis": "kernel begin/end stamped by the runtime on the launch (what a profiler's kernel trace reports), "
                                   "mean over the launches of 5 regulated rounds"})
    kernels = {k: {"launches": v["launches"], "ms_per_round": round(v["ms"], 4),
                   "TFLOP/s": round(v["flops"] / (v["ms"] * 1e-3) / 1e12, 2) if v["ms"] > 0 else None,
                   "GB/s": round(v["bytes"] / (v["ms"] * 1e-3) / 1e9, 1) if v["ms"] > 0 else None}
               for k, v in sorted(per_kernel.items(), key=lambda kv: -kv[1]["ms"])}
    return roof, kernels


def run_config(config, args, cpu_budget_s):
    """One workload: plan selection, three timed modes, per-kernel trace, CPU baseline."""
    import synth
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    tenants, data = synth.build_config(config, args.scale)
    items = sum(t.batch for t in tenants)
    dtype = tenants[0].dtype
    macs = sum(synth.gemm_macs(t) for t in tenants)
    sess = harness.Session(tenants, data, "cuda:0")
    sess.run(B.GACER_MODE_SEQUENTIAL, 3)

    plan_info = {"chosen": "unsplit", "chosen_kind": "stream-parallel (the plan holds no decomposition and no pointers)"}
    if args.plan == "auto":
        plan_info = choose_plan(sess, B, 10)
    # host side of the plan: one issuing thread for all tenants, or one per tenant (the deployment model of Section 2.1);
    # measured like every other candidate, before the timed region
    trial = {}
    for thr in (False, True):
        sess.set_issue_threads(thr)
        sess.run(B.GACER_MODE_PLAN, 5)
        t0 = time.perf_counter()
        sess.run(B.GACER_MODE_PLAN, 20)
        trial[thr] = (time.perf_counter() - t0) * 1e3 / 20
    use_threads = len(tenants) > 1 and trial[True] < 0.97 * trial[False]
    sess.set_issue_threads(use_threads)
    plan_info["issue_threads"] = use_threads
    plan_info["issue_trial_ms"] = {"one_thread": round(trial[False], 4), "thread_per_tenant": round(trial[True], 4)}
    log(f"config {config} plan selection:", json.dumps(plan_info))

    if args.only_regulated:
        seq_ms = par_ms = None
        seq_rounds = par_rounds = [float("nan")]
    else:
        seq_ms, seq_rounds = timed_rounds(sess, B.GACER_MODE_SEQUENTIAL, args.steps, args.warmup)
        par_ms, par_rounds = timed_rounds(sess, B.GACER_MODE_STREAM_PARALLEL, args.steps, args.warmup)
    reg_ms, reg_rounds = timed_rounds(sess, B.GACER_MODE_PLAN, args.steps, args.warmup)

    roof, kernels = dominant_roofline(sess.trace(B.GACER_MODE_PLAN, 5), dtype, config)
    out = {
        "workload": (f"configs[{config - 1}]: " if config <= 5 else "tenant mix of the evaluation (Table 2): ") + synth.CONFIG_NAMES[config] +
                    (" (small)" if args.scale == "small" else ""),
        "items_per_round": items, "tenants": [f"{t.name}({t.batch})" for t in tenants], "dtype": dtype,
        "plan": plan_info.get("chosen"), "plan_kind": plan_info.get("chosen_kind"), "issue_threads": plan_info.get("issue_threads"),
        "launches_per_round": sess.launch_count(B.GACER_MODE_PLAN),
        "ms_per_step": reg_ms,
        "regulated_images_per_s": items / (reg_ms * 1e-3),
        "sequential_images_per_s": items / (seq_ms * 1e-3) if seq_ms else None,
        "stream_parallel_images_per_s": items / (par_ms * 1e-3) if par_ms else None,
        "speedup_vs_sequential": seq_ms / reg_ms if seq_ms else None,
        "speedup_vs_stream_parallel": par_ms / reg_ms if par_ms else None,
        "makespan_ms_median": {"sequential": statistics.median(seq_rounds), "stream_parallel": statistics.median(par_rounds),
                               "regulated": statistics.median(reg_rounds)},
        "makespan_ms_p10_p90": {"sequential": pct(seq_rounds), "stream_parallel": pct(par_rounds), "regulated": pct(reg_rounds)},
        "mfma_frac_of_peak": {"sequential": 2 * macs / (seq_ms * 1e-3) / PEAK[dtype] if seq_ms else None,
                              "stream_parallel": 2 * macs / (par_ms * 1e-3) / PEAK[dtype] if par_ms else None,
                              "regulated": 2 * macs / (reg_ms * 1e-3) / PEAK[dtype]},
        "plan_selection": plan_info,
        "kernels": kernels,
        "roofline": roof,
    }
    sess.close()
    if not args.no_cpu_baseline and cpu_budget_s > 0:
        out["cpu_baseline"] = cpu_baseline(tenants, data, cpu_budget_s, floor_s=min(10.0, 0.4 * cpu_budget_s))
    return out


def granularity_table(dtype, rounds):
    """The spatial-granularity experiment of Section 5.4 (its Table 3) on this executor: VGG-16(32) and ResNet-18(32)
    share the GPU; the rows differ in how one model's batch is decomposed, every operator of that model into the same
    chunk list, with the chunks alternating between the model's stream and its sibling stream (gacer_split.sibling), so
    that V16(16)+V16(16) really is two half batches side by side.  Synthetic inputs, seeded weights.  Prints one JSON line."""
    from synth import graphs as G
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    tenants = [G.vgg16(dtype, 32), G.resnet18(dtype, 32)]
    data = [G.materialise(t, 20230411, i << 20) for i, t in enumerate(tenants)]
    sess = harness.Session(tenants, data, "cuda:0")
    rows = {"1: V16(32) R18(32)": [],
            "2: V16(16)+V16(16) R18(32)": [(0, [16, 16])],
            "3: V16(24)+V16(8) R18(32)": [(0, [24, 8])],
            "4: V16(32) R18(16)+R18(16)": [(1, [16, 16])],
            "5: V16(8)x4 R18(32)": [(0, [8, 8, 8, 8])]}
    out = {}
    sess.run(B.GACER_MODE_SEQUENTIAL, 2)
    for name, spec in rows.items():
        for siblings in (True, False):
            splits = [(ti, oi, "batch", sizes, siblings) for (ti, sizes) in spec for oi in range(len(tenants[ti].ops))]
            sess.set_plan(splits, [])
            sess.run(B.GACER_MODE_PLAN, 5)
            ms = statistics.median(sess.run(B.GACER_MODE_PLAN, rounds))
            out.setdefault(name, {})["sibling_streams_ms" if siblings else "one_stream_per_model_ms"] = round(ms, 4)
        log(f"granularity {name}: {out[name]}")
    sess.close()
    base = out["1: V16(32) R18(32)"]["sibling_streams_ms"]
    for v in out.values():
        v["vs_row1"] = round(base / v["sibling_streams_ms"], 3)
    print(json.dumps({"experiment": "spatial granularity (Section 5.4, Table 3)", "dtype": dtype, "unit": "ms per round of 64 images",
                      "rows": out, "paper_context": "Titan V: 80 / 66 / 72 / 78 / 85 ms for rows 1-5; other hardware, context only"}), flush=True)


def pointer_sweep(config, rounds):
    """The temporal-granularity experiment of Section 5.4 (its Fig. 9) on this executor: the same workload with 0, 1, 2, ...
    synchronisation pointers per model, evenly spaced over each model's operator list (model-wise, then segment-wise, up
    to one pointer after every operator of the shortest model), no decomposition.  Also times the search at growing round
    limits (the paper's Table 4).  Synthetic inputs, seeded weights.  Prints one JSON line."""
    import synth
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    tenants, data = synth.build_config(config)
    sess = harness.Session(tenants, data, "cuda:0")
    n_ops = [len(t.ops) for t in tenants]
    table = sess.profile()
    t_sw = [r.ms for r in table if r.tenant < 0][0]
    sess.set_plan([], [])
    sess.run(B.GACER_MODE_PLAN, 5)
    seq = statistics.median(sess.run(B.GACER_MODE_SEQUENTIAL, rounds))
    out = {}
    counts = [0, 1, 2, 3, 5, 8, 12, 16, 24, min(n_ops) - 1]
    for k in sorted(set(c for c in counts if 0 <= c < min(n_ops))):
        P = [[round((j + 1) * n / (k + 1)) for j in range(k)] for n in n_ops]
        syncs = sess.edges_from_pointers(P) if k else []
        sess.set_plan([], syncs)
        sess.run(B.GACER_MODE_PLAN, 5)
        ms = statistics.median(sess.run(B.GACER_MODE_PLAN, rounds))
        out[str(k)] = {"ms": round(ms, 4), "event_edges": len(syncs), "model": model_makespan(sess, B, table, [], P)}
        log(f"pointer sweep config {config}: {k} pointers per model -> {ms:.4f} ms")
    search = {}
    for limit in (1, 10, 100, 1000, 10000):
        t0 = time.perf_counter()
        _, _, P, R = sess.search(table, limit)
        search[str(limit)] = {"seconds": round(time.perf_counter() - t0, 4), "pointers_per_model": len(P[0]) if P else 0, "residue": round(R, 4)}
    sess.close()
    print(json.dumps({"experiment": "temporal granularity (Section 5.4, Fig. 9) and search time (Table 4)", "config": config,
                      "tenants": [f"{t.name}({t.batch})" for t in tenants], "operators_per_model": n_ops, "unit": "ms per round",
                      "sequential_ms": round(seq, 4), "T_SW_ms": round(t_sw, 5), "pointers_per_model": out, "search_time_by_round_limit": search,
                      "paper_context": "Fig. 9: latency falls from model-wise to a middle granularity and rises again towards operator-wise; "
                                       "Table 4: 0.9 s at 100 rounds to 2 min 52 s at 10000 (Python, other hardware)"}), flush=True)


def line(head, steps, warmup, per_config, mixes):
    """The one JSON line: the headline workload's record, summaries of the others."""
    out = {
        "metric": "aggregate tenant images/s (regulated concurrent run)",
        "value": head["regulated_images_per_s"],
        "unit": "images/s",
        "n_gpus": 1, "steps": steps, "warmup": warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": head["dtype"], "data": "synthetic",
        "config": {"workload": head["workload"], "items_per_round": head["items_per_round"], "tenants": head["tenants"],
                   "plan": head["plan"], "plan_kind": head["plan_kind"], "issue_threads": head["issue_threads"],
                   "launches_per_round": head["launches_per_round"]},
    }
    for k in ("sequential_images_per_s", "stream_parallel_images_per_s", "speedup_vs_sequential", "speedup_vs_stream_parallel",
              "makespan_ms_median", "makespan_ms_p10_p90", "mfma_frac_of_peak", "kernels", "roofline"):
        out[k] = head[k]
    out["plan_selection"] = {k: v for k, v in head["plan_selection"].items()
                             if k in ("profile_s", "search_s", "refine_s", "searched_pointers", "searched_splits", "trial_ms", "issue_trial_ms")}
    if "cpu_baseline" in head:
        out["cpu_baseline"] = head["cpu_baseline"]
    out["paper_context"] = "GACER reports 1.37x-1.66x over sequential cuDNN on Titan V (Section 5.2); other hardware, context only"
    if per_config:
        out["per_config"] = {str(c): summary(r) for c, r in per_config.items()}
    if mixes:
        out["paper_mixes"] = {str(c): summary(r) for c, r in mixes.items()}
    return json.dumps(rounded(out))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--config", type=int, default=2, help="headline workload: 1..5 = the configurations, 6.. = tenant mixes of the paper's evaluation (default 2)")
    ap.add_argument("--also", default="3,4,5", help="further workloads reported under per_config (comma separated; '' for none)")
    ap.add_argument("--mixes", default=None, help="tenant mixes of the paper's evaluation reported under paper_mixes, without a CPU "
                                                  "baseline (comma separated; '' for none; default: 6,7,8 in the plain default run only)")
    ap.add_argument("--scale", default="full", choices=["full", "small"])
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--plan", default="auto", help="auto | unsplit")
    ap.add_argument("--only-regulated", action="store_true",
                    help="time the regulated mode only (profiling runs: every dispatch then belongs to the reported mode)")
    ap.add_argument("--print-sources-digest", action="store_true")
    ap.add_argument("--granularity-table", choices=["f32", "bf16"], default=None,
                    help="run the batch-decomposition-over-streams experiment (Section 5.4) instead of the benchmark")
    ap.add_argument("--pointer-sweep", type=int, default=None, metavar="CONFIG",
                    help="run the pointer-count sweep (Section 5.4, Fig. 9) on the given workload instead of the benchmark")
    ap.add_argument("--copy-probe", action="store_true",
                    help="also run a plain copy of known size (256 MiB in, 256 MiB out) three times, as the "
                         "reference dispatch for scaling hardware traffic counters")
    args = ap.parse_args()
    if args.print_sources_digest:
        print(sources_digest())
        return
    if args.granularity_table:
        granularity_table(args.granularity_table, max(10, args.steps // 4))
        return
    if args.pointer_sweep:
        pointer_sweep(args.pointer_sweep, max(10, args.steps // 2))
        return
    if args.gpus != 1:
        sys.exit("bench.py: the executor runs on exactly one GPU (tenants shard across GPUs with no exchange); use --gpus 1")

    import torch  # noqa: F401
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness

    if args.copy_probe:
        from synth import graphs as G
        b = G._B("copy_probe", "f32", 64)
        x = b.tensor(64, 256, 64, 64)                      # 64 Mi floats = 256 MiB
        t = b.done(x, b.act(x, "none"))
        probe = harness.Session([t], [G.materialise(t, 1)], "cuda:0")
        probe.run(B.GACER_MODE_SEQUENTIAL, 3)
        probe.close()
        log("copy probe: eltwise kernel, 3 dispatches, 268435456 bytes read + 268435456 bytes written each")

    head = run_config(args.config, args, 25.0)
    log(f"config {args.config}:", json.dumps(head))
    also = [int(c) for c in args.also.split(",") if c.strip() and int(c) != args.config]
    per_config, mix_records = {}, {}
    for c in also:
        per_config[c] = run_config(c, args, 12.0)
        log(f"config {c}:", json.dumps(per_config[c]))
    if args.mixes is None:                                 # any narrowing flag means: exactly what was asked for
        args.mixes = "6,7,8" if (args.config == 2 and args.also == "3,4,5" and not args.only_regulated and args.scale == "full") else ""
    mixes = [int(c) for c in args.mixes.split(",") if c.strip() and int(c) != args.config and int(c) not in also]
    for c in mixes:
        mix_records[c] = run_config(c, args, 0.0)
        log(f"mix {c}:", json.dumps(mix_records[c]))
    print(line(head, args.steps, args.warmup, per_config, mix_records), flush=True)


if __name__ == "__main__":
    main()
