"""Throughput benchmark of the ProbeWalk hot path on one MI355X.

Workload: Chung-Lu graph n=100,000, mean degree 10, exponent 2.5, largest
connected component (99,163 nodes, 997,038 adjacency entries); uniform (s,t)
pairs; eps = 0.05, L = 1000; walk counts from the scaled policy of Algorithm 1
(constants in paper_2512_05460_amd/budgets.py); tables in the compact
hubs-first layout with the probe on storage ids. One step = one batch of
queries run in the plain mode (one query per launch, fixed tiling). The same
batch is also run in the batched (persistent, work-stealing) mode, through
the server (continuous batching) and with walk sharing, reported beside the
headline; so are the small-query, grid (mixed eps and L, hipGraph), served
Chung-Lu n=10^7 (Poisson arrivals; plain, batched and served at calibrated
walk counts) and Chung-Lu n=4*10^7 (calibrated reference pairs and a
throughput-setting launch) workloads; --scale adds the full n=4*10^7 report
over three layouts.

Prints one JSON line. The graph is resident on the device before the timed
region; each query's 48-byte descriptor travels host->device inside the call
and its result device->host.
"""

from __future__ import annotations

import argparse
import hashlib
import re
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

WORKLOAD = "cl100k"
EPS = 0.05
L = 1000
BYTES_PER_STEP = 12   # algorithmic: next node id + its row offset and degree (4 + 4 + 4 bytes)
HBM_PEAK_GBS = 8000.0
L2_PEAK_REQ_PER_S = 8 * 16 * 2.4e9   # one request per L2 channel per clock, 16 channels per XCD
COUNTERS = os.path.join(ROOT, "profiles", "walk_kernel_cl100k_counters.txt")
FAT_SCALE_COUNTERS = os.path.join(ROOT, "profiles", "walk_kernel_fat_cl40m_counters.txt")
KERNEL_SOURCES = ["pw_kernels.hip", "pw_signs.hip", "pw_chunk.hpp", "pw_device.hpp", "pw_internal.hpp", "pw_runs.hpp"]
LAYOUT_NAMES = {0: "csr", 1: "fat", 2: "compact", 3: "compact, hubs first", 4: "hubs first, 4-byte ids",
                5: "hubs first, probe on storage ids"}


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def kernel_source_hash() -> str:
    """sha256[:16] of the device sources with comments and blank lines removed:
    it changes when the compiled kernels can, not when a comment does."""
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2512_05460_amd", "csrc", f), encoding="utf-8") as fh:
            src = re.sub(r"/\*.*?\*/", "", fh.read(), flags=re.S)
        lines = (re.sub(r"//.*", "", ln).rstrip() for ln in src.splitlines())
        h.update("\n".join(ln for ln in lines if ln).encode())
    return h.hexdigest()[:16]


def read_counters(path):
    """key = value lines of a committed rocprofv3 summary, or (None, why) when
    it is missing or the kernel sources changed since the counters were taken."""
    if not os.path.exists(path):
        return None, "no counter summary"
    kv = {}
    for ln in open(path):
        if "=" in ln and not ln.startswith("#"):
            k, v = ln.split("=", 1)
            kv[k.strip()] = v.split("(")[0].strip()
    if kv.get("kernel_source_sha256_16") != kernel_source_hash():
        return None, "kernel changed since the counters were taken"
    return kv, ""


def counter_traffic():
    """HBM bytes per walk step of the headline kernel from the committed
    rocprofv3 summary, or None when the kernel sources changed since."""
    kv, why = read_counters(COUNTERS)
    if kv is None:
        return None, why
    try:
        fetch = float(kv["fetch_kib_per_dispatch"]) * float(kv["fetch_scale"])
        write = float(kv["write_kib_per_dispatch"]) * float(kv["write_scale"])
        steps = float(kv["walk_steps_per_dispatch"])
    except (KeyError, ValueError):
        return None, "incomplete counter summary"
    return (fetch + write) * 1024.0 / steps, "bytes per walk step, FETCH_SIZE and WRITE_SIZE scaled by a copy kernel"


def l2_requests(kernel_sps):
    """The resource that binds the L2-resident headline kernel: L2 requests per
    walk step from the committed counters, at the walk-step rate measured here."""
    kv, why = read_counters(COUNTERS)
    if kv is None:
        return {"note": why}
    try:
        rps = float(kv["l2_requests_per_step"])
        hit = float(kv["l2_hit_rate"])
    except (KeyError, ValueError):
        return {"note": "incomplete counter summary"}
    achieved = rps * kernel_sps
    return {"requests_per_step": rps, "hit_rate": hit, "requests_per_s": achieved,
            "peak_requests_per_s": L2_PEAK_REQ_PER_S, "frac": achieved / L2_PEAK_REQ_PER_S,
            "note": ("random L2 requests per walk step (TCC_REQ); the tables are L2-resident; peak = one "
                     "request per L2 channel per clock: 8 XCDs x 16 channels x 2.4 GHz")}


def host_cpus():
    """The host's CPUs as this process sees them: the model name and socket
    layout (lscpu, else /proc/cpuinfo), the logical CPUs of the machine and of
    this process's affinity mask, and how many threads the oracle may use --
    all of the affinity mask, capped by OMP_NUM_THREADS when the machine sets
    one (the CPU share a job on a shared GPU machine is given)."""
    info = {"model": "", "logical_cpus": os.cpu_count() or 1}
    try:
        info["affinity_cpus"] = len(os.sched_getaffinity(0))
    except AttributeError:
        info["affinity_cpus"] = info["logical_cpus"]
    try:
        import subprocess
        out = subprocess.run(["lscpu"], capture_output=True, text=True, timeout=10).stdout
        kv = {ln.split(":", 1)[0].strip(): ln.split(":", 1)[1].strip() for ln in out.splitlines() if ":" in ln}
        info["model"] = kv.get("Model name", "")
        for k in ("Socket(s)", "Core(s) per socket", "Thread(s) per core", "CPU max MHz"):
            if k in kv:
                info[k] = kv[k]
    except (OSError, ValueError, IndexError):
        pass
    if not info["model"]:
        try:
            with open("/proc/cpuinfo") as fh:
                info["model"] = next((ln.split(":", 1)[1].strip() for ln in fh if ln.startswith("model name")), "")
        except OSError:
            pass
    usable = info["affinity_cpus"]
    share = os.environ.get("OMP_NUM_THREADS", "")
    if share.isdigit() and int(share) > 0:
        usable = min(usable, int(share))
        info["cpu_share"] = f"OMP_NUM_THREADS={share}"
    info["usable"] = usable
    return info


def cpu_baseline(g, s, t, plans, seed, target_s=20.0):
    """The oracle on a bounded sample: each of `threads` queries runs its first
    few probes at the full R and L; queries/s is the measured step rate divided
    by the mean full-query step count."""
    from oracle import estimator as E

    host = host_cpus()
    threads = max(1, min(host["usable"], len(plans)))
    sub = [plans[i] for i in range(threads)]
    per_probe = np.array([2.0 * p[3] * L for p in sub])
    kend = np.maximum(1, np.minimum([p[2] for p in sub], (1.5e7 * target_s / per_probe).astype(np.int64)))
    t0 = time.perf_counter()
    E.estimate(g, s[:threads], t[:threads], L, sub, seed, uid=np.arange(threads), threads=threads, k_end=kend)
    dt = time.perf_counter() - t0
    steps = float((kend * per_probe).sum())
    full = np.array([2.0 * p[2] * p[3] * L for p in plans])
    sps = steps / dt
    return {"value": sps / full.mean(), "unit": "queries/s", "cores": threads, "kind": "oracle",
            "cpu_model": host["model"], "host": host,
            "walk_steps_per_s": sps, "walk_steps_per_s_per_core": sps / threads,
            "single_thread_seconds_per_query": full.mean() / (sps / threads),
            "sample": (f"{threads} of the step's queries, first {int(kend.min())}-{int(kend.max())} of their "
                       f"probes each at full R and L, one query per thread; {steps:.3e} walk steps in "
                       f"{dt:.1f} s; queries/s = steps/s / mean full-query steps of the batch")}


def small_queries(B, torch, stream, layout="compact"):
    """The regime where one query cannot fill the GPU: BA n=1,000, 256 uniform
    pairs, eps=0.1, L=200 (a few 10^8 walk steps per query), plain vs batched
    vs batched replayed from a captured hipGraph; tables compact, or
    layout="hubsid" hubs first with the probe on storage ids."""
    from paper_2512_05460_amd.budgets import budget_policy
    from synth import graphs, queries

    g = graphs.workload_graph("ba1k")
    s, t = queries.uniform_pairs(g.n, 256, graphs.GRAPH_SEED + 0 + graphs.QUERY_SEED_OFFSET)
    flags = {"compact": B.BD_LAYOUT_COMPACT,
             "hubsid": B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS}[layout]
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
    pol = budget_policy("ba1k")
    seed = graphs.PHILOX_SEED
    out = {"workload": "Barabasi-Albert n=1,000 m=3; 256 uniform pairs; eps=0.1, L=200",
           "layout": LAYOUT_NAMES[dg.info()["layout"]], "lds_nodes": dg.info()["lds_hubs"]}

    def timed(fn, reps=3):
        fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / reps

    plain = B.exec_cfg("plain")
    dt_plain = timed(lambda: [B.bd_query_batch(dg, s[i:i + 1], t[i:i + 1], 0.1, 200, seed, pol, plain,
                                               uid=[i], stream=stream) for i in range(256)], reps=1)
    dt_batched = timed(lambda: B.bd_query_batch(dg, s, t, 0.1, 200, seed, pol, B.exec_cfg("batched"),
                                                stream=stream))
    dt_graph = timed(lambda: B.bd_query_batch(dg, s, t, 0.1, 200, seed, pol,
                                              B.exec_cfg("batched", use_graph=True), stream=stream))
    steps = float(B.bd_plan(dg, s, t, 0.1, 200, pol)["walk_steps"].sum())
    out.update({"walk_steps": steps, "plain_qps": 256 / dt_plain, "batched_qps": 256 / dt_batched,
                "graph_qps": 256 / dt_graph, "batched_vs_plain": dt_plain / dt_batched,
                "graph_vs_plain": dt_plain / dt_graph})
    dg.free()
    return out


def grid_batched(B, torch, stream, plain_sample=512, layout="hubsid", profile_chunk_pairs=0):
    """Mixed eps and L in one persistent launch: the 1,414 x 1,414 grid (5% of
    edges removed), 65,536 queries, eps over {0.02, 0.05, 0.1}, L over {500,
    2000, 5000}, throughput walk counts; tables hubs first with the probe on
    storage ids (every node's entry from the degree-run table in LDS), or with
    layout="auto" the library's choice (fat at this size); chunking from the
    autotuner, the launches captured into a hipGraph and run from it. The
    plain mode (one query per launch) runs the first `plain_sample` queries
    of the same set on the same tables. With profile_chunk_pairs > 0 only one
    eager batched launch of the whole set runs, with that chunking and eight
    queues (for a profiler's counters on exactly that launch)."""
    from paper_2512_05460_amd.budgets import BUDGETS, budget_policy
    from synth import graphs, queries

    g = graphs.workload_graph("grid1414")
    s, t, eps, Ls = queries.workload_batch("grid1414", g.n)
    nq = s.size
    flags = {"auto": B.BD_LAYOUT_AUTO,
             "hubsid": B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS}[layout]
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
    info = dg.info()
    pol = budget_policy("grid1414")
    seed = graphs.PHILOX_SEED
    plan = B.bd_plan(dg, s, t, eps, Ls, pol)
    steps = float(plan["walk_steps"].sum())
    if profile_chunk_pairs > 0:
        ex = B.exec_cfg("batched", chunk_pairs=profile_chunk_pairs, queues=8)
        log(f"grid: one batched launch of {nq} queries, {steps:.3e} walk steps, chunk_pairs={profile_chunk_pairs}")
        r, st = B.bd_query_batch(dg, s, t, eps, Ls, seed, pol, ex, stream=stream, with_stats=True)
        torch.cuda.synchronize()
        assert np.all(r["status"] == 0)
        dg.free()
        return {"profile_launch": {"chunk_pairs": profile_chunk_pairs, "queues": 8, "walk_steps": steps,
                                   "walk_kernel_launches": int(st["launches"]), "kernel_ms": st["walk_kernel_ms"],
                                   "kernel_walk_steps_per_s": steps / (st["walk_kernel_ms"] / 1e3)},
                "lds_nodes": info["lds_hubs"]}
    na = min(nq, 2048)
    log(f"grid: {nq} queries, {steps:.3e} walk steps; autotune on the first {na}")
    best, times = B.bd_autotune(dg, s[:na], t[:na], eps[:na], Ls[:na], seed, pol, stream=stream)
    ex = B.exec_cfg("batched", chunk_pairs=best.chunk_pairs, use_graph=True, queues=best.queues)
    log(f"grid: chunk_pairs={best.chunk_pairs} queues={best.queues}; capture and launch the whole set")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r, st = B.bd_query_batch(dg, s, t, eps, Ls, seed, pol, ex, stream=stream, with_stats=True)
    torch.cuda.synchronize()
    dt_graph = time.perf_counter() - t0
    assert np.all(r["status"] == 0)
    roof = max((B.bd_gather_roofline(dg, c, 2000) for c in (2, 4, 8)), key=lambda x: x["steps_per_s"])
    m = plain_sample
    plain = B.exec_cfg("plain")
    log(f"grid: plain mode on the first {m} queries")
    t0 = time.perf_counter()
    for i in range(m):
        B.bd_query_batch(dg, s[i:i + 1], t[i:i + 1], eps[i:i + 1], Ls[i:i + 1], seed, pol, plain,
                         uid=[i], stream=stream)
    torch.cuda.synchronize()
    dt_plain = time.perf_counter() - t0
    steps_m = float(plan["walk_steps"][:m].sum())
    t0 = time.perf_counter()
    B.bd_query_batch(dg, s[:m], t[:m], eps[:m], Ls[:m], seed, pol, B.exec_cfg("batched", chunk_pairs=best.chunk_pairs),
                     stream=stream)
    torch.cuda.synchronize()
    dt_batched_m = time.perf_counter() - t0
    dg.free()
    c_B, c_R, how = BUDGETS["grid1414"]
    return {
        "workload": ("1,414 x 1,414 grid, 5% of edges removed, connected (bipartite); 65,536 uniform pairs, "
                     "eps over {0.02, 0.05, 0.1}, L over {500, 2000, 5000}"),
        "layout": LAYOUT_NAMES[info["layout"]], "lds_nodes": info["lds_hubs"], "device_bytes": info["device_bytes"],
        "policy": {"kind": "scaled", "c_B": c_B, "c_R": c_R, "calibration": how},
        "R_range": [int(plan["R"].min()), int(plan["R"].max())],
        "walk_steps": steps,
        "autotune": {"chunk_pairs": best.chunk_pairs, "queues": best.queues,
                     "sample_queries": na, "kernel_ms": [float(x) for x in times]},
        "graph_qps": nq / dt_graph,
        "graph_walk_steps_per_s": steps / dt_graph,
        "kernel_ms": st["walk_kernel_ms"],
        "kernel_walk_steps_per_s": steps / (st["walk_kernel_ms"] / 1e3),
        "random_start_gather_steps_per_s": roof["steps_per_s"],
        "vs_random_start_gather": steps / (st["walk_kernel_ms"] / 1e3) / roof["steps_per_s"],
        "random_start_gather_note": ("the same loads from random start nodes; the walks' locality (all replicas "
                                     "of a chunk start at the same two nodes) runs above it, so this ratio is "
                                     "not a roofline fraction"),
        "plain_sample": m,
        "plain_qps": m / dt_plain,
        "plain_walk_steps_per_s": steps_m / dt_plain,
        "batched_same_sample_qps": m / dt_batched_m,
        "graph_vs_plain_walk_steps_per_s": (steps / dt_graph) / (steps_m / dt_plain),
    }


def served_cl10m(B, torch, seconds_per_load=10.0, calibrated_queries=8, profile=False):
    """Continuous batching under Poisson arrivals: Chung-Lu n=10^7 (mean degree
    10, exponent 2.3, largest component, resident on the device in the layout
    the library picks: fat at this size); request batches of 2^U uniform pairs (U uniform
    on 0..12, 1 to 4,096 pairs), eps per query from {0.02, 0.05, 0.1}, L=1000,
    throughput walk counts. Capacity comes from a burst of requests submitted
    at once; then Poisson arrivals at 50%, 80% and 95% of it, each for
    `seconds_per_load` seconds of arrivals. Latency is per request, from
    submission to completion as the server records it. Last, one set at
    eps = 0.05, L = 1000 in the plain, batched and served modes."""
    from paper_2512_05460_amd.budgets import BUDGETS, budget_policy
    from synth import graphs, queries

    log("served: building Chung-Lu n=10^7")
    g = graphs.workload_graph("cl10m")
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_AUTO)
    pol = budget_policy("cl10m")
    seed = graphs.PHILOX_SEED
    base = graphs.GRAPH_SEED + 3 + graphs.QUERY_SEED_OFFSET + 0x10
    Lq = 1000
    mean_size = (2 ** 13 - 1) / 13.0
    srv = B.Server(dg, pol)
    warm = queries.served_requests(g.n, 2, base - 7, max_log2=4)
    for i, (s, t, e) in enumerate(warm):
        srv.wait(srv.submit(s, t, e, Lq, seed + 999 + i))
    burst = queries.served_requests(g.n, 24, base)
    nq_burst = sum(x[0].size for x in burst)
    log(f"served: capacity burst of {len(burst)} requests, {nq_burst} queries")
    t0 = time.perf_counter()
    rids = [srv.submit(s, t, e, Lq, seed + i) for i, (s, t, e) in enumerate(burst)]
    for rid in rids:
        out, _ = srv.wait(rid)
        assert np.all(out["status"] == 0)
    dt = time.perf_counter() - t0
    cap_qps = nq_burst / dt
    if profile:  # the capacity burst only (for a profiler's counters on its slices)
        steps = sum(float(B.bd_plan(dg, x[0], x[1], x[2], Lq, pol)["walk_steps"].sum()) for x in burst)
        srv.destroy()
        dg.free()
        return {"profile_burst": {"requests": len(burst), "queries": nq_burst, "seconds": dt,
                                  "queries_per_s": cap_qps, "walk_steps": steps, "walk_steps_per_s": steps / dt}}
    out = {"workload": ("Chung-Lu n=10,000,000 mean degree 10 exponent 2.3 LCC; Poisson arrivals of request "
                        "batches of 2^U uniform pairs, U uniform on 0..12; eps per query from {0.02, 0.05, 0.1}; "
                        "L=1000"),
           "graph": {"n": g.n, "nnz": g.nnz, "layout": LAYOUT_NAMES[dg.info()["layout"]],
                     "device_bytes": dg.info()["device_bytes"]},
           "policy": {"kind": "scaled", "c_B": BUDGETS["cl10m"][0], "c_R": BUDGETS["cl10m"][1],
                      "calibration": BUDGETS["cl10m"][2]},
           "admission": "slots 65,536 queries; per-probe accumulator arena; no walk-step cap",
           "capacity_queries_per_s": cap_qps, "capacity_burst": {"requests": len(burst), "queries": nq_burst,
                                                                 "seconds": dt},
           "loads": []}
    for li, f in enumerate((0.5, 0.8, 0.95)):
        count = max(8, int(round(f * cap_qps / mean_size * seconds_per_load)))
        reqs = queries.served_requests(g.n, count, base + 1000 * (li + 1))
        # the arrival rate is set from the drawn request sizes, so that the
        # offered queries/s is exactly f times the capacity whatever the draw
        rate = count * f * cap_qps / sum(x[0].size for x in reqs)
        arr = queries.poisson_arrivals(count, rate, base + 1000 * (li + 1) + 1)
        log(f"served: offered load {f:.0%} of capacity, {count} requests at {rate:.2f}/s")
        start = time.perf_counter()
        sub, rids = [], []
        for i, (s, t, e) in enumerate(reqs):
            d = start + arr[i] - time.perf_counter()
            if d > 0:
                time.sleep(d)
            sub.append(time.perf_counter() - start)
            rids.append(srv.submit(s, t, e, Lq, seed + 100000 * (li + 1) + i))
        lat = []
        for rid in rids:
            o, l_ms = srv.wait(rid)
            assert np.all(o["status"] == 0)
            lat.append(l_ms)
        lat = np.array(lat)
        end = max(sub[i] + lat[i] / 1e3 for i in range(count))
        nq = sum(x[0].size for x in reqs)
        sizes = np.array([x[0].size for x in reqs])
        out["loads"].append({"offered_fraction": f, "offered_queries_per_s": f * cap_qps,
                             "offered_requests_per_s": rate, "requests": count,
                             "queries": int(nq), "queries_per_s": nq / end,
                             "latency_ms": {"p50": float(np.percentile(lat, 50)),
                                            "p99": float(np.percentile(lat, 99)), "max": float(lat.max())},
                             "latency_ms_requests_le_64": float(np.percentile(lat[sizes <= 64], 50))
                             if np.any(sizes <= 64) else None})
    # The three modes on one set at eps = 0.05, L = 1000 (4,096 uniform pairs):
    # the served requests are 16 of 256 pairs submitted together; the plain
    # mode (one query per launch) runs the first 256 queries.
    log("served: plain / batched / served at eps=0.05, L=1000")
    s5, t5 = queries.uniform_pairs(g.n, 4096, base + 0x5005)
    r_b, _ = B.bd_query_batch(dg, s5, t5, 0.05, Lq, seed, pol, B.exec_cfg("batched"), with_stats=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r_b = B.bd_query_batch(dg, s5, t5, 0.05, Lq, seed, pol, B.exec_cfg("batched"))
    torch.cuda.synchronize()
    dt_b = time.perf_counter() - t0
    t0 = time.perf_counter()
    rids = [srv.submit(s5[j:j + 256], t5[j:j + 256], 0.05, Lq, seed, uid=np.arange(j, j + 256))
            for j in range(0, 4096, 256)]
    for k, rid in enumerate(rids):
        o, _ = srv.wait(rid)
        assert np.array_equal(o["beta"], r_b["beta"][256 * k:256 * k + 256])
    dt_s = time.perf_counter() - t0
    plain = B.exec_cfg("plain")
    t0 = time.perf_counter()
    for i in range(256):
        o = B.bd_query_batch(dg, s5[i:i + 1], t5[i:i + 1], 0.05, Lq, seed, pol, plain, uid=[i])
        assert o["beta"][0] == r_b["beta"][i]
    torch.cuda.synchronize()
    dt_p = time.perf_counter() - t0
    steps5 = B.bd_plan(dg, s5, t5, 0.05, Lq, pol)["walk_steps"].astype(float)
    out["modes_eps005_L1000"] = {
        "walk_counts": ("throughput setting, not calibrated: about 1/150 of the walk steps that meet eps "
                        "(see modes_eps005_L1000_calibrated)"),
        "queries": 4096, "walk_steps_per_query_mean": float(steps5.mean()),
        "plain_queries_per_s": 256 / dt_p, "batched_queries_per_s": 4096 / dt_b,
        "served_queries_per_s": 4096 / dt_s,
        "batched_vs_plain": (4096 / dt_b) / (256 / dt_p), "served_vs_plain": (4096 / dt_s) / (256 / dt_p),
        "plain_walk_steps_per_s": float(steps5[:256].sum()) / dt_p,
        "batched_walk_steps_per_s": float(steps5.sum()) / dt_b}
    srv.destroy()
    out["modes_eps005_L1000_calibrated"] = calibrated_modes(B, torch, dg, s5[:calibrated_queries],
                                                            t5[:calibrated_queries], seed)
    dg.free()
    return out


def calibrated_modes(B, torch, dg, s, t, seed):
    """Plain (one query per launch), batched and served on the same queries at
    the walk counts calibrated for this graph at eps = 0.05, L = 1000."""
    from paper_2512_05460_amd.budgets import BUDGETS, budget_policy

    pol = budget_policy("cl10m@1000")
    nq = s.size
    plan = B.bd_plan(dg, s, t, 0.05, 1000, pol)
    steps = plan["walk_steps"].astype(float)
    log(f"served: calibrated walk counts, {nq} queries, {steps.sum():.3e} walk steps per mode")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ref = [B.bd_query_batch(dg, s[i:i + 1], t[i:i + 1], 0.05, 1000, seed, pol, B.exec_cfg("plain"), uid=[i])
           for i in range(nq)]
    torch.cuda.synchronize()
    dt_p = time.perf_counter() - t0
    t0 = time.perf_counter()
    rb = B.bd_query_batch(dg, s, t, 0.05, 1000, seed, pol, B.exec_cfg("batched"))
    torch.cuda.synchronize()
    dt_b = time.perf_counter() - t0
    srv = B.Server(dg, pol)
    t0 = time.perf_counter()
    rids = [srv.submit(s[j:j + 4], t[j:j + 4], 0.05, 1000, seed, uid=np.arange(j, j + 4)) for j in range(0, nq, 4)]
    outs = [srv.wait(r)[0] for r in rids]
    dt_s = time.perf_counter() - t0
    srv.destroy()
    beta_p = np.array([r["beta"][0] for r in ref])
    assert np.array_equal(beta_p, rb["beta"]) and np.array_equal(np.concatenate([o["beta"] for o in outs]), rb["beta"])
    c_B, c_R, how = BUDGETS["cl10m@1000"]
    return {
        "walk_counts": "calibrated against binary64 CG distances (tests/golden): eps-accurate",
        "policy": {"kind": "scaled", "c_B": c_B, "c_R": c_R, "calibration": how},
        "queries": nq, "B": int(plan["B"][0]), "K": int(plan["K"][0]),
        "R": {"median": float(np.median(plan["R"])), "max": int(plan["R"].max())},
        "walk_steps_per_query": {"mean": float(steps.mean()), "median": float(np.median(steps)),
                                 "max": float(steps.max())},
        "plain_queries_per_s": nq / dt_p, "batched_queries_per_s": nq / dt_b, "served_queries_per_s": nq / dt_s,
        "batched_vs_plain": dt_p / dt_b, "served_vs_plain": dt_p / dt_s,
        "plain_walk_steps_per_s": steps.sum() / dt_p, "batched_walk_steps_per_s": steps.sum() / dt_b,
        "note": ("each query carries ~1e6-1e7 walk pairs against ~5e5 lane slots, so one query already fills "
                 "the device and batching adds little; the >= 5x regime is queries too small to fill it")}


def scale_cl40m_default(B, torch, stream, pairs=32, thr_queries=65536):
    """The scale graph in the default run: Chung-Lu n=4*10^7 (mean degree 25,
    exponent 2.2, largest component, about 10^9 adjacency entries) in the
    layout the library picks (fat). (1) The first `pairs` of its 64 CG
    reference pairs at eps = 0.05, L = 1000 and the calibrated walk counts:
    fraction within eps of the exact distance and the rate; the L = 10000 half
    of the workload is priced from the planner at the measured rate. (2) The
    first `thr_queries` of its 262,144 queries (L over {1000, 10000}) at the
    throughput setting, in one persistent launch: walk steps/s and the HBM
    bytes per step from the committed counters."""
    from paper_2512_05460_amd.budgets import BUDGETS, budget_policy
    from paper_2512_05460_amd.calibrate import load_reference
    from synth import graphs, queries

    log("scale: building Chung-Lu n=4e7")
    t0 = time.perf_counter()
    g = graphs.workload_graph("cl40m")
    t_gen = time.perf_counter() - t0
    t0 = time.perf_counter()
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_AUTO | B.BD_SKIP_VALIDATION)
    t_load = time.perf_counter() - t0
    info = dg.info()
    seed = graphs.PHILOX_SEED
    ref = load_reference(os.path.join(ROOT, "tests", "golden", "cl40m_cg_reference.txt"))
    s = ref["s"][:pairs].astype(np.int32)
    t = ref["t"][:pairs].astype(np.int32)
    pol = budget_policy("cl40m@1000")
    log(f"scale: {pairs} reference pairs at calibrated walk counts, L=1000")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r, st = B.bd_query_batch(dg, s, t, 0.05, 1000, seed, pol, B.exec_cfg("batched"), stream=stream,
                             uid=ref["index"][:pairs].astype(np.uint32), with_stats=True)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    assert np.all(r["status"] == 0)
    err = np.abs(r["beta"] - ref["beta_cg"][:pairs]) / ref["beta_cg"][:pairs]
    steps = r["walk_steps"].astype(float)
    sps = steps.sum() / dt
    # the L = 10000 half at its own calibrated walk counts, priced by the
    # planner (a query takes ~1.7e12 walk steps, ~30 s of the GPU: run by the
    # calibration tool, not here)
    c_B, c_R, how = BUDGETS["cl40m@1000"]
    c_B10, c_R10, how10 = BUDGETS["cl40m@10000"]
    p10 = B.bd_plan(dg, s, t, 0.05, 10000, budget_policy("cl40m@10000"))["walk_steps"].astype(float)
    calibrated = {
        "walk_counts": "calibrated against binary64 CG distances (tests/golden): eps-accurate",
        "policy": {"kind": "scaled", "c_B": c_B, "c_R": c_R, "calibration": how},
        "pairs": pairs, "L": 1000, "within_eps": float((err <= 0.05).mean()),
        "median_rel_err": float(np.median(err)),
        "R": {"median": float(np.median(r["R"])), "max": int(r["R"].max())},
        "walk_steps_per_query": {"mean": float(steps.mean()), "max": float(steps.max())},
        "queries_per_s": pairs / dt, "walk_steps_per_s": sps,
        "kernel_walk_steps_per_s": steps.sum() / (st["walk_kernel_ms"] / 1e3),
        "L10000": {"policy": {"kind": "scaled", "c_B": c_B10, "c_R": c_R10, "calibration": how10},
                   "walk_steps_per_query_mean": float(p10.mean()),
                   "seconds_per_query_at_measured_rate": float(p10.mean() / sps),
                   "note": ("planner: these pairs at L=10000; accuracy from the calibration tool's runs "
                            "(budgets.py), not run here")}}
    s2, t2, eps2, L2 = queries.workload_batch("cl40m", g.n, thr_queries)
    tpol = budget_policy("cl40m")
    tplan = B.bd_plan(dg, s2, t2, eps2, L2, tpol)
    tsteps = float(tplan["walk_steps"].sum())
    log(f"scale: {thr_queries} queries at the throughput setting, {tsteps:.3e} walk steps")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r2, st2 = B.bd_query_batch(dg, s2, t2, eps2, L2, seed, tpol, B.exec_cfg("batched"), stream=stream,
                               with_stats=True)
    torch.cuda.synchronize()
    dt2 = time.perf_counter() - t0
    assert np.all(r2["status"] == 0)
    ksps = tsteps / (st2["walk_kernel_ms"] / 1e3)
    thr = {"walk_counts": BUDGETS["cl40m"][2] + " (not eps-accurate: compare walk_steps_per_query_mean "
                                                 "with calibrated_L1000)",
           "queries": thr_queries, "walk_steps": tsteps, "walk_steps_per_query_mean": tsteps / thr_queries,
           "queries_per_s": thr_queries / dt2,
           "walk_steps_per_s": tsteps / dt2, "kernel_walk_steps_per_s": ksps}
    kv, why = read_counters(FAT_SCALE_COUNTERS)
    if info["layout"] == 1 and kv is not None:
        bps = float(kv["hbm_read_bytes_per_step"])
        thr["hbm_roofline"] = {"bound": "hbm", "bytes_per_step": bps, "achieved": bps * ksps / 1e9,
                               "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": bps * ksps / 1e9 / HBM_PEAK_GBS,
                               "algorithmic_bytes_per_step": BYTES_PER_STEP,
                               "algorithmic_frac": BYTES_PER_STEP * ksps / 1e9 / HBM_PEAK_GBS}
    else:
        thr["hbm_roofline"] = {"note": why if kv is None else "not the fat layout"}
    dg.free()
    return {"workload": ("Chung-Lu n=40,000,000 mean degree 25 exponent 2.2 LCC; eps=0.05; 64 CG reference "
                         "pairs; 262,144 uniform pairs with L over {1000, 10000}"),
            "graph": {"n": g.n, "nnz": g.nnz, "generate_s": t_gen, "load_s": t_load,
                      "layout": LAYOUT_NAMES[info["layout"]], "device_bytes": info["device_bytes"]},
            "calibrated_L1000": calibrated, "throughput_setting": thr}


def scale_cl40m(B, torch, stream, served_queries=65536, which=("csr", "hubs", "auto"), refs=False):
    """The scale workload: Chung-Lu n=4*10^7 (mean degree 25, exponent 2.2,
    largest component, about 10^9 adjacency entries; native generator); the
    262,144 queries (eps = 0.05, L over {1000, 10000}) in one persistent launch
    on the CSR layout, the compact layout with hubs first (4-byte ids at this
    size) and the layout the library picks (fat), then on the last the first
    `served_queries` of them as requests of 4,096 submitted together to the
    server; throughput walk counts. `which` selects among the three layouts
    (the served part runs on the last one selected)."""
    from paper_2512_05460_amd.budgets import BUDGETS, budget_policy
    from synth import graphs, queries

    log("scale: building Chung-Lu n=4e7")
    t0 = time.perf_counter()
    g = graphs.workload_graph("cl40m")
    t_gen = time.perf_counter() - t0
    s, t, eps, Ls = queries.workload_batch("cl40m", g.n)
    pol = budget_policy("cl40m")
    seed = graphs.PHILOX_SEED
    layouts = {}
    r = dg = None
    # CSR (16-byte node entries), the compact layout with hubs first (8-byte
    # entries, 4-byte ids above 2^24 nodes, hubs in LDS), then the automatic
    # choice (fat: one 16-byte entry per step), which also runs the served
    # part; the first load validates the graph, the others reuse its arrays
    cand = [("csr", "csr, hubs first", B.BD_LAYOUT_CSR | B.BD_RELABEL_DEGREE),
            ("hubs", "compact, hubs first", B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE),
            ("fatt", "fat, ordinary loads", B.BD_LAYOUT_FAT | B.BD_TEMPORAL),
            ("auto", "automatic", B.BD_LAYOUT_AUTO)]
    for key, name, flags in [c for c in cand if c[0] in which]:
        if dg is not None:
            dg.free()
            flags |= B.BD_SKIP_VALIDATION
        log(f"scale: n={g.n} nnz={g.nnz}; loading ({name})")
        t0 = time.perf_counter()
        dg = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
        t_load = time.perf_counter() - t0
        plan = B.bd_plan(dg, s, t, eps, Ls, pol)
        steps = float(plan["walk_steps"].sum())
        log(f"scale: {s.size} queries, {steps:.3e} walk steps, batched ({name})")
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        r, st = B.bd_query_batch(dg, s, t, eps, Ls, seed, pol, B.exec_cfg("batched"), stream=stream,
                                 with_stats=True)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        assert np.all(r["status"] == 0)
        roof = max((B.bd_gather_roofline(dg, c, 1000) for c in (2, 4, 8)), key=lambda x: x["steps_per_s"])
        layouts[name] = {"layout": LAYOUT_NAMES[dg.info()["layout"]], "nontemporal": dg.info()["nontemporal"],
                         "device_bytes": dg.info()["device_bytes"], "load_s": t_load,
                         "batched_queries_per_s": s.size / dt, "batched_walk_steps_per_s": steps / dt,
                         "kernel_walk_steps_per_s": steps / (st["walk_kernel_ms"] / 1e3),
                         "random_start_gather_steps_per_s": roof["steps_per_s"],
                         "vs_random_start_gather": steps / (st["walk_kernel_ms"] / 1e3) / roof["steps_per_s"]}
    m = served_queries
    dg_layout = dg.info()["layout"]
    srv = B.Server(dg, pol)
    log(f"scale: served, {m} queries as requests of 4096")
    t0 = time.perf_counter()
    rids = [srv.submit(s[j:j + 4096], t[j:j + 4096], eps[j:j + 4096], Ls[j:j + 4096], seed,
                       uid=np.arange(j, j + 4096)) for j in range(0, m, 4096)]
    lat = []
    for k, rid in enumerate(rids):
        o, l_ms = srv.wait(rid)
        assert np.array_equal(o["beta"], r["beta"][4096 * k:4096 * k + 4096])
        lat.append(l_ms)
    dts = time.perf_counter() - t0
    srv.destroy()
    steps_m = float(plan["walk_steps"][:m].sum())
    # the reference routines at this size: lambda by power iteration (section
    # 2.1) and beta^(L) by sparse products (Lemma 2.3), on the device
    ref_routines = None
    if not refs:
        dg.free()
        dg = None
    else:
        log("scale: lambda (200 power iterations) and beta^(1000) of 8 pairs")
        free0 = torch.cuda.mem_get_info()[0]
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        lam = B.bd_graph_lambda(dg, 200, 7, stream=stream)
        dt_lam = time.perf_counter() - t0
        t0 = time.perf_counter()
        bl = B.bd_truncated_beta(dg, s[:8], t[:8], 1000, stream=stream)
        dt_bl = time.perf_counter() - t0
        ref_routines = {
            "lambda": {"iterations": 200, "estimate": lam, "seconds": dt_lam,
                       "device_bytes": 2 * 8 * g.n + 4 * 512 * 8 + 8},
            "beta_truncated": {"pairs": 8, "L": 1000, "seconds": dt_bl, "beta": [float(x) for x in bl],
                               "device_bytes_per_pass": 2 * 8 * g.n * 8, "free_device_bytes_before": int(free0)}}
        dg.free()
    c_B, c_R, how = BUDGETS["cl40m"]
    best = max(layouts.values(), key=lambda x: x["batched_queries_per_s"])
    # the fat layout's HBM roofline: bytes per step from the committed counters
    # (one 128-byte line per step), at the walk-step rate measured here
    if "automatic" in layouts and layouts["automatic"]["layout"] == "fat":
        kv, why = read_counters(FAT_SCALE_COUNTERS)
        a = layouts["automatic"]
        if kv is None:
            a["hbm_roofline"] = {"note": why}
        else:
            bps = float(kv["hbm_read_bytes_per_step"])
            achieved = bps * a["kernel_walk_steps_per_s"] / 1e9
            a["hbm_roofline"] = {"bound": "hbm", "bytes_per_step": bps, "achieved": achieved, "peak": HBM_PEAK_GBS,
                                 "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS,
                                 "note": "HBM read bytes per step from TCC_EA0_RDREQ_* counters (128-byte requests)"}
    return {
        "workload": ("Chung-Lu n=40,000,000 mean degree 25 exponent 2.2 LCC; 262,144 uniform pairs; eps=0.05; "
                     "L over {1000, 10000}"),
        "graph": {"n": g.n, "nnz": g.nnz, "generate_s": t_gen},
        "policy": {"kind": "scaled", "c_B": c_B, "c_R": c_R, "calibration": how},
        "walk_steps": steps,
        "layouts": layouts,
        "best_layout": best["layout"], "served_layout": LAYOUT_NAMES[dg_layout],
        "batched_queries_per_s": best["batched_queries_per_s"],
        "batched_walk_steps_per_s": best["batched_walk_steps_per_s"],
        "served_queries": m, "served_queries_per_s": m / dts, "served_walk_steps_per_s": steps_m / dts,
        "served_request_latency_ms": {"p50": float(np.percentile(lat, 50)), "max": float(max(lat))},
        "reference_routines": ref_routines,
    }


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--queries", type=int, default=32, help="queries per step")
    ap.add_argument("--layout", choices=["hubs", "hubsid", "hubsidw", "hubsidd", "hubsidn", "compact", "csr", "fat",
                                         "auto"],
                    default="hubsid",
                    help="hubs: compact layout with nodes in descending-degree order and hub entries in LDS; "
                         "hubsid: the same with the probe on storage ids (every node's row offset and degree in "
                         "LDS from the degree-run table; two work groups per CU, one replica pair per thread, "
                         "at this size); hubsidw: hubsid with one work group per CU and two pairs per thread; "
                         "hubsidd: hubsid with the row offsets of the 36,864 highest-degree nodes in LDS instead; "
                         "hubsidn: hubsid forced to two work groups per CU; auto: the library's choice (hubs at "
                         "this size)")
    ap.add_argument("--no-batched", action="store_true")
    ap.add_argument("--no-served", action="store_true")
    ap.add_argument("--no-roofline", action="store_true")
    ap.add_argument("--no-small", action="store_true")
    ap.add_argument("--no-grid", action="store_true")
    ap.add_argument("--served-profile", action="store_true",
                    help="n=1e7 served block: only the capacity burst (for profiler counters on its slices)")
    ap.add_argument("--small-layout", choices=["compact", "hubsid"], default="compact",
                    help="tables of the small-query block")
    ap.add_argument("--grid-profile", type=int, default=0, metavar="CHUNK_PAIRS",
                    help="grid block: only one eager batched launch of the whole set with this chunking (for "
                         "profiler counters)")
    ap.add_argument("--grid-layout", choices=["auto", "hubsid"], default="hubsid",
                    help="grid tables: hubs first with the probe on storage ids (the degree-run table in LDS; "
                         "the default), or the library's choice (fat at this size)")
    ap.add_argument("--no-sharing", action="store_true")
    ap.add_argument("--no-stabilize", action="store_true")
    ap.add_argument("--scale-layouts", default="csr,hubs,auto",
                    help="layouts of the scale report, from csr, hubs, fatt (fat with ordinary loads), auto")
    ap.add_argument("--scale", action="store_true",
                    help="also run the Chung-Lu n=4e7 workload (about 3 minutes more)")
    ap.add_argument("--scale-refs", action="store_true",
                    help="with --scale: time lambda and beta^(1000) of 8 pairs at n=4e7")
    ap.add_argument("--no-served-cl10m", action="store_true")
    ap.add_argument("--no-scale-cl40m", action="store_true",
                    help="leave out the default n=4e7 block (calibrated reference pairs, throughput setting)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--copy-calib", type=int, default=0,
                    help="also run a device copy of this many MiB (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) > 1:
        print("bench.py runs on one GPU only (--gpus 1): queries shard across GPUs with nothing "
              "exchanged but a few block sums per query, so it reports one GPU's share.",
              file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_2512_05460_amd import binding as B
    from paper_2512_05460_amd.budgets import BUDGETS, budget_policy
    from synth import graphs, queries

    torch.cuda.set_device(0)
    dev = B.bd_device_info()
    log("device:", dev)
    g = graphs.workload_graph(WORKLOAD)
    s_all, t_all = queries.uniform_pairs(g.n, 4096, graphs.GRAPH_SEED + 1 + graphs.QUERY_SEED_OFFSET)
    nq = args.queries
    s, t = s_all[:nq], t_all[:nq]
    flags = {"hubs": B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE,
             "hubsid": B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS,
             "hubsidw": B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS | B.BD_WIDE_HUBS,
             "hubsidd": B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS | B.BD_DIRECT_HUBS,
             "hubsidn": B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS | B.BD_NARROW_HUBS,
             "compact": B.BD_LAYOUT_COMPACT,
             "csr": B.BD_LAYOUT_CSR | B.BD_RELABEL_DEGREE,
             "fat": B.BD_LAYOUT_FAT | B.BD_RELABEL_DEGREE, "auto": B.BD_LAYOUT_AUTO}[args.layout]
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
    pol = budget_policy(WORKLOAD)
    seed = graphs.PHILOX_SEED
    plan = B.bd_plan(dg, s, t, EPS, L, pol)
    assert np.all(plan["status"] == 0), plan["status"]
    steps_per_batch = float(plan["walk_steps"].sum())
    # the timed batch is the first nq of the 4,096 pairs; its walk work against
    # the whole set's (host planner only), since per-query budgets are heavy-tailed
    plan_set = B.bd_plan(dg, s_all, t_all, EPS, L, pol)
    set_steps = plan_set["walk_steps"].astype(np.float64)
    log(f"batch: {nq} queries, K={int(plan['K'][0])}, R median {int(np.median(plan['R']))} "
        f"max {int(plan['R'].max())}, {steps_per_batch:.3e} walk steps "
        f"({steps_per_batch / nq / set_steps.mean():.2f}x the set's mean per query)")
    plain = B.exec_cfg("plain")
    stream = torch.cuda.current_stream()

    def run_plain():
        lat, kms, launches = [], 0.0, 0
        for i in range(nq):
            t0 = time.perf_counter()
            r, st = B.bd_query_batch(dg, s[i:i + 1], t[i:i + 1], EPS, L, seed, pol, plain, uid=[i],
                                     stream=stream, with_stats=True)
            lat.append((time.perf_counter() - t0) * 1e3)
            kms += st["walk_kernel_ms"]
            launches += st["launches"]
            assert r["status"][0] == 0
        return lat, kms, launches

    for w in range(args.warmup):
        log(f"warmup {w + 1}/{args.warmup}")
        run_plain()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    lat_all, kms_all, launches_all = [], 0.0, 0
    for k in range(args.steps):
        lat, kms, launches = run_plain()
        lat_all += lat
        kms_all += kms
        launches_all += launches
        log(f"step {k + 1}/{args.steps}: {sum(lat):.0f} ms")
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    qps = nq * args.steps / elapsed
    walk_sps = steps_per_batch * args.steps / elapsed
    kernel_sps = steps_per_batch * args.steps / (kms_all / 1e3)
    achieved_gbs = kernel_sps * BYTES_PER_STEP / 1e9

    extra = {}
    if not args.no_batched:
        log("batched mode, same batch")
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        r, st = B.bd_query_batch(dg, s, t, EPS, L, seed, pol, B.exec_cfg("batched"), stream=stream,
                                 with_stats=True)
        torch.cuda.synchronize()
        dtb = time.perf_counter() - t1
        assert np.all(r["status"] == 0)
        extra["batched"] = {"queries_per_s": nq / dtb, "walk_steps_per_s": steps_per_batch / dtb,
                            "kernel_ms": st["walk_kernel_ms"], "vs_plain": (nq / dtb) / qps}
    if not args.no_served:
        log("served mode, same batch as 4 requests")
        srv = B.Server(dg, pol)
        t1 = time.perf_counter()
        rids = [srv.submit(s[i::4], t[i::4], EPS, L, seed, uid=np.arange(nq)[i::4]) for i in range(4)]
        lats = []
        for rid in rids:
            out, lat = srv.wait(rid)
            assert np.all(out["status"] == 0)
            lats.append(lat)
        dts = time.perf_counter() - t1
        srv.destroy()
        extra["served"] = {"queries_per_s": nq / dts, "vs_plain": (nq / dts) / qps,
                           "request_latency_ms": lats}
    if not args.no_sharing:
        # the same batch, plain mode, with walk sharing at its own calibrated budget
        from paper_2512_05460_amd.budgets import SHARED_BUDGETS
        log("walk sharing, same batch, plain mode")
        spol = budget_policy(WORKLOAD, shared=True)
        splan = B.bd_plan(dg, s, t, EPS, L, spol)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        kms_sh = 0.0
        for i in range(nq):
            r, st = B.bd_query_batch(dg, s[i:i + 1], t[i:i + 1], EPS, L, seed, spol, plain, uid=[i],
                                     stream=stream, with_stats=True)
            assert r["status"][0] == 0
            kms_sh += st["walk_kernel_ms"]
        torch.cuda.synchronize()
        dts = time.perf_counter() - t1
        M, cb, cr, how = SHARED_BUDGETS[WORKLOAD]
        extra["walk_sharing"] = {
            "what": ("probes of each median-of-means block scored in groups of M on one set of walks "
                     "(an extension of Algorithm 1), at its own calibrated walk counts"),
            "policy": {"kind": "scaled", "share": M, "c_B": cb, "c_R": cr, "calibration": how},
            "queries_per_s": nq / dts, "vs_plain": (nq / dts) / qps,
            "walk_steps_per_s": float(splan["walk_steps"].sum()) / dts,
            "kernel_walk_steps_per_s": float(splan["walk_steps"].sum()) / (kms_sh / 1e3)}
    if not args.no_stabilize:
        # the stabilization rule (section 4.3) and its proxy relative error
        # against the estimate at L_max = 256, eps = 0.1, on the same graph
        log("stabilization rule, 32 pairs, eps=0.1, L_max=256")
        s_st, t_st = s_all[-32:], t_all[-32:]
        t1 = time.perf_counter()
        r_st, Ls = B.bd_query_stabilized(dg, s_st, t_st, 0.1, 256, seed, pol)
        dt_st = time.perf_counter() - t1
        r_mx = B.bd_query_batch(dg, s_st, t_st, 0.1, 256, seed, pol)
        proxy = np.abs(r_st["beta"] - r_mx["beta"]) / np.abs(r_mx["beta"])
        extra["stabilization"] = {
            "eps": 0.1, "L_max": 256, "queries": 32, "seconds": dt_st,
            "L_stop_counts": {str(int(v)): int((Ls == v).sum()) for v in np.unique(Ls)},
            "proxy_rel_error": {"p50": float(np.median(proxy)), "p90": float(np.percentile(proxy, 90)),
                                "max": float(proxy.max()), "frac_within_eps": float((proxy <= 0.1).mean())}}
    if not args.no_small:
        extra["small_queries"] = small_queries(B, torch, stream, layout=args.small_layout)
    if not args.no_grid:
        extra["grid_batched"] = grid_batched(B, torch, stream, layout=args.grid_layout,
                                             profile_chunk_pairs=args.grid_profile)
    if not args.no_served_cl10m:
        extra["served_cl10m"] = served_cl10m(B, torch, profile=args.served_profile)
    if not args.no_scale_cl40m and not args.scale:
        extra["scale_cl40m"] = scale_cl40m_default(B, torch, stream)
    if args.scale:
        which = args.scale_layouts.split(",")
        if not which or not set(which) <= {"csr", "hubs", "fatt", "auto"}:
            raise SystemExit(f"--scale-layouts takes csr, hubs, fatt, auto; got {args.scale_layouts}")
        extra["scale_cl40m"] = scale_cl40m(B, torch, stream, which=which, refs=args.scale_refs)
    roof = None
    if not args.no_roofline:
        log("gather roofline")
        best = max((B.bd_gather_roofline(dg, c, 1000) for c in (2, 4, 8)), key=lambda r: r["steps_per_s"])
        roof = {"steps_per_s": best["steps_per_s"], "chains_per_lane": best["chains_per_lane"],
                "frac": kernel_sps / best["steps_per_s"],
                "what": ("the general walk kernel's dependent loads on this layout's tables, no Philox or probe "
                         "arithmetic; sign_kernel reads one 3-byte position a step from tables of its own")}
    if args.copy_calib:
        n = args.copy_calib * (1 << 20) // 4
        x = torch.empty(n, dtype=torch.float32, device="cuda")
        y = torch.empty_like(x)
        y.copy_(x)
        torch.cuda.synchronize()
        extra["copy_calib_bytes"] = n * 4

    cpu = None
    if not args.no_cpu_baseline:
        from oracle import planner as OP
        c_B, c_R, _ = BUDGETS[WORKLOAD]
        op = OP.Policy("scaled", c_B=c_B, c_R=c_R)
        plans = [OP.plan(EPS, L, int(g.deg[s[i]]), int(g.deg[t[i]]), g.d_min, op) for i in range(nq)]
        log("cpu baseline (oracle, bounded sample)")
        cpu = cpu_baseline(g, s, t, plans, seed)

    traffic_per_step, traffic_note = counter_traffic()
    steps_per_launch = steps_per_batch * args.steps / max(1, launches_all)
    c_B, c_R, how = BUDGETS[WORKLOAD]
    out = {
        "metric": "queries/s at eps=0.05, L=1000",
        "value": qps,
        "unit": "queries/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": elapsed / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": ("Chung-Lu n=100,000 mean degree 10 exponent 2.5 LCC; uniform (s,t) pairs; "
                         "eps=0.05, L=1000; plain mode, one query per launch"),
            "queries_per_step": nq,
            "layout": args.layout,
            "lds_nodes": int(dg.info()["lds_hubs"]),
            "policy": {"kind": "scaled", "c_B": c_B, "c_R": c_R, "delta": 0.01, "calibration": how},
            "K": int(plan["K"][0]), "R_median": int(np.median(plan["R"])),
            "walk_steps_per_step": steps_per_batch,
            "sample": (f"the first {nq} of 4,096 uniform pairs, the same batch every step; latency "
                       "percentiles are over these queries"),
            "sample_walk_steps_per_query": steps_per_batch / nq,
            "set_walk_steps_per_query": {"mean": float(set_steps.mean()), "median": float(np.median(set_steps)),
                                         "max": float(set_steps.max())},
            "sample_vs_set_walk_steps": steps_per_batch / nq / float(set_steps.mean()),
            "set_queries_per_s_at_measured_rate": walk_sps / float(set_steps.mean()),
        },
        "walk_steps_per_s": walk_sps,
        "latency_ms": {"p50": float(np.percentile(lat_all, 50)), "p99": float(np.percentile(lat_all, 99))},
        "roofline": {
            "bound": "hbm",
            "achieved": achieved_gbs,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved_gbs / HBM_PEAK_GBS,
            "traffic": None if traffic_per_step is None else traffic_per_step * steps_per_launch / 1e9,
            "traffic_unit": "GB per launch",
            "traffic_note": traffic_note,
            "kernel": ("sign_kernel; walk_kernel for queries that score a probe less often than its table "
                       "would be evaluated"),
            "avg_launch_ms": kms_all / max(1, launches_all),
            "walk_steps_per_launch": steps_per_launch,
            "kernel_walk_steps_per_s": kernel_sps,
            "bytes_per_step": BYTES_PER_STEP,
            "gather_roofline": roof,
            "l2": l2_requests(kernel_sps),
        },
        "cpu_baseline": cpu,
        "paper_context": ("per-query times of the same estimator in the paper (Table 3): one thread of an "
                          "AMD EPYC 7713, Python, eps=0.01, L by the stabilization rule; median 1.4 s / 9.9 s / "
                          "9.4 s and mean 34 s / 55 s / 301 s on Bluesky, Twitter-2010, Friendster (other graphs "
                          "and unstated walk counts: context, not a baseline)"),
        "device": dev,
        **extra,
    }
    print(json.dumps(out), flush=True)
    dg.free()


if __name__ == "__main__":
    main()
