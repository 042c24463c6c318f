"""Benchmark of the randomized mini-batch Bellman operator on one MI355X.

Workload (default): dense random MDP, n = 8192 states, m = 16 actions, rows
Dirichlet(0.1) stored FP32 (4.3 GB), costs U[0, 1), gamma = 0.99.  A step is
one MB-VI solve (vi_solve: every sweep runs the sweep order, the batch
partition, the row gather + backup, the action minimum, the batch commit,
the re-centring and the device-side stopping rule) from V = 0 until
max|V - V*| <= 1e-6, at the batch size with the best time to 1e-6.

Prints ONE JSON line with state-action backups/s over the timed steps, the
achieved HBM bandwidth of the solve kernel against the 8 TB/s peak, time to
1e-6 for each batch size (VI and MPI with K = 5), and the CPU oracle timed on
a bounded sample of the same workload.

    python bench.py [--steps K] [--warmup W] [--gpus 1]
"""
import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0
# batch size of each workload's counter runs: the one its bench line selects
PROFILE_B = {"dense-8192x16": 1024, "csr-1M-banded": 1_000_000, "csr-1M-uniform": 1_000_000}
METRIC = "state-action backups/s + HBM GB/s; time-to-ε=1e-6 vs batch size b"


def log(msg):
    print("[bench] " + msg, file=sys.stderr, flush=True)


# Device sources of each profiled kernel: a committed counter summary is
# used only while these files are unchanged.
_KERNEL_SOURCES = {
    "solve": ("mbdp_device.h", "mbdp_engines.h", "mbdp_kernels.hip", "mbdp_kernels_lp_dense.hip",
              "mbdp_kernels_lp_ell.hip", "mbdp_kernels_lp_band.hip", "mbdp_resident.h",
              "mbdp_resident.hip", "mbdp_resident_lp.hip"),
    "batch": ("mbdp_device.h", "mbdp_engines.h", "mbdp_batch.hip"),
    "multi": ("mbdp_device.h", "mbdp_multi.hip"),
}


def sources_hash(kernel="solve"):
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2110_02901_amd", "csrc")
    for f in _KERNEL_SOURCES[kernel]:
        with open(os.path.join(csrc, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def _traffic_file(workload):
    path = os.path.join(ROOT, "profiles", "traffic_%s.txt" % workload)
    if not os.path.exists(path):
        return {}
    vals = {}
    for line in open(path):
        if "=" in line and not line.startswith("#"):
            k, v = line.split("=", 1)
            vals[k.strip()] = v.strip()
    return vals


def committed_traffic(workload, b, sweeps_per_launch):
    """HBM bytes per launch from the committed rocprofv3 counter summary
    (sweeps x bytes per sweep + the one-off prologue), if the counters were
    taken with the current kernel sources at this batch size; else None."""
    vals = _traffic_file(workload)
    if vals.get("sources_hash") != sources_hash("solve") or vals.get("b") != str(b):
        return None
    try:
        per_sweep = float(vals["hbm_bytes_per_sweep"])
        prologue = float(vals["hbm_bytes_prologue"])
    except (KeyError, ValueError):
        return None
    return sweeps_per_launch * per_sweep + prologue


def host_info():
    """The host the CPU baseline runs on: logical CPUs, CPU model, BLAS threads."""
    model = "unknown"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    blas = 1
    try:
        from threadpoolctl import threadpool_info
        blas = max((t.get("num_threads", 1) for t in threadpool_info()), default=1)
    except Exception:
        pass
    return {"nproc": os.cpu_count(), "cpu_model": model, "blas_threads": int(blas)}


def _oracle_sweep_rate(mdp, b, seed, budget_s, threads=None):
    """Whole FP64 oracle sweeps of B_b from V = 0 until the budget is spent
    (at least one): (sweeps, seconds)."""
    import oracle
    from contextlib import nullcontext
    try:
        from threadpoolctl import threadpool_limits
        ctx = threadpool_limits(threads) if threads else nullcontext()
    except Exception:
        ctx = nullcontext()
    n = mdp.n
    V = np.zeros(n)
    sweeps = 0
    with ctx:
        t0 = time.perf_counter()
        c0 = time.process_time()
        while True:
            V, _, _ = oracle.mb_sweep(mdp, V, b, oracle.sweep_permutation(n, seed, sweeps))
            sweeps += 1
            if time.perf_counter() - t0 >= budget_s:
                break
        dt = time.perf_counter() - t0
        busy = time.process_time() - c0
    return sweeps, dt, busy / dt


def _oracle_small_time_to_eps(eps):
    """The oracle's MB-VI on the 64-state workload (its J* by policy
    iteration, untimed), timed from V = 0 to the first sweep with
    max|V - J*| <= eps: the whole time to eps, where the oracle finishes."""
    import oracle
    from paper_2110_02901_amd import inputs
    wl = inputs.WORKLOADS["dense-64x4"]
    P, c = inputs.dense_mdp(wl["n"], wl["m"], wl["alpha"], wl["data_seed"], dtype=np.float32)
    mdp = oracle.DenseMDP(P, c, wl["gamma"])
    Vs, _, _ = oracle.policy_iteration(mdp)
    b = wl["batch_sizes"][0]
    t0 = time.perf_counter()
    _, _, st = oracle.value_iteration(mdp, b, wl["perm_seed"], tol_dv=-1.0, V_ref=Vs, eps=eps)
    return {"workload": "dense-64x4", "b": b, "sweeps": st.sweeps,
            "seconds": time.perf_counter() - t0}


def cpu_baseline(mdp, wl_name, b, seed, budget_s=20.0, gpu_sweeps=None, eps=1e-6):
    """The FP64 oracle on the same MDP, timed on the host with every BLAS
    thread and with one thread (half the budget each), plus the oracle's time
    to eps on the 64-state workload and, for this workload, the measured
    sweep time times the GPU's sweep count (an extrapolation)."""
    host = host_info()
    n, m = mdp.n, mdp.m
    sw_all, dt_all, used_all = _oracle_sweep_rate(mdp, b, seed, budget_s / 2)
    sw_one, dt_one, _ = _oracle_sweep_rate(mdp, b, seed, budget_s / 2, threads=1)
    # cores: the threads the run kept busy (process CPU time over wall time)
    out = {"value": sw_all * n * m / dt_all, "unit": "backups/s",
           "cores": max(1, int(round(used_all))), "cores_busy": used_all,
           "kind": "oracle",
           "sample": "%d FP64 sweeps of B_b (b=%d) on the full %s MDP (n=%d, m=%d) from V=0 "
                     "in %.1f s with up to %d BLAS threads (%.1f busy on average); %d sweeps "
                     "in %.1f s with one"
                     % (sw_all, b, wl_name, n, m, dt_all, host["blas_threads"], used_all,
                        sw_one, dt_one),
           "one_thread_value": sw_one * n * m / dt_one,
           "host": host,
           "small_time_to_eps": _oracle_small_time_to_eps(eps)}
    if gpu_sweeps:
        out["time_to_eps_extrapolated_s"] = {
            "sweeps": gpu_sweeps, "all_threads": gpu_sweeps * dt_all / sw_all,
            "one_thread": gpu_sweeps * dt_one / sw_one,
            "note": "the GPU's sweep count to eps times the oracle's measured time per sweep"}
    return out


def run_multi(args, dev):
    """r cost vectors against the dense-8192x16 transitions stored in BF16
    (n = 8192, m = 16, rows Dirichlet(0.1), one scale per row), C[s, a, j] ~
    U[0, 1), gamma = 0.99, b = 1024, V0 = 0: one mdp_multi_solve until the
    largest change of a sweep over all vectors is <= 1e-8 (so every column is
    within 1e-8 gamma / (1 - gamma) ~ 1e-6 of its J*)."""
    import torch
    from paper_2110_02901_amd import binding as mb
    from paper_2110_02901_amd import inputs

    wl = inputs.WORKLOADS["dense-8192x16"]
    n, m, gamma, r, b, tol = wl["n"], wl["m"], wl["gamma"], args.multi_r, 1024, 1e-8
    seed = wl["perm_seed"]
    t0 = time.perf_counter()
    P, c = inputs.dense_mdp(n, m, wl["alpha"], wl["data_seed"], dtype=np.float32)
    rows = torch.from_numpy(P.reshape(n * m, n)).to(dev)
    codes, rscale = mb.mdp_quantize_rows(rows, "bf16")
    del rows
    h = mb.mdp_create_dense_q(codes.reshape(-1), "bf16", rscale, torch.from_numpy(c).to(dev), gamma)
    C = inputs.multi_costs(n, m, r, wl["data_seed"] + 100, dtype=np.float32)
    Cd = torch.from_numpy(C).to(dev)
    ws = mb.multi_workspace(h, r, b)
    log("multi-%dx%d: P in BF16 (%.2f GB), r = %d cost vectors, ready in %.1f s"
        % (n, m, codes.numel() * 2 / 1e9, r, time.perf_counter() - t0))
    V = torch.zeros(n, r, dtype=torch.float64, device=dev)
    bytes_sweep = n * m * (2 * n + 4) + n * m * r * 4 + n * r * 16
    if args.profile_sweeps:
        # counter runs: solves of exactly S and 3S sweeps, each after a fill of V
        out = {"workload": "multi-8192x16", "r": r, "b": b, "launches": [],
               "sources_hash": sources_hash("multi"), "algorithmic_bytes_per_sweep": bytes_sweep}
        for sweeps in (args.profile_sweeps, args.profile_sweeps, 3 * args.profile_sweeps):  # warm-up, S, 3S
            V.zero_()
            st = mb.mdp_multi_solve(h, Cd, V, b, seed, ws, tol_dv=-1.0, max_sweeps=sweeps)
            out["launches"].append({"sweeps": st["sweeps"], "recentrings": st["recentrings"]})
        print(json.dumps(out), flush=True)
        return

    def solve():
        V.zero_()
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        w0 = time.perf_counter()
        e0.record()
        st = mb.mdp_multi_solve(h, Cd, V, b, seed, ws, tol_dv=tol, max_sweeps=100000)
        e1.record()
        e1.synchronize()
        return st, e0.elapsed_time(e1) / 1e3, time.perf_counter() - w0

    for _ in range(args.warmup):
        solve()
    walls, gpus = [], []
    for _ in range(args.steps):
        st, g, w = solve()
        gpus.append(g)
        walls.append(w)
    if not st["converged"]:
        raise RuntimeError("multi-vector solve did not converge")
    sweeps = st["sweeps"]
    # per sweep of the single-vector BF16 kernel on the same handle, for comparison
    V1 = torch.zeros(n, dtype=torch.float32, device=dev)
    ws1 = mb.workspace(h, n)
    mb.vi_solve(h, V1, b, seed, ws1, tol_dv=-1.0, max_sweeps=5)
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    mb.vi_solve(h, V1, b, seed, ws1, tol_dv=-1.0, max_sweeps=40)
    e1.record()
    e1.synchronize()
    single_sweep_s = e0.elapsed_time(e1) / 1e3 / 40
    wall = float(np.mean(walls))
    gpu = float(np.mean(gpus))
    backups = sweeps * n * m * r
    gbps = sweeps * bytes_sweep / gpu / 1e9
    traffic = None
    vals = _traffic_file("multi-8192x16-r%d" % r)
    if vals.get("sources_hash") == sources_hash("multi"):
        try:
            traffic = sweeps * float(vals["hbm_bytes_per_sweep"]) + float(vals["hbm_bytes_prologue"])
        except (KeyError, ValueError):
            traffic = None
    tflops = sweeps * 2.0 * 2 * n * m * n * r / gpu / 1e12  # two BF16 terms of W
    log("multi r=%d: %d sweeps, %d re-centrings, %.1f ms (%.3f ms per sweep; single-vector "
        "BF16 sweep %.3f ms, so %.1fx the backups per second of r single-vector solves)"
        % (r, sweeps, st["recentrings"], gpu * 1e3, gpu / sweeps * 1e3, single_sweep_s * 1e3,
           r * single_sweep_s / (gpu / sweeps)))
    cpu = None
    if not args.no_cpu_baseline:
        # the oracle's backups of a sample of states against the same stored rows
        import oracle
        from oracle import multi as om
        from oracle import quantize as qz
        try:
            from threadpoolctl import threadpool_info
            cores = max((t.get("num_threads", 1) for t in threadpool_info()), default=1)
        except Exception:
            cores = 1
        sample = oracle.sweep_permutation(n, seed, 0)[:64]
        q_ref, s_ref = qz.quantize_rows(P[sample].reshape(-1, n), "bf16")
        Ps = qz.dequantized(q_ref, s_ref, "bf16").reshape(len(sample), m, n)
        Vh = np.random.Generator(np.random.Philox(1)).random((n, r))
        reps, t0 = 0, time.perf_counter()
        while time.perf_counter() - t0 < 10.0:
            om.multi_q_values(Ps, C[sample].astype(np.float64), gamma,
                              np.arange(len(sample)), Vh).min(axis=1)
            reps += 1
        dt = time.perf_counter() - t0
        cpu = {"value": reps * len(sample) * m * r / dt, "unit": "backups/s", "cores": int(cores),
               "kind": "oracle",
               "sample": "%d x the FP64 multi-vector backups of 64 states (m = %d, r = %d) against "
                         "their stored BF16 rows, %.1f s" % (reps, m, r, dt)}
    line = {
        "metric": METRIC, "value": backups / wall, "unit": "backups/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": wall * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "multi-8192x16", "n": n, "m": m, "r": r, "alpha": wl["alpha"],
                   "gamma": gamma, "b": b, "storage": "bf16", "tol_dv": tol},
        "sweeps": sweeps, "recentrings": st["recentrings"], "solve_ms": gpu * 1e3,
        "single_vector_sweep_ms": single_sweep_s * 1e3, "mfma_tflops": tflops,
        "roofline": {"bound": "hbm", "achieved": gbps, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": gbps / HBM_PEAK_GBPS, "traffic": traffic,
                     "kernel": "multi_gemm_kernel + multi_commit_kernel (whole solve)",
                     "algorithmic_bytes_per_backup": "(2 n + 4) / r + 4 + 16 / m"},
        "cpu_baseline": cpu,
    }
    print(json.dumps(line), flush=True)


def run_batch(args, dev):
    """512 independent dense MDPs, n ~ U[256, 4096], m = 8, Dirichlet(1) rows in
    BF16 with one scale per row, c ~ U[0, 1), gamma ~ U[0.9, 0.99], b =
    ceil(n / 8), all solved in one launch (replayed from a hipGraph) until
    max |dV| <= 1e-8 (so max |V - J*| <= 1e-8 gamma / (1 - gamma) < 1e-6).
    The MDPs are drawn on the GPU (torch's seeded generator)."""
    import torch
    from paper_2110_02901_amd import binding as mb
    from paper_2110_02901_amd import inputs
    from paper_2110_02901_amd import tune

    count, m, tol = 512, 8, 1e-8
    g = np.random.Generator(np.random.Philox(104))
    ns = g.integers(256, 4097, count)
    gammas = g.uniform(0.9, 0.99, count)
    gen = torch.Generator(device=dev)
    gen.manual_seed(104)
    t0 = time.perf_counter()
    items = []
    total_bytes = 0
    padded_bytes = 0
    for i in range(count):
        n = int(ns[i])
        ld = (n + 63) // 64 * 64  # rows of whole 128-byte lines
        rows = torch.zeros(n * m, ld, dtype=torch.float32, device=dev)
        w = torch._standard_gamma(torch.ones(n * m, n, device=dev), generator=gen)
        rows[:, :n] = w / w.sum(dim=1, keepdim=True)
        del w
        codes, scale = mb.mdp_quantize_rows(rows, "bf16")
        del rows
        c = torch.rand(n, m, device=dev, generator=gen)
        items.append({"n": n, "m": m, "dtype": "bf16", "ld": ld, "P": codes.reshape(-1),
                      "row_scale": scale, "c": c, "gamma": float(gammas[i]),
                      "b": (n + 7) // 8, "seed": 2000 + i,
                      "V": torch.zeros(n, dtype=torch.float64, device=dev), "policy": None,
                      "lanes": 0})
        total_bytes += n * m * (2 * n + 8)  # the method's bytes: row, scale, cost
        padded_bytes += n * m * (2 * ld + 8)
    torch.cuda.synchronize()
    log("generated %d MDPs (%.1f GB of BF16 rows) in %.1f s"
        % (count, total_bytes / 1e9, time.perf_counter() - t0))
    tuned = None
    if not args.no_tune:
        t0 = time.perf_counter()
        tuned = tune.tune_lanes(items)
        log("lane widths tuned in %.1f s: %s" % (time.perf_counter() - t0,
            {"%s/%d" % k: v[0] for k, v in tuned.items()}))
    tuned_b = None
    if args.tune_b:
        t0 = time.perf_counter()
        tuned_b = {"%s/%d" % k: v[0] for k, v in tune.tune_batch_size(items).items()}
        log("batch sizes tuned in %.1f s: divisors %s" % (time.perf_counter() - t0, tuned_b))
    ws = mb.batch_workspace(count)
    mb.mdp_batch_upload(items, ws)
    if args.profile_sweeps:
        # counter runs: two eager launches of exactly S and 3S sweeps of every MDP
        out = {"workload": "batch-512", "launches": [], "sources_hash": sources_hash("batch"),
               "algorithmic_bytes_per_sweep": float(total_bytes),
               "padded_bytes_per_sweep": float(padded_bytes)}
        for sweeps in (args.profile_sweeps, args.profile_sweeps, 3 * args.profile_sweeps):  # warm-up, S, 3S
            for it in items:
                it["V"].zero_()
            torch.cuda.synchronize()
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e0.record()
            mb.mdp_batch_launch(count, -1.0, sweeps, ws)
            e1.record()
            e1.synchronize()
            out["launches"].append({"sweeps": sweeps, "ms": e0.elapsed_time(e1)})
        print(json.dumps(out), flush=True)
        return
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            mb.mdp_batch_launch(count, tol, 1000000, ws)
    torch.cuda.current_stream().wait_stream(stream)

    def step():
        for it in items:
            it["V"].zero_()
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        graph.replay()
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1) / 1e3

    for _ in range(args.warmup):
        step()
    kernel_s = 0.0
    wall = 0.0
    for _ in range(args.steps):
        t0 = time.perf_counter()
        kernel_s += step()
        wall += time.perf_counter() - t0
    stats = mb.mdp_batch_read_stats(ws, count)
    if not all(st["converged"] for st in stats):
        raise RuntimeError("batch did not converge")
    backups = sum(st["sweeps"] * int(ns[i]) * m for i, st in enumerate(stats))
    bytes_step = sum(st["sweeps"] * int(ns[i]) * m * (2 * int(ns[i]) + 8)
                     for i, st in enumerate(stats))
    bytes_padded = sum(st["sweeps"] * int(ns[i]) * m * (2 * items[i]["ld"] + 8)
                       for i, st in enumerate(stats))
    gbps = bytes_step * args.steps / kernel_s / 1e9
    traffic = None
    vals = _traffic_file("batch-512")
    if vals.get("sources_hash") == sources_hash("batch"):
        try:
            # counters per padded byte moved (rows of whole 128-byte lines), scaled
            # to this solve's padded bytes
            per = float(vals.get("padded_bytes_per_sweep", vals["algorithmic_bytes_per_sweep"]))
            traffic = (float(vals["hbm_bytes_per_sweep"]) / per * bytes_padded
                       + float(vals["hbm_bytes_prologue"]))
        except (KeyError, ValueError):
            traffic = None
    sweeps = [st["sweeps"] for st in stats]
    log("batch: %d MDPs, sweeps %d..%d (mean %.0f), %.1f ms per solve of all"
        % (count, min(sweeps), max(sweeps), float(np.mean(sweeps)), kernel_s / args.steps * 1e3))
    # schedule of the last launch: how long the compute units were busy
    span = max(st["end_us"] for st in stats)
    busy = sum((st["end_us"] - st["start_us"]) * st["team"] for st in stats)
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    teams = [st["team"] for st in stats if st["team"] > 1]
    log("schedule: span %.1f ms, compute units busy %.0f%%, %d teams (%d workgroups)"
        % (span / 1e3, 100.0 * busy / (cus * span), len(teams), sum(teams)))
    for i in sorted(range(count), key=lambda i: -stats[i]["end_us"])[:6]:
        st = stats[i]
        log("  n=%d gamma=%.3f team=%d sweeps=%d: %.1f .. %.1f ms"
            % (ns[i], gammas[i], st["team"], st["sweeps"], st["start_us"] / 1e3,
               st["end_us"] / 1e3))
    cpu = None
    if not args.no_cpu_baseline:
        # the oracle's FP64 MB-VI sweeps on 4 MDPs of the same sizes, drawn on the
        # host with the same recipe and stored in BF16 by the oracle's quantiser
        import oracle
        from oracle import quantize as qz
        try:
            from threadpoolctl import threadpool_info
            cores = max((t.get("num_threads", 1) for t in threadpool_info()), default=1)
        except Exception:
            cores = 1
        mdps = []
        for i in range(4):
            n = int(ns[i])
            P, c = inputs.dense_mdp(n, m, 1.0, 600 + i, dtype=np.float32)
            q, sc = qz.quantize_rows(P.reshape(n * m, n), "bf16")
            mdps.append(oracle.DenseMDP(qz.dequantized(q, sc, "bf16").reshape(n, m, n), c,
                                        float(gammas[i])))
        Vs = [np.zeros(md.n) for md in mdps]
        done, sw, t0 = 0, 0, time.perf_counter()
        while time.perf_counter() - t0 < 10.0:
            for i, md in enumerate(mdps):
                Vs[i], _, _ = oracle.mb_sweep(md, Vs[i], (md.n + 7) // 8,
                                              oracle.sweep_permutation(md.n, 2000 + i, sw))
                done += md.n * m
            sw += 1
        dt = time.perf_counter() - t0
        cpu = {"value": done / dt, "unit": "backups/s", "cores": int(cores), "kind": "oracle",
               "sample": "%d FP64 sweeps of B_b on each of 4 MDPs of the workload's first sizes "
                         "(n = %s, m = %d, b = ceil(n/8), BF16 rows), %.1f s"
                         % (sw, ", ".join(str(int(x)) for x in ns[:4]), m, dt)}
    line = {
        "metric": METRIC, "value": backups * args.steps / wall, "unit": "backups/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f64", "cpu_baseline": cpu,
        "data": "synthetic", "replay_ms": kernel_s / args.steps * 1e3,
        "config": {"workload": "batch-512", "count": count, "n": "U[256, 4096]", "m": m,
                   "alpha": 1.0, "gamma": "U[0.9, 0.99]",
                   "b": "ceil(n / 8)" if tuned_b is None else "ceil(n / d), d tuned: %s" % tuned_b,
                   "storage": "bf16", "tol_dv": tol, "launch": "hipGraph replay",
                   "accumulate": "f64 (rows decoded exactly, FP64 FMA; a departure from the "
                                 "workload's FP32 accumulation)"},
        "hbm_gbps": gbps,
        "sweeps": {"min": min(sweeps), "max": max(sweeps), "mean": float(np.mean(sweeps))},
        "schedule": {"span_ms": span / 1e3, "cu_busy": busy / (cus * span),
                     "teams": len(teams), "team_workgroups": sum(teams)},
        "lanes": None if tuned is None else {"%s/%d" % k: v[0] for k, v in tuned.items()},
        "roofline": {"bound": "hbm", "achieved": gbps, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": gbps / HBM_PEAK_GBPS, "traffic": traffic,
                     "kernel": "batch_kernel (a workgroup or a team per MDP)",
                     "algorithmic_bytes_per_backup": "2 n + 8",
                     "padding_overhead": bytes_padded / bytes_step},
    }
    print(json.dumps(line), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    workloads = ["dense-8192x16", "csr-1M-banded", "csr-1M-uniform", "batch-512",
                 "multi-8192x16"]
    ap.add_argument("--workload", default="dense-8192x16",
                    help="one of %s (with --profile-sweeps, a comma-separated list of the "
                         "first three)" % ", ".join(workloads))
    ap.add_argument("--multi-r", type=int, default=32, choices=[16, 32, 48, 64],
                    help="multi-8192x16: number of cost vectors")
    ap.add_argument("--no-tune", action="store_true",
                    help="batch-512: keep the default lane-group widths")
    ap.add_argument("--tune-b", action="store_true",
                    help="batch-512: let the autotuner pick b = ceil(n / d) per size class "
                         "instead of the workload's ceil(n / 8)")
    ap.add_argument("--batch-sizes", default=None,
                    help="comma-separated batch sizes (default: the workload's)")
    ap.add_argument("--eps", type=float, default=1e-6)
    ap.add_argument("--precision", default="f32",
                    help="storage of the transition probabilities: f32, bf16 or fp8 (BF16 / "
                         "FP8 rows with one scale per row, quantised on the GPU; the solve "
                         "targets the stored MDP); with --profile-sweeps, a comma-separated list")
    ap.add_argument("--cpu-baseline-seconds", type=float, default=20.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-mpi", action="store_true")
    ap.add_argument("--copy-probe", action="store_true",
                    help="only run a plain 1 GiB device copy (counter calibration)")
    ap.add_argument("--profile-sweeps", type=int, default=0,
                    help="only run two vi_solve launches of exactly S and 3 S sweeps at the "
                         "first batch size (per-sweep counters: the difference of the two)")
    args = ap.parse_args()
    names = args.workload.split(",")
    if any(w not in workloads for w in names) or (len(names) > 1 and (
            not args.profile_sweeps or any(w in ("batch-512", "multi-8192x16") for w in names))):
        ap.error("--workload: %s" % args.workload)
    precs = args.precision.split(",")
    if any(p not in ("f32", "bf16", "fp8") for p in precs) or (
            len(precs) > 1 and not args.profile_sweeps):
        ap.error("--precision: %s" % args.precision)
    if args.gpus != 1:
        print("bench.py measures one GPU only: the mini-batch sweep is built and timed on a "
              "single MI355X (sharding over several GPUs is described, not implemented); "
              "run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2110_02901_amd import binding as mb
    from paper_2110_02901_amd import inputs

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    if args.copy_probe:
        # a plain copy kernel of known size: 1 GiB read + 1 GiB written per launch
        x = torch.ones(1 << 28, dtype=torch.float32, device=dev)
        y = torch.empty_like(x)
        for _ in range(3):
            y.copy_(x)
        torch.cuda.synchronize()
        # a second kernel of known bytes: a sum that reads the 1 GiB once
        tot = 0.0
        for _ in range(3):
            tot += float(x.sum())
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes_read": x.numel() * 4,
                          "copy_probe_bytes_written": y.numel() * 4, "launches": 3,
                          "sum_probe_bytes_read": x.numel() * 4, "sum_launches": 3,
                          "sum": tot}))
        return
    wl_name = args.workload
    if wl_name == "batch-512":
        run_batch(args, dev)
        return
    if wl_name == "multi-8192x16":
        run_multi(args, dev)
        return
    if args.profile_sweeps and len(names) * len(precs) > 1:
        # counter runs of several workloads / storages in one process (one
        # rocprofv3 run)
        for name in names:
            for prec in precs:
                run_single(argparse.Namespace(**dict(vars(args), precision=prec)), dev, name)
        return
    run_single(args, dev, wl_name)


def run_single(args, dev, wl_name):
    """One dense or sparse workload: the time-to-eps table, the timed steps
    and the JSON line (or, with --profile-sweeps, the counter launches)."""
    import torch
    from paper_2110_02901_amd import binding as mb
    from paper_2110_02901_amd import inputs

    wl = inputs.WORKLOADS[wl_name]
    n, m, gamma = wl["n"], wl["m"], wl["gamma"]
    seed = wl["perm_seed"]
    batch_sizes = ([int(x) for x in args.batch_sizes.split(",")] if args.batch_sizes
                   else list(wl["batch_sizes"]))
    dense = wl["kind"] == "dense"

    t0 = time.perf_counter()
    if dense:
        P, c = inputs.dense_mdp(n, m, wl["alpha"], wl["data_seed"], dtype=np.float32)
        nbytes = P.nbytes
        Pd = torch.from_numpy(P).to(dev)
        cd = torch.from_numpy(c).to(dev)
        h = mb.mdp_create_dense(Pd, cd, gamma)
        bytes_per_backup = 4 * n + 4  # one P row + its cost
    else:
        rp, col, val, c = inputs.csr_mdp(n, m, wl["k"], wl["alpha"], wl["data_seed"],
                                         band=wl["band"])
        nbytes = col.nbytes + val.nbytes
        dev_arrays = [torch.from_numpy(a).to(dev) for a in (rp, col, val, c)]
        h = mb.mdp_create_csr(*dev_arrays, gamma)
        bytes_per_backup = 8 * wl["k"] + 4  # k (column, weight) pairs + the cost
        if mb.mdp_engine(h, n) == "ell" and args.precision == "f32":
            # no band to stage: b = n runs on column-sorted blocks (a second
            # copy of the entries, built on the host; untimed set-up)
            t1 = time.perf_counter()
            dev_arrays.append(mb.mdp_column_blocks(h))
            log("column blocks built and attached in %.1f s (%.2f GB)"
                % (time.perf_counter() - t1, dev_arrays[-1].numel() * 4 / 1e9))
    log("generated and uploaded %s (%.2f GB) in %.1f s"
        % (wl_name, nbytes / 1e9, time.perf_counter() - t0))
    stream = torch.cuda.current_stream()
    h32 = h
    if args.precision != "f32":
        # BF16 / FP8 rows with one scale per row, quantised by the library
        t0 = time.perf_counter()
        vbytes = 2 if args.precision == "bf16" else 1
        rows = Pd.reshape(n * m, n) if dense else dev_arrays[2].reshape(n * m, wl["k"])
        codes, rscale = mb.mdp_quantize_rows(rows, args.precision)
        torch.cuda.synchronize()
        if dense:
            h = mb.mdp_create_dense_q(codes.reshape(-1), args.precision, rscale, cd, gamma)
            bytes_per_backup = vbytes * n + 8  # one row, its scale and its cost
        else:
            h = mb.mdp_create_csr_q(dev_arrays[0], dev_arrays[1], codes.reshape(-1),
                                    args.precision, rscale, dev_arrays[3], gamma)
            bytes_per_backup = (4 + vbytes) * wl["k"] + 8
        log("quantised to %s in %.1f s" % (args.precision, time.perf_counter() - t0))
    ws = mb.workspace(h, n)

    if args.profile_sweeps:
        # the batch size each workload's bench line selects, unless given
        b = batch_sizes[0] if args.batch_sizes else PROFILE_B.get(wl_name, batch_sizes[0])
        out = {"b": b, "engine": mb.mdp_engine(h, b), "launches": [],
               "algorithmic_bytes_per_sweep": n * m * bytes_per_backup,
               "sources_hash": sources_hash("solve")}
        # a warm-up launch of S sweeps, then the S and 3S launches whose
        # counter difference is the per-sweep traffic (same cache state before
        # each); each launch is one solve_kernel dispatch after one zero_kernel
        for sweeps in (args.profile_sweeps, args.profile_sweeps, 3 * args.profile_sweeps):
            V = torch.zeros(n, dtype=torch.float32, device=dev)
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            st = mb.vi_solve(h, V, b, seed, ws, tol_dv=-1.0, max_sweeps=sweeps)
            e1.record(stream)
            e1.synchronize()
            out["launches"].append({"sweeps": st["sweeps"], "recentrings": st["recentrings"],
                                    "ms": e0.elapsed_time(e1)})
        out["workload"] = wl_name
        out["precision"] = args.precision
        print(json.dumps(out), flush=True)
        return

    # Reference V* for the time-to-eps rule (not timed): MPI at b = n until
    # the policy is stable and the Bellman residual is <= 1e-11, returned in
    # FP64, so max|V_ref - J*| <= 1e-11 / (1 - gamma) <= 2e-9.  The parity
    # tests show separately that the solves reach the oracle's J* within eps.
    t0 = time.perf_counter()
    Vtmp = torch.zeros(n, dtype=torch.float32, device=dev)
    Vref = torch.zeros(n, dtype=torch.float64, device=dev)
    pol = torch.zeros(n, dtype=torch.int32, device=dev)
    st = mb.mpi_solve(h, Vtmp, pol, 20, n, 999, ws, policy_is_init=False, tol_dv=1e-11,
                      max_outer=2000, V64_out=Vref)
    if not st["converged"]:
        raise RuntimeError("reference solve did not converge: %s" % st)
    log("reference: %d sweeps, %d improvements, residual %.3g, %.1f s"
        % (st["sweeps"], st["outer_iters"], st["final_dv_inf"], time.perf_counter() - t0))
    if h32 is not h:
        # the FP32 MDP's own solution, for the error of the stored MDP's
        Vref32 = torch.zeros(n, dtype=torch.float64, device=dev)
        st = mb.mpi_solve(h32, Vtmp, pol, 20, n, 999, ws, policy_is_init=False, tol_dv=1e-11,
                          max_outer=2000, V64_out=Vref32)
        if not st["converged"]:
            raise RuntimeError("FP32 reference solve did not converge: %s" % st)
        lp_err = float((Vref - Vref32).abs().max())
        log("%s storage: max|J*(stored) - J*(FP32)| = %.3g" % (args.precision, lp_err))

    V = torch.zeros(n, dtype=torch.float32, device=dev)

    def timed_solve(b, mpi=False):
        V.zero_()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        if mpi:
            pol.zero_()
            s = mb.mpi_solve(h, V, pol, wl.get("K", 5), b, seed, ws, policy_is_init=False,
                             tol_dv=-1.0, eps=args.eps, V_ref=Vref, max_outer=4000)
        else:
            s = mb.vi_solve(h, V, b, seed, ws, tol_dv=-1.0, eps=args.eps, V_ref=Vref,
                            max_sweeps=20000)
        e1.record(stream)
        e1.synchronize()
        if not s["converged"]:
            raise RuntimeError("solve did not reach eps: %s" % s)
        return e0.elapsed_time(e1) / 1e3, s

    results = {}
    for b in batch_sizes:
        for _ in range(max(1, args.warmup)):
            timed_solve(b)
        secs, st = timed_solve(b)
        results[b] = (secs, st)
        log("VI b=%d: %d sweeps, %.1f ms to eps" % (b, st["sweeps"], secs * 1e3))
    best_b = min(batch_sizes, key=lambda b: results[b][0])

    mpi_res = {}
    if not args.no_mpi:
        for b in batch_sizes:
            timed_solve(b, mpi=True)
            secs, st = timed_solve(b, mpi=True)
            mpi_res[b] = (secs, st)
            log("MPI K=5 b=%d: %d sweeps, %d improvements, %.1f ms to eps"
                % (b, st["sweeps"], st["outer_iters"], secs * 1e3))

    # the timed steps
    for _ in range(args.warmup):
        timed_solve(best_b)
    torch.cuda.synchronize()
    t_wall = time.perf_counter()
    total_s = 0.0
    total_sweeps = 0
    for _ in range(args.steps):
        secs, st = timed_solve(best_b)
        total_s += secs
        total_sweeps += st["sweeps"]
    torch.cuda.synchronize()
    wall = time.perf_counter() - t_wall
    backups = total_sweeps * n * m
    value = backups / wall
    kernel_gbps = backups * bytes_per_backup / total_s / 1e9
    traffic = committed_traffic(wl_name if args.precision == "f32"
                                else "%s-%s" % (wl_name, args.precision),
                                best_b, total_sweeps / args.steps)
    engine = mb.mdp_engine(h, best_b)

    precision = None
    if h32 is not h:
        # The stored MDP's solve stops once its own certified distance to
        # J*(stored), gamma dV / (1 - gamma), is below the storage error
        # (measured above, untimed): sweeping further cannot bring V closer
        # to the FP32 MDP's J*.  The FP64 correction (mdp_refine, on the FP32
        # handle) then takes V to eps of J*(FP32): certified (its own stop
        # rule, no reference), by sweeps (K = 0) or by Algorithm 1 (K = 5),
        # and in measurement mode (first crossing of eps against the FP32
        # reference, the rule every other time here uses).
        tol_stored = lp_err * (1.0 - gamma) / gamma
        V64 = torch.zeros(n, dtype=torch.float64, device=dev)

        K_mpi = wl.get("K", 5)

        def lp_run(stored, K, certified):
            V.zero_()
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e2 = torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            if stored == "vi":
                s1 = mb.vi_solve(h, V, best_b, seed, ws, tol_dv=tol_stored, max_sweeps=20000,
                                 V64_out=V64)
            else:  # residual <= (1 - gamma) err  =>  max|V - J*(stored)| <= err
                pol.zero_()
                s1 = mb.mpi_solve(h, V, pol, K_mpi, best_b, seed, ws, policy_is_init=False,
                                  tol_dv=lp_err * (1.0 - gamma), max_outer=4000, V64_out=V64)
            e1.record(stream)
            s2 = mb.mdp_refine(h32, V64, best_b, seed, ws, K=K, eps=args.eps,
                               V_ref=None if certified else Vref32, first_sweep=s1["sweeps"],
                               max_iters=20000)
            e2.record(stream)
            e2.synchronize()
            err = float((V64 - Vref32).abs().max())
            out = {"stored_solve": {"solver": stored, "sweeps": s1["sweeps"],
                                    "improvements": s1["outer_iters"],
                                    "ms": e0.elapsed_time(e1)},
                   "fp64_correction": {"K": K, "sweeps": s2["sweeps"],
                                       "improvements": s2["outer_iters"],
                                       "residual_in": s2["residual_in"],
                                       "residual_out": s2["residual_out"],
                                       "certified_bound": s2["bound_out"],
                                       "ms": e1.elapsed_time(e2),
                                       "converged": bool(s2["converged"])},
                   "total_ms": e0.elapsed_time(e2),
                   "err_vs_f32_reference": err}
            log("%s %s + FP64 correction K=%d (%s): stored %d sweeps %.1f ms, correction %d "
                "sweeps %d improvements %.1f ms (residual in %.3g, bound %.3g), total %.1f ms, "
                "max|V - J*(FP32)| = %.3g"
                % (args.precision, stored, K,
                   "certified" if certified else "to eps of the reference",
                   s1["sweeps"], e0.elapsed_time(e1), s2["sweeps"], s2["outer_iters"],
                   e1.elapsed_time(e2), s2["residual_in"], s2["bound_out"], e0.elapsed_time(e2),
                   err))
            return out

        runs = {}
        for stored, K, certified in (("vi", 0, True), ("vi", K_mpi, True), ("mpi", K_mpi, True),
                                     ("vi", 0, False), ("mpi", K_mpi, False)):
            lp_run(stored, K, certified)  # warm-up
            runs["%s_k%d_%s" % (stored, K, "certified" if certified else "measured")] = \
                lp_run(stored, K, certified)
        f32 = {}
        for solver in ("vi", "mpi"):
            for _ in range(2):  # warm-up, then timed
                e3 = torch.cuda.Event(enable_timing=True)
                e4 = torch.cuda.Event(enable_timing=True)
                V.zero_()
                pol.zero_()
                e3.record(stream)
                if solver == "vi":
                    s3 = mb.vi_solve(h32, V, best_b, seed, ws, tol_dv=-1.0, eps=args.eps,
                                     V_ref=Vref32, max_sweeps=20000)
                else:
                    s3 = mb.mpi_solve(h32, V, pol, K_mpi, best_b, seed, ws, policy_is_init=False,
                                      tol_dv=-1.0, eps=args.eps, V_ref=Vref32, max_outer=4000)
                e4.record(stream)
                e4.synchronize()
            f32[solver] = {"sweeps": s3["sweeps"], "improvements": s3["outer_iters"],
                           "ms": e3.elapsed_time(e4),
                           "rule": "first sweep with max|V - J*(FP32)| <= eps"}
            log("FP32 alone (%s): %d sweeps %.1f ms" % (solver, s3["sweeps"], f32[solver]["ms"]))
        best_lp = min(runs, key=lambda k: runs[k]["total_ms"] if k.endswith("measured") else 1e30)
        best_cert = min(runs, key=lambda k: runs[k]["total_ms"] if k.endswith("certified")
                        else 1e30)
        best_f32 = min(f32, key=lambda k: f32[k]["ms"])
        precision = {
            "storage": args.precision,
            "err_stored_vs_f32_solution": lp_err,
            "stored_solve_stop": "certified max|V - J*(stored)| <= err_stored_vs_f32_solution",
            "stored_then_fp64_correction": runs,
            "f32_alone": f32,
            "equal_accuracy": {"eps": args.eps, "best_stored_then_correction": best_lp,
                               "ms": runs[best_lp]["total_ms"], "best_f32_alone": best_f32,
                               "f32_ms": f32[best_f32]["ms"],
                               "speedup": f32[best_f32]["ms"] / runs[best_lp]["total_ms"]},
            "best_certified": {"run": best_cert, "ms": runs[best_cert]["total_ms"],
                               "bound": runs[best_cert]["fp64_correction"]["certified_bound"]},
        }

    line = {
        "metric": METRIC,
        "value": value,
        "unit": "backups/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",  # arithmetic; the storage of P is config.storage
        "data": "synthetic",
        "config": dict({"workload": wl_name, "n": n, "m": m, "alpha": wl["alpha"],
                        "gamma": gamma, "solver": "vi", "b": best_b, "eps": args.eps,
                        "perm_seed": seed, "data_seed": wl["data_seed"],
                        "storage": args.precision},
                       **({} if dense else {"k": wl["k"], "band": wl["band"]})),
        "hbm_gbps": kernel_gbps,
        "time_to_eps": {
            "vi": {str(b): {"ms": results[b][0] * 1e3, "sweeps": results[b][1]["sweeps"]}
                   for b in batch_sizes},
            "mpi_k5": {str(b): {"ms": mpi_res[b][0] * 1e3, "sweeps": mpi_res[b][1]["sweeps"],
                                "improvements": mpi_res[b][1]["outer_iters"]}
                       for b in mpi_res},
            "plain_form_b": n,
            "chosen_b": best_b,
        },
        "roofline": {
            "bound": "hbm",
            "achieved": kernel_gbps,
            "peak": HBM_PEAK_GBPS,
            "unit": "GB/s",
            "frac": kernel_gbps / HBM_PEAK_GBPS,
            "traffic": traffic,
            "kernel": ("resident_kernel, VI (one launch per solve)" if dense and n <= 16384 else
                       "solve_kernel, %s engine, VI (one launch per solve)" % engine),
            "algorithmic_bytes_per_backup": bytes_per_backup,
        },
    }
    if precision:
        line["precision"] = precision
    if not args.no_cpu_baseline:
        log("timing the CPU oracle (~%.0f s)" % args.cpu_baseline_seconds)
        import oracle
        mdp = (oracle.DenseMDP(P, c, gamma) if dense
               else oracle.CsrMDP(rp, col, val, c, gamma))
        line["cpu_baseline"] = cpu_baseline(mdp, wl_name, best_b, seed,
                                            args.cpu_baseline_seconds,
                                            gpu_sweeps=results[best_b][1]["sweeps"],
                                            eps=args.eps)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
