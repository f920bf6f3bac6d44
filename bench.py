#!/usr/bin/env python3
"""SpMM benchmark on one MI355X: C = A.B through sd_plan / sd_spmm.

One step is one pass of the workload's SpMMs (one product for most
workloads; the four products A.X, A.H, A^T.G64, A^T.G128 for ``gcn``) on
inputs already resident in HBM.  Plan construction (validation, analysis,
conversion, upload) is one-time preprocessing, timed separately and reported
under ``preprocess_s``, as in the paper's protocol, which excludes it from
kernel time.  To keep the 256 MiB Infinity Cache from serving a step's dense
operands out of earlier steps, steps rotate over R >= 2 independent (B, C)
buffer sets whose B operands alone add up to at least twice that cache (C is
written with non-temporal stores, which do not displace cached B rows, so
only the bytes read count towards flushing it).

Output: one JSON line (see the keys below).  ``value`` is whole-job GFLOP/s
= 2 nnz N (summed over the step's products) / step time.
"""
from __future__ import annotations

import argparse
import dataclasses
import glob
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0          # MI355X HBM3E
FP32_MFMA_PEAK_TFLOPS = 157.3   # MI355X dense fp32 matrix
MALL_BYTES = 256 << 20

WORKLOAD_LABEL = {
    "uniform": "uniform 1024x1024, 8 nnz/row, N=32",
    "laplace": "7-point Laplacian 64^3 (262144 rows, Dirichlet), N=64",
    "rmat20": "R-MAT 2^20 vertices, 16Mi edges, GCN-normalised, N=128",
    "block16": "131072^2 from 16x16 blocks, 32/block-row, 90% fill, N=64",
    "gcn": "GCN SpMMs on R-MAT 2.4M vertices / 62M edges: A.X128 + A.H64 + A^T.G64 + A^T.G128",
}


def kernel_source_sha() -> str:
    h = hashlib.sha256()
    # the kernels and their launchers, and the plan rules that pick the kernel
    # and its launch parameters
    for f in ("kernels.hip", "runtime.hip", "host_plan.cpp"):
        with open(os.path.join(ROOT, "paper_2608_05033_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def stored_traffic(workload: str, kernel: str, sha: str):
    """HBM bytes per launch from committed rocprofv3 counter summaries, only if
    they were taken on the current kernel sources."""
    path = os.path.join(ROOT, "profiles", f"{kernel}_{workload}.txt")
    if not os.path.exists(path):
        return None
    kv = {}
    with open(path) as f:
        for line in f:
            if ":" in line and not line.lstrip().startswith("#"):
                key, val = line.split(":", 1)
                kv[key.strip()] = val.strip()
    if kv.get("source_sha") != sha:
        return None
    try:
        return float(kv["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def _cpu_model() -> str:
    """The first CPU's model name, with its family / model / stepping numbers
    (a virtualised host may report only a generic name)."""
    info = {}
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if not line.strip():
                    break  # the first CPU's block only
                if ":" in line:
                    key, val = line.split(":", 1)
                    info.setdefault(key.strip(), val.strip())
    except OSError:
        pass
    name = info.get("model name", "unknown")
    ids = [f"{k} {info[k]}" for k in ("cpu family", "model", "stepping") if k in info]
    return f"{name} ({', '.join(ids)})" if ids else name


def _gpu_clocks() -> dict:
    """DPM clock levels of the first GPU from sysfs (the levels rocm-smi shows);
    the current level carries a '*'.  Read right after the timed region, while
    the GPU is still at its working clock."""
    out = {}
    cards = sorted(glob.glob("/sys/class/drm/card*/device/pp_dpm_sclk"))
    if not cards:
        return out
    dev = os.path.dirname(cards[0])
    for clk in ("sclk", "mclk"):
        try:
            with open(os.path.join(dev, f"pp_dpm_{clk}")) as f:
                levels = [ln.strip() for ln in f if ln.strip()]
        except OSError:
            continue
        cur = [ln for ln in levels if ln.endswith("*")]
        out[clk] = cur[0].rstrip(" *") if cur else None
        out[f"{clk}_levels"] = [ln.rstrip(" *") for ln in levels]
    return out


def _cpu_ranges(cpus) -> str:
    """Affinity set as compact ranges, e.g. "0-15,32-47"."""
    cpus = sorted(cpus)
    out, i = [], 0
    while i < len(cpus):
        j = i
        while j + 1 < len(cpus) and cpus[j + 1] == cpus[j] + 1:
            j += 1
        out.append(str(cpus[i]) if i == j else f"{cpus[i]}-{cpus[j]}")
        i = j + 1
    return ",".join(out)


def _oracle_rows(oracle, src, B, rows, bufs):
    """One timed oracle pass over `rows` into preallocated outputs."""
    t0 = time.perf_counter()
    oracle.spmm_rows(src, B, rows, out=bufs)
    return time.perf_counter() - t0


def cpu_baseline(A, products, dense, budget_s: float):
    """The fp64 oracle on the host cores, on a bounded sample of the same
    workload: every row when one pass fits the budget (then repeated to fill
    it), else an evenly strided row sample sized to the budget.  Outputs are
    allocated once, outside the timed passes.  The oracle computes C and the
    bound S = |A||B| together (4N fp64 flops per nonzero); the figure counts
    the metric's 2N per nonzero, so it is the oracle's time to the product.
    Also reported: the oracle on one thread over the whole uniform (1024^2,
    8 per row, N = 32) and Laplacian (64^3, N = 64) matrices, 1 warm-up and 3
    timed passes, median."""
    import numpy as np

    import gen
    import oracle

    affinity = os.sched_getaffinity(0)
    threads = oracle.threads(0)
    rng = np.random.default_rng(0)
    share = budget_s / len(products)
    flops = 0.0
    elapsed = 0.0
    samples = []
    for pi, prod in enumerate(products):
        src = dense["AT"] if prod.transpose else A
        lens = np.diff(src.rowptr.astype(np.int64))
        probe = np.sort(rng.choice(src.m, size=min(src.m, 4096), replace=False)).astype(np.int32)
        bufs = (np.empty(probe.size * prod.n), np.empty(probe.size * prod.n))
        per_nnz_s = max(_oracle_rows(oracle, src, dense[pi], probe, bufs), 1e-6) / max(1, int(lens[probe].sum()))
        want_nnz = share / per_nnz_s
        if want_nnz >= src.nnz:
            rows = np.arange(src.m, dtype=np.int32)
            what = f"all {src.m} rows"
        else:
            stride = max(1, int(np.ceil(src.nnz / want_nnz)))
            rows = np.arange(0, src.m, stride, dtype=np.int32)
            what = f"every {stride}th row ({rows.size} rows)"
        bufs = (np.empty(rows.size * prod.n), np.empty(rows.size * prod.n))
        # repeat the sample until this product's share of the budget is spent
        reps, spent = 0, 0.0
        while reps == 0 or (spent < share and reps < 100000):
            spent += _oracle_rows(oracle, src, dense[pi], rows, bufs)
            reps += 1
        elapsed += spent
        flops += 2.0 * float(lens[rows].sum()) * prod.n * reps
        samples.append(f"product {pi} (N={prod.n}{', A^T' if prod.transpose else ''}): {what} x{reps}")
        del bufs
    single = {}
    oracle.threads(1)
    try:
        for name, mat, n in (("uniform", gen.uniform_rows(1024, 1024, 8, 0), 32),
                             ("laplace", gen.laplacian3d(64), 64)):
            B = gen.dense_uniform(mat.k, n, seed=0)
            rows = np.arange(mat.m, dtype=np.int32)
            bufs = (np.empty(mat.m * n), np.empty(mat.m * n))
            _oracle_rows(oracle, mat, B, rows, bufs)
            t = float(np.median([_oracle_rows(oracle, mat, B, rows, bufs) for _ in range(3)]))
            single[name] = {"gflops": round(2.0 * mat.nnz * n / t / 1e9, 3), "ms": round(t * 1e3, 3)}
    finally:
        oracle.threads(threads)
    return {"value": round(flops / elapsed / 1e9, 3), "unit": "GFLOP/s", "cores": threads, "kind": "oracle",
            "sample": "; ".join(samples) + f"; {elapsed:.1f} s",
            "arithmetic": "fp64; C and the bound |A||B| together (4N flops per nonzero), credited 2N per nonzero",
            "cpu_model": _cpu_model(), "affinity": _cpu_ranges(affinity), "host_cpus": os.cpu_count(),
            "single_thread": single}


def gcn_training(A, epochs: int, dev, warmup: int = 10, in_feats: int = 128, hidden: int = 128,
                 classes: int = 64):
    """Full-batch training of the two-layer GCN (aggregations through sd_spmm at
    widths `hidden` and `classes`, forward and transposed), timed per epoch
    after `warmup` epochs.  Synthetic features N(0,1) and labels from a fixed
    random teacher GCN."""
    import torch

    import gen
    from paper_2608_05033_amd import gcn

    t0 = time.perf_counter()
    X = torch.from_numpy(gen.dense_normal(A.m, in_feats, seed=0, stream=9)).to(dev)
    teacher = gcn.GCN2(A, in_feats, hidden, classes, device=dev, seed=99)
    with torch.no_grad():
        labels = teacher(X).argmax(dim=1)
    teacher.agg.destroy()
    model = gcn.GCN2(A, in_feats, hidden, classes, device=dev, seed=1)
    opt = torch.optim.Adam(model.parameters(), lr=0.01)
    setup_s = time.perf_counter() - t0
    losses = [gcn.train_epoch(model, X, labels, opt) for _ in range(warmup)]
    torch.cuda.synchronize(dev)
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(epochs):
        losses.append(gcn.train_epoch(model, X, labels, opt))
    end.record()
    torch.cuda.synchronize(dev)
    epoch_ms = start.elapsed_time(end) / epochs
    model.agg.destroy()
    return {"epochs": epochs, "warmup_epochs": warmup, "epoch_ms": round(epoch_ms, 3),
            "in_feats": in_feats, "hidden": hidden, "classes": classes,
            "spmm_per_epoch": 4, "loss_first": round(losses[0].item(), 5), "loss_last": round(losses[-1].item(), 5),
            "setup_s": round(setup_s, 2)}


def main():
    ap = argparse.ArgumentParser(description=__doc__.splitlines()[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="gcn", choices=sorted(WORKLOAD_LABEL))
    ap.add_argument("--family", default="auto")
    ap.add_argument("--engine", default="auto")
    ap.add_argument("--heavy-threshold", type=int, default=0)
    ap.add_argument("--chunk-nnz", type=int, default=0)
    ap.add_argument("--units", type=int, default=0)
    ap.add_argument("--row-slices", type=int, default=0, help="lane groups sharing a row (0 = planner default)")
    ap.add_argument("--col-tile", type=int, default=0, help="dense columns per column pass (0 = planner default)")
    ap.add_argument("--light-order", default="auto", choices=["auto", "ascending", "last_col"],
                    help="heavy split: order of the light rows")
    ap.add_argument("--chunk-order", default="auto", choices=["auto", "list", "mid_col"],
                    help="heavy split: order of the heavy rows' chunks")
    ap.add_argument("--wg-order", type=int, default=0, help="workgroup order over the XCDs (0 = planner default)")
    ap.add_argument("--window-rows", type=int, default=0, help="packed column windows: light rows per window")
    ap.add_argument("--rotate", type=int, default=0, help="buffer sets to rotate over (0 = auto)")
    ap.add_argument("--settle-ms", type=float, default=100.0,
                    help="untimed steps run before the warm-up until this much wall time has passed")
    ap.add_argument("--n", type=int, default=0, metavar="N",
                    help="dense width of every product instead of the workload's own (0 = the workload's)")
    ap.add_argument("--search", action="store_true", help="measured plan selection instead of the rules")
    ap.add_argument("--cpu-seconds", type=float, default=10.0, help="oracle budget; 0 disables")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="MIB",
                    help="first run 10 plain device copies of MIB MiB (reference for rocprofv3 byte counters)")
    ap.add_argument("--gcn-train-epochs", type=int, default=0, metavar="E",
                    help="gcn workload: also time E full-batch training epochs of the two-layer GCN "
                         "(after 10 warmup epochs) and report them under gcn_training")
    args = ap.parse_args()
    if args.gcn_train_epochs and args.workload != "gcn":
        ap.error("--gcn-train-epochs needs --workload gcn")

    if args.gpus != 1:
        print(f"bench.py: the library runs on one GPU; --gpus {args.gpus} is not supported "
              "(sharding rows across GPUs is a design, not built)", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import gen
    import paper_2608_05033_amd as sd

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    dev = torch.device("cuda:0")
    if args.calibrate_copy > 0:
        src = torch.ones(args.calibrate_copy << 18, device=dev)
        dst = torch.empty_like(src)
        for _ in range(10):
            dst.copy_(src)
        torch.cuda.synchronize(dev)
        print(f"# calibration: 10 device copies of {args.calibrate_copy} MiB", file=sys.stderr, flush=True)
        del src, dst
    wl = gen.WORKLOADS[args.workload]
    if args.n < 0:
        raise SystemExit("bench.py: --n must be positive")
    products = [dataclasses.replace(p, n=args.n) for p in wl.products] if args.n else list(wl.products)
    t0 = time.perf_counter()
    A = wl.matrix(seed=0)
    gen_s = time.perf_counter() - t0
    print(f"# workload {args.workload}: m={A.m} k={A.k} nnz={A.nnz} (generated in {gen_s:.1f} s)",
          file=sys.stderr, flush=True)

    # ---- plans (one-time preprocessing)
    plan_opts = dict(force=args.family, engine=args.engine, heavy_threshold=args.heavy_threshold,
                     chunk_nnz=args.chunk_nnz, units=args.units, search=args.search, row_slices=args.row_slices,
                     col_tile=args.col_tile, light_order=args.light_order, chunk_order=args.chunk_order,
                     wg_order=args.wg_order, window_rows=args.window_rows)
    plans, dense_host = [], {}
    t0 = time.perf_counter()
    for pi, prod in enumerate(products):
        plans.append(sd.sd_plan_ex(A, prod.n, transpose=prod.transpose, **plan_opts))
    plan_s = time.perf_counter() - t0
    t0 = time.perf_counter()
    stats = sd.sd_analyze(A)
    analyze_s = time.perf_counter() - t0
    # the same analysis on a device copy of A (HIP kernels; identical statistics)
    dev_csr = [torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in (A.rowptr, A.colidx, A.values)]
    sd.sd_analyze_device(*dev_csr, A.m, A.k, A.nnz)  # first call loads the kernels
    t0 = time.perf_counter()
    dstats = sd.sd_analyze_device(*dev_csr, A.m, A.k, A.nnz)
    analyze_dev_s = time.perf_counter() - t0
    if dstats["nnzb16"] != stats["nnzb16"] or dstats["row_cv"] != stats["row_cv"]:
        raise RuntimeError("device analysis disagrees with the host analysis")
    # the same plans built from the device copy (converted on the device where
    # the family allows); they must equal the host-built plans
    t0 = time.perf_counter()
    dplans = [sd.sd_plan_device(*dev_csr, A.m, A.k, A.nnz, prod.n, stream=torch.cuda.current_stream(),
                                transpose=prod.transpose, **plan_opts)
              for prod in products]
    plan_dev_s = time.perf_counter() - t0
    plan_dev_built = [p.info["device_built"] for p in dplans]
    for hp, dp in zip(plans, dplans):
        same = {k: v for k, v in hp.info.items() if k != "device_built"} == \
            {k: v for k, v in dp.info.items() if k != "device_built"}
        dp.destroy()
        if not same and not args.search:
            raise RuntimeError("device-built plan disagrees with the host-built plan")
    del dev_csr
    for pi, prod in enumerate(products):
        rows_in = A.m if prod.transpose else A.k
        dense_host[pi] = prod.dense(rows_in, seed=0)
    print(f"# plans: {[p.family for p in plans]} in {plan_s:.2f} s", file=sys.stderr, flush=True)

    # ---- device buffers, rotated so a step's B is not served by the MALL
    read_bytes = sum(4 * p.info["k"] * p.info["n"] for p in plans)
    R = args.rotate or max(2, min(64, -(-2 * MALL_BYTES // max(1, read_bytes))))
    bufs = []
    for r in range(R):
        one = []
        for pi, p in enumerate(plans):
            Bd = torch.from_numpy(dense_host[pi]).to(dev)
            Cd = torch.empty((p.info["m"], p.info["n"]), dtype=torch.float32, device=dev)
            one.append((Bd, Cd))
        bufs.append(one)
    stream = torch.cuda.Stream(device=dev)
    torch.cuda.synchronize(dev)

    def step(i):
        for pi, p in enumerate(plans):
            Bd, Cd = bufs[i % R][pi]
            sd.sd_spmm(p, Bd, Cd, stream)

    # Clock settle (untimed): from idle the GPU takes some milliseconds of load
    # to reach its working clock, so a few short warm-up steps still leave the
    # first timed steps slow (block16: 122 against 110 us per step after 10
    # against 300 warm-up steps).  Steps are repeated until about 100 ms of
    # work has run, then come the W warm-up steps and the K timed steps.
    settle_steps, settle0 = 0, time.perf_counter()
    while time.perf_counter() - settle0 < args.settle_ms / 1e3 and settle_steps < 20000:
        for _ in range(8):
            step(settle_steps)
            settle_steps += 1
        torch.cuda.synchronize(dev)
    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize(dev)

    # ---- timed region: K whole steps back to back, HIP events on the launch stream
    K = args.steps
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize(dev)
    wall0 = time.perf_counter()
    start.record(stream)
    for i in range(K):
        step(i)
    end.record(stream)
    torch.cuda.synchronize(dev)
    wall = time.perf_counter() - wall0
    clocks = _gpu_clocks()
    total_ms = start.elapsed_time(end)
    ms_per_step = total_ms / K

    # ---- per-product launch duration: each product alone, back to back, same stream
    launch_ms = []
    for pi, p in enumerate(plans):
        # launch-bound steps (the 8,192-nonzero matrix) are averaged over 1,000 back-to-back calls
        reps = 1000 if ms_per_step < 0.05 else max(10, min(K, 200))
        for i in range(3):
            Bd, Cd = bufs[i % R][pi]
            sd.sd_spmm(p, Bd, Cd, stream)
        s0, s1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s0.record(stream)
        for i in range(reps):
            Bd, Cd = bufs[i % R][pi]
            sd.sd_spmm(p, Bd, Cd, stream)
        s1.record(stream)
        torch.cuda.synchronize(dev)
        launch_ms.append(s0.elapsed_time(s1) / reps)

    # ---- secondary figures (outside the timed region): the median of singly
    # timed steps, the step with one buffer set (B warm in L2 and the
    # Infinity Cache), and a device copy's rate on this machine for reference
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(min(K, 200))]
    for i, (e0, e1) in enumerate(ev):
        e0.record(stream)
        step(i)
        e1.record(stream)
    torch.cuda.synchronize(dev)
    median_ms = float(np.median([e0.elapsed_time(e1) for e0, e1 in ev]))
    warm_reps = max(10, min(K, 200))
    for i in range(3):
        step(0)
    w0, w1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    w0.record(stream)
    for i in range(warm_reps):
        step(0)
    w1.record(stream)
    torch.cuda.synchronize(dev)
    warm_ms = w0.elapsed_time(w1) / warm_reps
    # (not in counter runs: their --calibrate-copy copies must be the only ones)
    copy_gbps = None
    if args.calibrate_copy == 0:
        copy_bytes = 512 << 20
        csrc = torch.ones(copy_bytes // 4, device=dev)
        cdst = torch.empty_like(csrc)
        with torch.cuda.stream(stream):
            for _ in range(2):
                cdst.copy_(csrc)
            c0, c1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            c0.record(stream)
            for _ in range(10):
                cdst.copy_(csrc)
            c1.record(stream)
        torch.cuda.synchronize(dev)
        copy_gbps = 2 * copy_bytes * 10 / (c0.elapsed_time(c1) / 1e3) / 1e9
        del csrc, cdst

    flops = sum(2.0 * p.info["nnz"] * p.info["n"] for p in plans)
    compulsory = sum(p.info["compulsory_bytes"] for p in plans)
    value = flops / (ms_per_step / 1e3) / 1e9
    hbm_gbps = compulsory / (ms_per_step / 1e3) / 1e9

    # dominant launch: the product with the largest per-launch time
    dom = int(np.argmax(launch_ms))
    dp = plans[dom]
    fam = dp.family
    # the ELL launch takes the pipelined kernel when a row fits one entry load per lane
    ell_kernel = "k_ell_pipe" if dp.info["ell_width"] <= dp.info["lanes_per_row"] else "k_ell_rows"
    # narrow widths (at most 8 lanes cover a dense row) take the sliced row kernels
    lanes = dp.info["lanes_per_row"] // max(1, dp.info["row_slices"])
    row_kernel = "k_csr_slices" if dp.info["row_slices"] > 1 else "k_csr_rows"
    split_kernel = "k_split_slices" if lanes <= 8 else "k_csr_split"
    kernel = {"csr_row": row_kernel, "csr_split": split_kernel, "csr_merge": "k_csr_merge", "ell": ell_kernel,
              "win": "k_win_split", "sell": "k_sell_rows",
              "bsr": "k_bsr_mfma" if dp.info["engine"] == 1 else "k_bsr_valu",
              "bell": "k_bsr_mfma" if dp.info["engine"] == 1 else "k_bsr_valu"}[fam]
    sha = kernel_source_sha()
    dom_s = launch_ms[dom] / 1e3
    if fam in ("bsr", "bell") and dp.info["engine"] == 1:
        slots = dp.info["nnzb"] if fam == "bsr" else dp.info["bell_width"] * dp.info["block_rows"]
        dense_flops = 2.0 * 256 * slots * dp.info["n"]
        roof = {"bound": "mfma", "achieved": round(dense_flops / dom_s / 1e12, 3), "peak": FP32_MFMA_PEAK_TFLOPS,
                "unit": "TFLOP/s"}
        roof["frac"] = round(roof["achieved"] / roof["peak"], 4)
        roof["hbm_gbps_on_compulsory"] = round(dp.info["compulsory_bytes"] / dom_s / 1e9, 1)
    else:
        roof = {"bound": "hbm", "achieved": round(dp.info["compulsory_bytes"] / dom_s / 1e9, 1),
                "peak": HBM_PEAK_GBPS, "unit": "GB/s"}
        roof["frac"] = round(roof["achieved"] / roof["peak"], 4)
    # counter summaries are taken at the workload's own widths
    traffic = stored_traffic(args.workload, kernel, sha) if not args.n else None
    roof["traffic"] = traffic
    roof["kernel"] = kernel
    roof["kernel_source_sha"] = sha
    roof["launch_ms"] = round(launch_ms[dom], 5)
    roof["algorithmic_bytes_per_launch"] = dp.info["compulsory_bytes"]

    cpu = None
    if args.cpu_seconds > 0:
        dense_cpu = dict(dense_host)
        if any(p.transpose for p in products):
            import oracle
            tr, tc, tv = oracle.transpose(A)
            dense_cpu["AT"] = gen.CSR(A.k, A.m, tr, tc, tv)
        cpu = cpu_baseline(A, products, dense_cpu, args.cpu_seconds)

    out = {
        "metric": "SpMM GFLOP/s (2*nnz*N/t) and achieved HBM GB/s vs peak, 1xMI355X",
        "value": round(value, 2),
        "unit": "GFLOP/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 5),
        "settle_steps": settle_steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": args.workload,
            "description": WORKLOAD_LABEL[args.workload] + (f"; every product at N={args.n}" if args.n else ""),
            "m": A.m, "k": A.k, "nnz": A.nnz,
            "products": [{"n": p.info["n"], "transpose": bool(p.info["transpose"]), "family": p.family,
                          "launch_ms": round(launch_ms[i], 5)} for i, p in enumerate(plans)],
            "rotated_buffer_sets": R,
            "plan_selection": "measured" if args.search else "rules",
        },
        "hbm_gbps_compulsory": round(hbm_gbps, 1),
        "hbm_frac_compulsory": round(hbm_gbps / HBM_PEAK_GBPS, 4),
        "ms_per_step_median": round(median_ms, 5),
        "ms_per_step_warm": round(warm_ms, 5),
        "device_copy_gbps": round(copy_gbps, 1) if copy_gbps else None,
        "gpu_clocks": clocks,
        "frac_of_device_copy": round(hbm_gbps / copy_gbps, 4) if copy_gbps else None,
        "compulsory_bytes_per_step": compulsory,
        "wall_s_timed": round(wall, 4),
        "roofline": roof,
        "cpu_baseline": cpu,
        "preprocess_s": {"generate": round(gen_s, 3), "plan_all": round(plan_s, 3), "analyze": round(analyze_s, 3),
                         "analyze_device": round(analyze_dev_s, 4), "plan_device_all": round(plan_dev_s, 4),
                         "plan_device_built": plan_dev_built},
        "shape_class": stats["shape_class"],
    }
    if args.gcn_train_epochs > 0:
        for p in plans:  # free the SpMM-only plans and buffers before training
            p.destroy()
        plans = []
        del bufs
        torch.cuda.empty_cache()
        out["gcn_training"] = gcn_training(A, args.gcn_train_epochs, dev)
    print(json.dumps(out), flush=True)
    for p in plans:
        p.destroy()


if __name__ == "__main__":
    main()
