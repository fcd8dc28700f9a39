"""Benchmark of the sparse embedding step on one MI355X.

One step = lookup_pool_fwd (dedup, IDMap find-or-insert with row init, fused
gather + pool) + lookup_pool_bwd_opt (per-unique gradient sums fused with the
row-sparse optimizer) over one batch of synthetic input already resident in
HBM.  Default workload: the growing dynamic table -- 200 features (150
single-hot, 50 multi-hot with Poisson(10) bags) in one hash table that starts
at 2e7 live ids and takes 3e5 never-seen ids per step, dim 64 fp32 rows with
Adam state, batch 32768, sum pooling; the IDMap is resized inside the run.

Prints ONE JSON line (rank 0, N = 1):
  value       = ID occurrences per second over the timed steps (whole job)
  gbps        = algorithmic bytes per step / step time (rows of duplicate ids
                counted once); hbm_frac = gbps / 8 TB/s, frac_of_copy = gbps /
                a 1 GiB device copy (the library's copy probe) timed in the
                same run
  gbps_effective_occ = the same with every occurrence's row counted (B_occ):
                an effective bandwidth, not HBM traffic
  roofline    = the dominant kernel's algorithmic bytes (the step's byte terms
                that kernel moves) / its HIP-event time
  cpu_baseline= the CPU oracle timed on a bounded sample of the same workload
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# where the profile converters write their summaries (and the bench reads
# the traffic records back)
PROFILES = os.path.join(ROOT, "profiles")
OPTIMIZERS = ["adagrad", "adam", "adamw", "adam-eps-hat", "adagrad-rowwise", "adam-rowwise"]
METRIC = "embedding step IDs/sec (fwd+bwd+opt) and achieved HBM GB/s vs peak, 1 MI355X"
HBM_PEAK_GBPS = 8000.0


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None,
                    help="timed steps (default: 100 for the growing table, whose run includes resizes, and "
                         "for --op ids-partition; 200 for --op bucketize | mod; else 20)")
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", type=int, default=4)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=10.0, help="target CPU time of the oracle sample")
    ap.add_argument("--unfused", action="store_true", help="lookup_pool_bwd + sparse_opt_step instead of the fused call")
    ap.add_argument("--no-step-events", action="store_true",
                    help="no timing event at the step boundaries (no per-step times, no median)")
    ap.add_argument("--pipelined", action="store_true",
                    help="run the next batch's lookup_prepare on a second stream while the current batch pools and "
                         "runs its backward (default: one stream)")
    ap.add_argument("--optimizer", choices=OPTIMIZERS, default=None,
                    help="run the workload with another row-sparse optimizer (adamw: weight decay 0.01)")
    ap.add_argument("--gen-workers", type=int, default=16,
                    help="processes drawing the input batches before the GPU is touched (1: in-process, e.g. under "
                         "a profiler)")
    ap.add_argument("--evictable", action="store_true",
                    help="create the table with eviction (each row keeps its key and last-lookup clock)")
    ap.add_argument("--evict-age", type=int, default=-1,
                    help="after the timed steps, time one ht_evict(max_age) on the table (implies --evictable)")
    ap.add_argument("--op", choices=["step", "ids-partition", "bucketize", "mod"], default="step",
                    help="ids-partition: time the fused dedup + owner split alone on its one-million-id input; "
                         "bucketize / mod: the fused feature transforms on 100 columns of 10,000 values")
    ap.add_argument("--shards", type=int, default=None, help="owner shards of --op ids-partition (default 8)")
    ap.add_argument("--kernels-from", nargs=6,
                    metavar=("TRACE_DIR", "FETCH_DIR", "WRITE_DIR", "CAL_FETCH_DIR", "CAL_WRITE_DIR", "CEIL_JSON"),
                    help="write profiles/kernels_<workload>.md: each step kernel's time, traffic, real bandwidth and "
                         "its probe ceiling (no GPU needed)")
    ap.add_argument("--ceilings-from", nargs="+", metavar="PATH",
                    help="write profiles/ceilings_mi355x.md from a --ceilings JSON line [and its rocprofv3 "
                         "--kernel-trace --stats output directory] (no GPU needed)")
    ap.add_argument("--ceilings", action="store_true",
                    help="measure plain device read / write / copy / random-row gather bandwidth and exit")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run the library's 1 GiB copy probe 5 times (scales HBM byte counters)")
    ap.add_argument("--traffic-from", nargs=4, metavar=("FETCH_DIR", "WRITE_DIR", "CAL_FETCH_DIR", "CAL_WRITE_DIR"),
                    help="write profiles/traffic_<workload>*.{md,json} from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE "
                         "output directories of a step run and of a --copy-calibration run (no GPU needed)")
    ap.add_argument("--traffic-cmd", default="", help="the profiled command, recorded in the summary")
    ap.add_argument("--trace-from", metavar="DIR",
                    help="write profiles/step_kernels_<workload>.md from a rocprofv3 --kernel-trace --stats output "
                         "directory of a step run: per-kernel time over the timed steps and the --stats table")
    ap.add_argument("--counters-from", metavar="DIR",
                    help="write profiles/l2_<workload>.md from a rocprofv3 --pmc TCC_HIT_sum TCC_MISS_sum "
                         "TCC_ATOMIC_sum output directory (last dispatch of each step kernel)")
    return ap.parse_args()


def host_cpu() -> dict:
    """The host the CPU baseline ran on: its logical CPUs and CPU model."""
    model = None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"host_nproc": os.cpu_count(), "host_cpu_model": model}


def _probe_ms(fn, reps: int = 5) -> float:
    """Median time (ms) of fn() over reps launches, each bracketed by events."""
    import torch

    fn()
    torch.cuda.synchronize()
    ms = []
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        fn()
        e1.record()
        torch.cuda.synchronize()
        ms.append(e0.elapsed_time(e1))
    return float(np.median(ms))


def copy_ms(n: int = 1 << 30, reps: int = 5) -> float:
    """Time (ms) of the library's copy probe over n bytes (n read + n written)."""
    import torch

    from paper_2509_20883_amd import recis as R

    src = torch.empty(n, dtype=torch.uint8, device="cuda").fill_(1)
    dst = torch.empty_like(src)
    ms = _probe_ms(lambda: R.bandwidth_probe("copy", src, dst), reps)
    del src, dst
    torch.cuda.empty_cache()
    return ms


def ceilings():
    """Practical HBM ceilings of this GPU, from the library's bandwidth probes
    (hand-written kernels with the step's access widths and launch shapes) on
    2 GiB buffers: sequential read, streaming write, copy, a gather of random
    256-byte rows into a streamed output, and a random read-modify-write of
    768-byte rows (a dim-64 fp32 row with its two Adam moments).  Bytes moved /
    median time of 5 launches."""
    import torch

    from paper_2509_20883_amd import recis as R

    nb = 1 << 31
    x = torch.ones(nb // 4, dtype=torch.float32, device="cuda")
    y = torch.empty_like(x)
    sink = torch.zeros(4, dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(2509)
    n_g = nb // 256 // 4  # a quarter of the 256-byte rows, gathered
    idx_g = torch.randint(0, nb // 256, (n_g,), device="cuda", generator=g)
    out = torch.empty(n_g * 64, dtype=torch.float32, device="cuda")
    n_r = nb // 768 // 4  # a quarter of the 768-byte rows, updated (distinct rows)
    idx_r = torch.randperm(nb // 768, device="cuda", generator=g)[:n_r]
    tests = {
        "read": (lambda: R.bandwidth_probe("read", x, sink), nb),
        "write (streaming)": (lambda: R.bandwidth_probe("write", y), nb),
        "copy": (lambda: R.bandwidth_probe("copy", x, y), 2 * nb),
        "gather of random 256-byte rows (read + streamed write + index)":
            (lambda: R.bandwidth_probe("gather", x, out, idx_g, row_bytes=256), (2 * 256 + 8) * n_g),
        "read-modify-write of random 768-byte rows (+ index)":
            (lambda: R.bandwidth_probe("rmw", x, None, idx_r, row_bytes=768), (2 * 768 + 8) * n_r),
    }
    res = {}
    for name, (fn, nbytes) in tests.items():
        m = _probe_ms(fn)
        res[name] = {"bytes": nbytes, "ms": m, "GBps": nbytes / (m * 1e-3) / 1e9}
    print(json.dumps({"ceilings": res, "peak_GBps": HBM_PEAK_GBPS}))


# which probe ceiling bounds each step kernel's access pattern (none: the
# dedup passes' mixed random accesses of 8-32 bytes have no probe of their own)
KERNEL_CEILING = {
    "rs::k_bwd_short<": "read-modify-write of random 768-byte rows (+ index)",
    "rs::k_pool<": "gather of random 256-byte rows (read + streamed write + index)",
    "rs::k_pool_none<": "gather of random 256-byte rows (read + streamed write + index)",
    "rs::k_bwd_long<": "read",
    "rs::k_occ_list": "copy",
    "rs::k_occ_init<": "copy",
}


def kernels_from(a):
    """profiles/kernels_<workload>.md: per step kernel, its mean time over the
    timed steps (kernel trace), its HBM traffic per launch (FETCH_SIZE /
    WRITE_SIZE scaled by the copy probe), the real bandwidth that makes, and
    the probe ceiling of its access pattern (a --ceilings JSON line)."""
    from collections import defaultdict

    tdir, fdir, wdir, cfdir, cwdir, cjson = a.kernels_from
    wl = profile_label(a)
    by = defaultdict(list)
    for r in _csv_rows(tdir, "kernel_trace.csv"):
        by[_kname(r)].append((int(r["Dispatch_Id"]), (int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) / 1e3))
    us = {k: float(np.mean([t for _, t in sorted(v)[-a.steps:]])) for k, v in by.items() if k.startswith("rs::")}
    gib_kib = (1 << 30) / 1024

    def calib(d):
        return gib_kib / float(np.median([float(r["Counter_Value"]) for r in _counter_rows(d)
                                          if "k_probe_copy" in r["Kernel_Name"]]))

    def last(d):
        m = defaultdict(list)
        for r in _counter_rows(d):
            m[_kname(r)].append((int(r["Dispatch_Id"]), float(r["Counter_Value"]) * 1024))
        return _drop_setup_only({k: max(v) for k, v in m.items()})

    fs, ws = calib(cfdir), calib(cwdir)
    F, Wr = last(fdir), last(wdir)
    with open(cjson) as fh:
        ceil = json.loads([ln for ln in fh if ln.startswith("{")][-1])["ceilings"]
    lines = [f"# Step kernels against the bandwidth ceilings: {wl}", "",
             "Per kernel: mean time over the timed steps (kernel trace), HBM bytes per launch at the last step "
             f"(FETCH_SIZE x{fs:.3f}, WRITE_SIZE x{ws:.3f}, the copy probe's scale), the real bandwidth they make, and "
             "the library probe whose access pattern the kernel shares (`bench.py --ceilings`).  Converted by "
             "`bench.py --kernels-from` from the runs of these commands:", "", "```",
             a.traffic_cmd or "(commands not recorded)", "```", "",
             "| kernel | us | fetch MB | write MB | real GB/s | ceiling probe | probe GB/s | % of probe |",
             "|---|---|---|---|---|---|---|---|"]
    for k in sorted(us, key=lambda k: -us[k]):
        if ("probe" in k or "rehash" in k or "rereserve" in k or "map_rows" in k or "k_occ_init<false>" in k
                or k not in F):
            continue
        fb, wb = F[k] * fs, Wr.get(k, 0.0) * ws
        gbps = (fb + wb) / (us[k] * 1e-6) / 1e9
        probe = next((c for pre, c in KERNEL_CEILING.items() if k.startswith(pre)), None)
        pg = ceil[probe]["GBps"] if probe in ceil else None
        lines.append(f"| `{k}` | {us[k]:.1f} | {fb / 1e6:.1f} | {wb / 1e6:.1f} | {gbps:.0f} | "
                     f"{probe or 'none (mixed random 8-32-byte accesses)'} | {f'{pg:.0f}' if pg else '-'} | "
                     f"{f'{100 * gbps / pg:.0f}' if pg else '-'} |")
    lines.append("")
    os.makedirs(PROFILES, exist_ok=True)
    with open(os.path.join(PROFILES, f"kernels_{wl}.md"), "w") as fh:
        fh.write("\n".join(lines))
    print("\n".join(lines))


def ceilings_from(a):
    """profiles/ceilings_mi355x.md from the JSON line of a `--ceilings` run
    and, if given, the rocprofv3 `--kernel-trace --stats` output of the same
    command (the probe kernels' own durations)."""
    with open(a.ceilings_from[0]) as fh:
        d = json.loads([ln for ln in fh if ln.startswith("{")][-1])
    peak = d["peak_GBps"]
    lines = ["# Practical HBM ceilings of this MI355X: the library's probe kernels, 2 GiB buffers", "",
             "Commands (repository root copied to `<repo>`):", "", "```", a.traffic_cmd or "(command not recorded)",
             "```", "",
             "`bench.py --ceilings` times each probe (`rs_bandwidth_probe`, `csrc/probes.hip`: 256-thread blocks, "
             "16-byte lane accesses, one pass) with HIP events, the median of 5 launches after one untimed launch; "
             "bytes moved / time.  Converted by `bench.py --ceilings-from`.", "",
             "| operation | bytes per launch | ms | GB/s | % of 8 TB/s |", "|---|---|---|---|---|"]
    for name, r in d["ceilings"].items():
        lines.append(f"| {name} | {r['bytes']} | {r['ms']:.3f} | {r['GBps']:.0f} | {100 * r['GBps'] / peak:.1f} |")
    if len(a.ceilings_from) > 1:
        lines += ["", "The probe kernels in the rocprofv3 trace of the same command (every launch):", "",
                  "| kernel | calls | avg us | min us | max us |", "|---|---|---|---|---|"]
        for r in _csv_rows(a.ceilings_from[1], "kernel_stats.csv"):
            name = r["Name"].split("(")[0].replace("void ", "")
            if "k_probe" in name:
                lines.append(f"| `{name}` | {r['Calls']} | {float(r['AverageNs']) / 1e3:.2f} | "
                             f"{float(r['MinNs']) / 1e3:.2f} | {float(r['MaxNs']) / 1e3:.2f} |")
    lines += ["", "The read-modify-write probe writes its rows back with non-temporal stores, as the "
              "optimizer's update does; the gather and the streaming write and copy store their outputs "
              "non-temporally too.", ""]
    os.makedirs(PROFILES, exist_ok=True)
    with open(os.path.join(PROFILES, "ceilings_mi355x.md"), "w") as fh:
        fh.write("\n".join(lines))
    print("\n".join(lines))


def copy_calibration():
    """The library's copy probe over 1 GiB (1 GiB read + 1 GiB written per
    launch), five launches: the reference for scaling HBM byte counters."""
    n = 1 << 30
    ms = copy_ms(n)
    print(json.dumps({"copy_bytes_read": n, "copy_bytes_written": n, "ms": ms, "GBps": 2 * n / (ms * 1e-3) / 1e9}))


def _drop_setup_only(last):
    """{kernel: (last dispatch, value)} -> {kernel: value} without the kernels that only the set-up ran (the scratch
    table's step): their last dispatch is before the last step's first kernel."""
    first = last.get("rs::k_tile_dedup<1024>", (-1, None))[0]
    return {k: v for k, (d, v) in last.items() if d >= first}


def _counter_rows(d: str):
    """Rows of the counter_collection CSV under a rocprofv3 output directory."""
    import csv
    import glob

    files = glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True)
    if not files:
        raise FileNotFoundError(f"no counter_collection.csv under {d}")
    with open(files[0]) as fh:
        return list(csv.DictReader(fh))


# kernels whose last dispatch in a counter run is one step's launch, by the
# name the roofline uses (the hot-key backward is its unit sums + finish)
TRAFFIC_KERNELS = {"pool": ("rs::k_pool<", "rs::k_pool_none<"), "bwd_short": ("rs::k_bwd_short<",),
                   "bwd_long": ("rs::k_bwd_long<", "rs::k_bwd_long_finish<")}


def profile_label(a) -> str:
    """The workload a profile covers: the step's workload name, or the
    operator run by --op with its size."""
    if a.op == "ids-partition":
        return f"ids_partition_1M_{a.shards or 8}shards"
    if a.op in ("bucketize", "mod"):
        return f"{a.op}_100x10000"
    from paper_2509_20883_amd import workloads as W

    wl = W.describe(W.workload(a.workload))["workload"]
    age = getattr(a, "evict_age", -1)
    return f"{wl}_evictable_age{age}" if age is not None and age >= 0 else wl


def traffic_from(a):
    """HBM bytes per launch from FETCH_SIZE / WRITE_SIZE (KiB per dispatch),
    each scaled by what the same counter reads for the library's copy probe
    of 1 GiB read + 1 GiB written; the step's kernels are taken at their last
    dispatch (the last step of the profiled run)."""
    from collections import defaultdict


    fdir, wdir, cfdir, cwdir = a.traffic_from
    gib_kib = (1 << 30) / 1024

    def calib(d):
        vals = [float(r["Counter_Value"]) for r in _counter_rows(d) if "k_probe_copy" in r["Kernel_Name"]]
        if not vals:
            raise RuntimeError(f"no copy-probe dispatch in {d}")
        return gib_kib / float(np.median(vals))

    fs, ws = calib(cfdir), calib(cwdir)

    def last(d):
        by = defaultdict(list)
        for r in _counter_rows(d):
            name = r["Kernel_Name"].split("(")[0].replace("void ", "").strip()
            by[name].append((int(r["Dispatch_Id"]), float(r["Counter_Value"])))
        return {k: v * 1024 for k, v in _drop_setup_only({k: max(v) for k, v in by.items()}).items()}

    F, Wr = last(fdir), last(wdir)
    wl = profile_label(a)
    unit = "call" if a.op != "step" else "step"
    step = sorted((k for k in F if k.startswith("rs::") and "probe" not in k and "rehash" not in k
                   and "map_rows" not in k and "k_occ_init<false>" not in k), key=lambda k: -(F[k] + Wr.get(k, 0)))
    lines = [f"# HBM traffic per launch: {wl}", "",
             f"Counters `FETCH_SIZE` and `WRITE_SIZE` (KiB per dispatch), each in its own run, at the last {unit} of",
             "",
             "```", a.traffic_cmd or "(command not recorded)", "```", "",
             "scaled by the same counters on the library's copy probe of 1 GiB read + 1 GiB written "
             f"(`bench.py --copy-calibration`): fetch x{fs:.3f}, write x{ws:.3f}.  Converted by "
             "`bench.py --traffic-from`.", "",
             "| kernel | fetch MB | write MB |", "|---|---|---|"]
    tf = tw = 0.0
    for k in step:
        f, x = F[k] * fs / 1e6, Wr.get(k, 0.0) * ws / 1e6
        tf += f
        tw += x
        lines.append(f"| `{k}` | {f:.1f} | {x:.1f} |")
    lines += [f"| {unit} total | {tf:.0f} | {tw:.0f} |", ""]
    os.makedirs(PROFILES, exist_ok=True)
    with open(os.path.join(PROFILES, f"traffic_{wl}.md"), "w") as fh:
        fh.write("\n".join(lines))
    for kern, prefixes in TRAFFIC_KERNELS.items():
        names = [k for k in step if k.startswith(prefixes)]
        if not names:
            continue
        fb = sum(F[k] for k in names) * fs
        wb = sum(Wr.get(k, 0.0) for k in names) * ws
        rec = {"kernel": kern, "kernels": names, "workload": wl, "bytes_per_launch": fb + wb, "fetch_bytes": fb,
               "write_bytes": wb, "fetch_scale": fs, "write_scale": ws, "kernel_source_hash": kernel_source_hash(kern),
               "counters_from": f"profiles/traffic_{wl}.md"}
        with open(os.path.join(PROFILES, f"traffic_{wl}_{kern}.json"), "w") as fh:
            json.dump(rec, fh, indent=1)
    print("\n".join(lines))


def _csv_rows(d: str, suffix: str):
    import csv
    import glob

    files = glob.glob(os.path.join(d, "**", f"*{suffix}"), recursive=True)
    if not files:
        raise FileNotFoundError(f"no *{suffix} under {d}")
    with open(files[0]) as fh:
        return list(csv.DictReader(fh))


def _kname(r) -> str:
    return r["Kernel_Name"].split("(")[0].replace("void ", "").strip()


def trace_from(a):
    """Per-kernel time of the timed steps (their last a.steps launches of each
    step kernel, from the kernel trace) and rocprofv3's --stats table."""
    from collections import defaultdict


    wl = profile_label(a)
    unit = "call" if a.op != "step" else "step"
    rows = _csv_rows(a.trace_from, "kernel_trace.csv")
    by = defaultdict(list)
    for r in rows:
        by[_kname(r)].append((int(r["Dispatch_Id"]), (int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) / 1e3))
    step = {k: v for k, v in by.items() if k.startswith("rs::") and "probe" not in k and "rehash" not in k
            and "map_rows" not in k and "k_occ_init<false>" not in k and "rereserve" not in k}
    if getattr(a, "evict_age", -1) < 0:  # a kernel of the set-up alone (the scratch table's step) is no part of a step
        step = {k: v for k, v in step.items() if len(v) >= a.steps}
    how = (f"--op {a.op} --shards {a.shards or 8}" if a.op == "ids-partition" else
           f"--op {a.op}" if a.op != "step" else f"--workload {a.workload}")
    lines = [f"# Kernel time per {unit}: {wl}", "", "Command (MI355X, repository root copied to `<repo>`):", "", "```",
             a.traffic_cmd or "(command not recorded)", "```", "",
             f"Converted by `bench.py {how} --steps {a.steps} --trace-from <dir>`.", "",
             f"## Per {unit} (the last {a.steps} launches of each kernel: the timed {unit}s)", "",
             "| kernel | mean us | % of kernel time |", "|---|---|---|"]
    means = {k: float(np.mean([t for _, t in sorted(v)[-a.steps:]])) for k, v in step.items()}
    tot = sum(means.values())
    for k in sorted(means, key=lambda k: -means[k]):
        lines.append(f"| `{k}` | {means[k]:.1f} | {100 * means[k] / tot:.1f} |")
    lines += [f"| sum | {tot:.1f} | |", "", "## rocprofv3 `--stats` (all launches of the run, set-up included)", "",
              "| kernel | calls | avg us | min us | max us | % time |", "|---|---|---|---|---|---|"]
    for r in _csv_rows(a.trace_from, "kernel_stats.csv")[:16]:
        lines.append(f"| `{r['Name'].split('(')[0].replace('void ', '')[:70]}` | {r['Calls']} | "
                     f"{float(r['AverageNs']) / 1e3:.2f} | {float(r['MinNs']) / 1e3:.2f} | "
                     f"{float(r['MaxNs']) / 1e3:.2f} | {float(r['Percentage']):.1f} |")
    os.makedirs(PROFILES, exist_ok=True)
    with open(os.path.join(PROFILES, f"step_kernels_{wl}.md"), "w") as fh:
        fh.write("\n".join(lines) + "\n")
    print("\n".join(lines))


def counters_from(a):
    """L2 hit rate and atomics per step kernel (its last dispatch)."""
    from collections import defaultdict

    wl = profile_label(a)
    last, vals = {}, defaultdict(dict)
    rows = _csv_rows(a.counters_from, "counter_collection.csv")
    for r in rows:
        k, d = _kname(r), int(r["Dispatch_Id"])
        last[k] = max(last.get(k, -1), d)
    kept = _drop_setup_only({k: (d, d) for k, d in last.items()})
    for r in rows:
        k = _kname(r)
        if k in kept and int(r["Dispatch_Id"]) == last[k]:
            vals[k][r["Counter_Name"]] = float(r["Counter_Value"])
    lines = [f"# L2 hits and atomics per launch: {wl}", "", "Command (MI355X, repository root copied to `<repo>`):",
             "", "```", a.traffic_cmd or "(command not recorded)", "```", "",
             "Last dispatch of each step kernel (the last step); TCC_HIT / TCC_MISS are L2 requests over all "
             f"channels, TCC_ATOMIC the atomics that reach L2.  Converted by `bench.py --counters-from`.", "",
             "| kernel | L2 hits (M) | L2 misses (M) | hit rate | atomics (M) |", "|---|---|---|---|---|"]
    for k, v in sorted(vals.items(), key=lambda kv: -(kv[1].get("TCC_HIT_sum", 0) + kv[1].get("TCC_MISS_sum", 0))):
        if not k.startswith("rs::") or "probe" in k:
            continue
        h, m = v.get("TCC_HIT_sum", 0.0), v.get("TCC_MISS_sum", 0.0)
        lines.append(f"| `{k}` | {h / 1e6:.1f} | {m / 1e6:.1f} | {h / max(h + m, 1):.2f} | "
                     f"{v.get('TCC_ATOMIC_sum', 0.0) / 1e6:.2f} |")
    os.makedirs(PROFILES, exist_ok=True)
    with open(os.path.join(PROFILES, f"l2_{wl}.md"), "w") as fh:
        fh.write("\n".join(lines) + "\n")
    print("\n".join(lines))


KERNEL_SOURCES = {"pool": "pool.hip", "bwd_short": "backward.hip", "bwd_long": "backward.hip"}


def kernel_source_hash(kernel: str) -> str:
    """Hash of the sources a kernel is built from (its file + the shared headers)."""
    h = hashlib.sha256()
    for f in (KERNEL_SOURCES[kernel], "rs_internal.h", "device_common.h"):
        with open(os.path.join(ROOT, "paper_2509_20883_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def row_bytes(w):
    """Row bytes of w and of its optimizer state (the state's fp32 elements)."""
    R = w.dim * (2 if w.row_dtype == 1 else 4)
    S = 4 * {0: w.dim, 4: 1, 5: w.dim + 1}.get(w.opt, 2 * w.dim)
    return R, S


def b_alg(w, N, G, U, Nnew, V=None):
    """Algorithmic HBM bytes of one step (every array moved once; rows of
    duplicate ids counted once).  V: ids inside the padded modes' copied
    windows (sum over bags of min(len, pad_len))."""
    R, S = row_bytes(w)
    if w.mode in (2, 3):
        L = w.pad_len
        out = G * L * R + G * L            # padded rows + mask
        grad = (N if V is None else V) * R  # gradient rows of the copied ids only
    else:
        out = G * w.dim * 4
        grad = G * w.dim * 4
    return (8 * N + 8 * (G + 1) + 4 * N + 8 * U + 8 * U + 16 * U + 8 * U + 8 * U + Nnew * (16 + R + S)
            + 4 * N + R * U + out + grad + 4 * N + 2 * (R + S) * U)


def b_occ(w, N, G, U, Nnew, V=None):
    """B_occ: b_alg with the row of every gathered occurrence counted (no
    reuse of a duplicate id's row), the traffic if no row came from a cache;
    a bandwidth from it is an effective figure, not HBM traffic."""
    R, _ = row_bytes(w)
    return b_alg(w, N, G, U, Nnew, V) - R * U + R * (N if V is None else V)


def unit_count(c: int, unit: int = 32, max_units: int = 1024) -> int:
    """Backward units of a hot key with c occurrences (unit << shift positions, at most max_units)."""
    sh = 0
    while ((c - 1) >> (sh + 5)) >= max_units:
        sh += 1
    usz = unit << sh
    return (c + usz - 1) // usz


def window_mask(w, offsets: np.ndarray, n: int):
    """Positions whose id is copied by a padded mode (all positions otherwise)."""
    if w.mode not in (2, 3):
        return None
    lens = np.diff(offsets)
    t = np.arange(n) - np.repeat(offsets[:-1], lens)           # position inside the bag
    skip = np.repeat(np.maximum(lens - w.pad_len, 0), lens) if w.mode == 3 else 0
    return (t >= skip) & (t < skip + w.pad_len)


def key_stats(values: np.ndarray, offsets: np.ndarray, window=None, long_threshold: int = 32):
    """Host-side split of a batch into short keys (<= 32 occurrences) and hot
    keys; Nw_* count the occurrences that carry a gradient row (inside the
    padded modes' windows), Gb_* the distinct bags those occurrences lie in."""
    uk, inv, cnt = np.unique(values, return_inverse=True, return_counts=True)
    inv = inv.reshape(-1)
    cw = cnt if window is None else np.bincount(inv[window], minlength=uk.size)
    hot = cnt > long_threshold
    G = offsets.size - 1
    bag = np.repeat(np.arange(G, dtype=np.int64), np.diff(offsets))
    hot_occ = hot[inv]
    carry = np.ones(values.size, dtype=bool) if window is None else window

    def distinct_bags(sel):
        return int(np.count_nonzero(np.bincount(bag[sel & carry], minlength=G)))

    return {"U": int(cnt.size), "U_short": int((~hot).sum()), "N_short": int(cnt[~hot].sum()),
            "U_long": int(hot.sum()), "N_long": int(cnt[hot].sum()),
            "Nw_short": int(cw[~hot].sum()), "Nw_long": int(cw[hot].sum()), "V": int(cw.sum()),
            "Gb_short": distinct_bags(~hot_occ), "Gb_long": distinct_bags(hot_occ),
            "units": int(sum(unit_count(int(c)) for c in cnt[hot]))}


def kernel_bytes(w, kernel, N, G, ks):
    """Bytes of one launch of the largest kernels: (alg, impl).

    alg: the step's algorithmic byte terms (the B_alg formula) that this
    kernel moves -- pool: offsets, the inverse read, the row ids read, the
    unique rows, the output; backward: the upstream gradient rows (each
    gradient row once), the inverse read of the kernel's occurrences, the
    row + state read-modify-write of its keys.  impl: every array element the
    implementation touches, counted once (alg plus its own bookkeeping:
    occurrence lists, segment descriptors, partial rows)."""
    R, S = row_bytes(w)
    U = ks["U"]
    padded = w.mode in (2, 3)
    gr = R if padded else w.dim * 4
    if kernel == "pool":
        out = G * w.pad_len * R + G * w.pad_len if padded else G * w.dim * 4
        alg = 8 * (G + 1) + 4 * N + 8 * U + R * U + out
        # the kernel reads each id's row id (8 B) and writes the id's gradient
        # row (4 B), both in id order
        impl = 8 * (G + 1) + 8 * N + R * U + out + 4 * N
        return alg, impl
    if kernel == "bwd_short":
        Us, Ns, Nw = ks["U_short"], ks["N_short"], ks["Nw_short"]
        grad_alg = gr * (Nw if padded else ks["Gb_short"])
        alg = grad_alg + 4 * Ns + 2 * (R + S) * Us
        # segment descriptors of every key, one gradient row per occurrence
        # (mean pooling: the bag offsets for the scales)
        impl = 16 * U + 4 * Ns + gr * Nw + 2 * (R + S) * Us + (8 * (G + 1) if w.mode == 1 else 0)
        return alg, impl
    if kernel == "bwd_long":
        Ul, Nl, Nw, nu = ks["U_long"], ks["N_long"], ks["Nw_long"], ks["units"]
        grad_alg = gr * (Nw if padded else ks["Gb_long"])
        alg = grad_alg + 4 * Nl + 2 * (R + S) * Ul
        # unit descriptors, one gradient row per occurrence, one partial row
        # written and read back per unit
        impl = (16 * nu + 4 * Nl + gr * Nw + 2 * 4 * w.dim * nu + 2 * (R + S) * Ul
                + (8 * (G + 1) if w.mode == 1 else 0))
        return alg, impl
    raise KeyError(kernel)


def _gen_batch(arg):
    """Worker: the host arrays of one step's batch (generator only)."""
    k, s = arg
    from paper_2509_20883_amd import workloads as W

    b = W.make_batch(W.workload(k), s)
    return s, b.values, b.offsets


def progress(msg: str):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def host_batches(k: int, nsteps: int, workers: int = 16):
    """Every step's batch, drawn by a pool of forked worker processes before
    the GPU is touched (the draws are seeded per step, so the result does
    not depend on the number of workers)."""
    import multiprocessing as mp

    nw = max(1, min(workers, os.cpu_count() or 1, nsteps))
    out = [None] * nsteps
    t0 = time.time()
    if nw == 1:
        it = map(_gen_batch, [(k, s) for s in range(nsteps)])
        for s, v, o in it:
            out[s] = (v, o)
    else:
        with mp.get_context("fork").Pool(nw) as pool:
            for j, (s, v, o) in enumerate(pool.imap_unordered(_gen_batch, [(k, s) for s in range(nsteps)])):
                out[s] = (v, o)
                if (j + 1) % 8 == 0 or j + 1 == nsteps:
                    progress(f"generated {j + 1}/{nsteps} batches ({time.time() - t0:.0f} s)")
    return out


def cpu_baseline(w, target_s):
    """The oracle as it stands, single-threaded, on consecutive full batches of the
    workload until about target_s seconds of step time have been measured."""
    import oracle as O
    from paper_2509_20883_amd import workloads as W

    ot = O.Table(w.dim, row_dtype=w.row_dtype, opt=w.opt, lo=w.init_lo, hi=w.init_hi, seed=w.table_seed)
    present = set()
    pool_keys = None
    ids = secs = 0.0
    steps = 0
    while secs < target_s and steps < 50:
        b = W.make_batch(w, steps)
        if w.mode in (2, 3):
            grad = W.make_grad(w, b, steps)
        else:
            grad = np.random.default_rng(steps).standard_normal((b.bags, w.dim)).astype(np.float32)
        # pre-populated keys are materialised lazily, on first sight (untimed)
        if w.prepop != "none":
            uk = np.unique(b.values)
            uk = uk[[k not in present for k in uk.tolist()]] if present else uk
            if w.prepop == "frac90":
                member = np.zeros(uk.size, dtype=bool)
                fid = uk >> 40
                for f in np.unique(fid):
                    sel = fid == f
                    member[sel] = W.prepop_member(w, int(f), uk[sel] & ((1 << 40) - 1))
                ot.find_or_insert(uk[member])
            elif w.prepop == "all":
                ot.find_or_insert(uk)
            elif w.prepop == "pool":
                if pool_keys is None:
                    pool_keys = np.sort(np.concatenate(list(W.prepop_keys(w))))
                ot.find_or_insert(uk[np.isin(uk, pool_keys, assume_unique=True)])
            present.update(uk.tolist())
        t0 = time.perf_counter()
        ot.step(b.values, b.offsets, w.mode, grad, w.lr, w.eps, w.beta1, w.beta2, pad_len=w.pad_len,
                weight_decay=w.weight_decay)
        secs += time.perf_counter() - t0
        ids += b.n
        steps += 1
    return {"value": ids / secs, "unit": "IDs/s", "cores": 1, "kind": "oracle",
            "sample": f"{steps} consecutive full steps (batch {w.batch} x {w.n_features} features, "
                      f"{int(ids)} ids), {secs:.1f} s of single-threaded step time", **host_cpu()}


IDS_METRIC = "ids partition (dedup + split by owner shard) IDs/sec and achieved HBM GB/s vs peak, 1 MI355X"


def ids_partition_bytes(n: int, U: int, G: int) -> int:
    """Algorithmic bytes of one ids partition: ids read once; distinct keys,
    shard offsets, the inverse and the two info words written once."""
    return 8 * n + 8 * U + 8 * (G + 1) + 4 * n + 16


def bench_ids_partition(a):
    from paper_2509_20883_amd import workloads as W

    G = a.shards or W.IDS_PARTITION_SHARDS
    seed = W.IDS_PARTITION_SEED
    nring = 4
    host = [W.ids_partition_values(step=s) for s in range(nring)]
    import torch

    from paper_2509_20883_amd import recis as R

    torch.cuda.set_device(0)
    dev = torch.device("cuda", 0)
    vals = [torch.from_numpy(v).to(dev) for v in host]
    n = int(max(v.numel() for v in vals))
    part = R.IdsPartition()
    keys = torch.empty(n, dtype=torch.int64, device=dev)
    offs = torch.empty(G + 1, dtype=torch.int64, device=dev)
    inv = torch.empty(n, dtype=torch.int32, device=dev)
    infos = torch.zeros(a.warmup + a.steps, 2, dtype=torch.int64, device=dev)
    for i in range(a.warmup):
        part(vals[i % nring], G, seed, keys, offs, inv, infos[i])
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for j in range(a.steps):
        i = a.warmup + j
        part(vals[i % nring], G, seed, keys, offs, inv, infos[i])
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / a.steps
    info = infos.cpu().numpy()
    if np.any(info[:, 1] != 0):
        raise RuntimeError(f"ids_partition reported error bits {info[:, 1].tolist()}")
    Us = [int(info[a.warmup + j, 0]) for j in range(a.steps)]
    ns = [int(vals[(a.warmup + j) % nring].numel()) for j in range(a.steps)]
    byts = float(np.mean([ids_partition_bytes(nn, U, G) for nn, U in zip(ns, Us)]))
    achieved = byts / (ms * 1e-3) / 1e9
    res = {
        "metric": IDS_METRIC,
        "value": float(np.mean(ns)) / (ms * 1e-3),
        "unit": "IDs/s",
        "n_gpus": 1,
        "steps": a.steps,
        "warmup": a.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int64",
        "data": "synthetic (26 single-hot Zipf(1.05) features, 4 batches resident in HBM, used in turn)",
        "config": {"workload": "ids-partition-1M", "ids": int(np.mean(ns)), "shards": G, "U_mean": float(np.mean(Us))},
        "roofline": {"bound": "hbm", "kernel": "ids_partition (whole call)", "achieved": achieved,
                     "peak": HBM_PEAK_GBPS, "unit": "GB/s", "frac": achieved / HBM_PEAK_GBPS, "traffic": None,
                     "kernel_ms": ms, "kernel_bytes_alg": byts},
    }
    if not a.no_cpu_baseline:
        import oracle as O

        t0 = time.perf_counter()
        calls = 0
        while calls == 0 or time.perf_counter() - t0 < a.cpu_seconds:
            O.ids_partition(host[calls % nring], G, seed)
            calls += 1
        dt = time.perf_counter() - t0
        cpu = {"value": calls * float(np.mean([h.size for h in host])) / dt, "unit": "IDs/s", "cores": 1,
               "kind": "oracle", "sample": f"{calls} whole calls on the same inputs", **host_cpu()}
        cpu["gpu_speedup"] = res["value"] / cpu["value"]
        res["cpu_baseline"] = cpu
    print(json.dumps(res), flush=True)


FEAT_METRIC = "fused {op} over 100 columns x 10,000 values: values/sec and achieved HBM GB/s vs peak, 1 MI355X"


def bench_feature_op(a):
    from paper_2509_20883_amd import workloads as W

    nring = 4
    host = [W.bucketize_columns(step=s) if a.op == "bucketize" else W.mod_columns(step=s) for s in range(nring)]
    import torch

    from paper_2509_20883_amd import recis as R

    torch.cuda.set_device(0)
    dev = torch.device("cuda", 0)
    ins = [tuple(torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in h) for h in host]
    n = int(host[0][0].size)
    out = torch.empty(n, dtype=torch.int64, device=dev)

    def call(i):
        x = ins[i % nring]
        if a.op == "bucketize":
            R.fused_bucketize(x[0], x[1], x[2], x[3], out=out)
        else:
            R.fused_mod(x[0], x[1], x[2], out=out)

    for i in range(a.warmup):
        call(i)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for j in range(a.steps):
        call(a.warmup + j)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / a.steps
    ncols = int(host[0][1].size - 1)
    if a.op == "bucketize":  # values, column offsets, boundaries + offsets read; buckets written
        byts = 4 * n + 8 * (ncols + 1) + 4 * int(host[0][2].size) + 8 * (ncols + 1) + 8 * n
    else:                    # ids, column offsets, moduli read; buckets written
        byts = 8 * n + 8 * (ncols + 1) + 8 * ncols + 8 * n
    achieved = byts / (ms * 1e-3) / 1e9
    res = {
        "metric": FEAT_METRIC.format(op=a.op),
        "value": n / (ms * 1e-3), "unit": "values/s", "n_gpus": 1, "steps": a.steps, "warmup": a.warmup,
        "ms_per_step": ms, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32->int64" if a.op == "bucketize" else "int64",
        "data": "synthetic (log-normal prices with quantile boundaries / Zipf ids with log-uniform moduli; "
                "4 inputs resident in HBM, used in turn)",
        "config": {"workload": f"{a.op}-100x10000", "columns": ncols, "values": n},
        "roofline": {"bound": "hbm", "kernel": f"k_{a.op}", "achieved": achieved, "peak": HBM_PEAK_GBPS,
                     "unit": "GB/s", "frac": achieved / HBM_PEAK_GBPS, "traffic": None, "kernel_ms": ms,
                     "kernel_bytes_alg": byts},
    }
    if not a.no_cpu_baseline:
        import oracle as O

        t0 = time.perf_counter()
        calls = 0
        while calls == 0 or time.perf_counter() - t0 < a.cpu_seconds:
            h = host[calls % nring]
            O.bucketize(*h) if a.op == "bucketize" else O.mod(*h)
            calls += 1
        dt = time.perf_counter() - t0
        cpu = {"value": calls * n / dt, "unit": "values/s", "cores": 1, "kind": "oracle",
               "sample": f"{calls} whole calls on the same inputs", **host_cpu()}
        cpu["gpu_speedup"] = res["value"] / cpu["value"]
        res["cpu_baseline"] = cpu
    print(json.dumps(res), flush=True)


def main():
    a = parse()
    if a.traffic_from:
        traffic_from(a)
        return
    if a.trace_from:
        if a.steps is None:
            a.steps = 100 if a.workload == 4 else 20
        trace_from(a)
        return
    if a.counters_from:
        counters_from(a)
        return
    if a.copy_calibration:
        copy_calibration()
        return
    if a.ceilings_from:
        ceilings_from(a)
        return
    if a.kernels_from:
        if a.steps is None:
            a.steps = 20
        kernels_from(a)
        return
    if a.ceilings:
        ceilings()
        return
    if a.gpus != 1:
        print(json.dumps({"error": "single-GPU build: run with --gpus 1 (the multi-GPU path is a design only)"}))
        sys.exit(2)
    if a.op == "ids-partition":
        a.steps = 100 if a.steps is None else a.steps
        bench_ids_partition(a)
        return
    if a.op in ("bucketize", "mod"):
        a.steps = 200 if a.steps is None else a.steps
        bench_feature_op(a)
        return
    from paper_2509_20883_amd import workloads as W

    w = W.workload(a.workload)
    if a.steps is None:
        a.steps = 100 if a.workload == 4 else 20
    if a.optimizer:
        w.opt = OPTIMIZERS.index(a.optimizer)
        if w.opt == 2:
            w.weight_decay = 0.01
    nsteps = a.warmup + a.steps
    t_setup = time.time()
    hb = host_batches(a.workload, nsteps, a.gen_workers)  # before the GPU is initialised (forked workers)

    import torch

    from paper_2509_20883_amd import recis as R

    torch.cuda.set_device(0)
    dev = torch.device("cuda", 0)
    evictable = a.evictable or a.evict_age >= 0
    table = R.Table(w.dim, w.row_dtype, w.opt, w.init_lo, w.init_hi, w.table_seed, w.capacity_slots, w.max_load,
                    w.block_rows, auto_grow=True, evictable=evictable)
    npre = 0
    for keys in W.prepop_keys(w):
        table.find_or_insert(torch.from_numpy(keys).to(dev))
        npre += keys.size
        if npre % (1 << 25) < keys.size:
            progress(f"pre-populated {npre} keys")
    live0 = table.size()
    progress(f"table ready: {live0} live rows")
    # every step's ids are resident in HBM before timing; the upstream
    # gradients (whose values do not change the work) come from a ring of 4
    # tensors, and long runs reuse a ring of step contexts (the per-step
    # counters are then copied out after each step)
    ring = nsteps if nsteps <= 32 else 8
    if a.pipelined and ring < nsteps:
        print(json.dumps({"error": "--pipelined needs at most 32 steps (one context per step)"}))
        sys.exit(2)
    batches, grads = [], []
    gen = torch.Generator(device=dev)
    gen.manual_seed(2509)
    # host-side key statistics (for the dominant kernel's bytes) of at most 5
    # evenly spaced timed steps
    stat_steps = set(np.linspace(a.warmup, nsteps - 1, num=min(a.steps, 5)).round().astype(int).tolist())
    host_values, host_windows = {}, {}
    for s in range(nsteps):
        bv, bo = hb[s]
        hb[s] = None
        nb, gb = int(bv.shape[0]), int(bo.shape[0] - 1)
        win = window_mask(w, bo, nb)
        if win is not None:
            host_windows[s] = int(win.sum())
        if s in stat_steps:
            host_values[s] = (bv, bo, win)
        batches.append((torch.from_numpy(bv).to(dev), torch.from_numpy(bo).to(dev), nb, gb))
        if s < 4:
            if w.mode in (2, 3):
                shape = (gb, w.pad_len, w.dim)
                gdt = torch.bfloat16 if w.row_dtype == 1 else torch.float32
            else:
                shape, gdt = (gb, w.dim), torch.float32
            grads.append(torch.randn(shape, generator=gen, device=dev, dtype=torch.float32).to(gdt))
    maxg = max(b[3] for b in batches)
    if w.mode != 2 and any(b[3] > grads[0].shape[0] for b in batches):
        grads = [torch.randn(maxg, w.dim, generator=gen, device=dev, dtype=torch.float32) for _ in grads]
    ctxs = [R.Ctx() for _ in range(ring)]
    stepscal = torch.zeros(nsteps, 4, dtype=torch.int64, device=dev)
    maxb = max(b[3] for b in batches)
    if w.mode in (2, 3):
        odt = torch.bfloat16 if w.row_dtype == 1 else torch.float32
        out = torch.empty(maxb, w.pad_len, w.dim, dtype=odt, device=dev)
        mask = torch.empty(maxb, w.pad_len, dtype=torch.uint8, device=dev)
    else:
        out = torch.empty(maxb, w.dim, dtype=torch.float32, device=dev)
        mask = None
    for c in ctxs:
        c.ensure(max(table.workspace_bytes(n, g, w.pad_len) for (v, o, n, g) in batches), dev)
    gu = None
    if a.unfused:
        gu = torch.empty(max(b[2] for b in batches), w.dim, dtype=torch.float32, device=dev)
    torch.cuda.synchronize()
    setup_s = time.time() - t_setup
    progress(f"setup done in {setup_s:.0f} s; {nsteps} steps")
    # plain device copy in the same run (untimed for the step): the practical
    # bandwidth the step's GB/s is also reported against
    copy_gbps = 2 * (1 << 30) / (copy_ms(1 << 30) * 1e-3) / 1e9
    progress(f"device copy: {copy_gbps:.0f} GB/s")

    def grad_of(i):
        g = batches[i][3]
        x = grads[i % len(grads)]
        return x if x.shape[0] == g else x[:g]

    def step(i):
        v, o, n, g = batches[i]
        ob = out[:g]
        mb = mask[:g] if mask is not None else None
        c = ctxs[i % ring]
        table.forward(v, o, w.mode, pad_len=w.pad_len, ctx=c, out=ob, mask=mb)
        if a.unfused:
            table.backward(c, grad_of(i), gu)
            table.optimizer_step(c, gu, w.lr, w.eps, w.beta1, w.beta2, w.weight_decay)
        else:
            table.backward_optimizer(c, grad_of(i), w.lr, w.eps, w.beta1, w.beta2, w.weight_decay)
        if ring < nsteps:
            stepscal[i].copy_(c.scalars())

    side = torch.cuda.Stream(device=dev)  # default priority

    # a code object is loaded at the first launch from it: one step of bags
    # spread over the first batch (the same mix of bag lengths), 1024 of them
    # or about 16384 ids (past the small batches' own kernels), on a small
    # scratch table of the same kind loads the step's code objects, so the
    # first warm-up step is no cold start
    scratch = R.Table(w.dim, w.row_dtype, w.opt, w.init_lo, w.init_hi, w.table_seed, 1 << 17, w.max_load,
                      w.block_rows, auto_grow=True, evictable=evictable)
    try:
        v0, o0, _, g0 = batches[0]
        oh = o0.cpu().numpy()
        some = min(g0, max(1024, int(16384 * g0 / max(int(oh[-1]), 1))))
        pick = np.unique(np.linspace(0, g0 - 1, num=some).round().astype(np.int64))
        lens = oh[pick + 1] - oh[pick]
        so_h = np.zeros(pick.size + 1, dtype=np.int64)
        np.cumsum(lens, out=so_h[1:])
        idx = np.concatenate([np.arange(oh[b], oh[b + 1]) for b in pick]) if so_h[-1] else np.zeros(0, np.int64)
        sv = v0[torch.from_numpy(idx).to(dev)]
        so = torch.from_numpy(so_h).to(dev)
        _, _, sctx = scratch.forward(sv, so, w.mode, pad_len=w.pad_len)
        gs = pick.size
        sg = grad_of(0)[:gs]
        if a.unfused:
            sgu = torch.empty(sv.numel(), w.dim, dtype=torch.float32, device=dev)
            scratch.backward(sctx, sg, sgu)
            scratch.optimizer_step(sctx, sgu, w.lr, w.eps, w.beta1, w.beta2, w.weight_decay)
        else:
            scratch.backward_optimizer(sctx, sg, w.lr, w.eps, w.beta1, w.beta2, w.weight_decay)
        torch.cuda.synchronize()
    finally:
        scratch.close()

    # untimed pass over the warm-up steps with per-kernel events: find the dominant kernel
    names = ["tile_dedup", "partition", "compact_insert", "occ", "pool", "occ_list", "bwd_short", "bwd_long"]
    if a.unfused:
        names.append("opt")
    prof = {k: [] for k in names}
    first_step = None
    for i in range(a.warmup):
        if i == 0 and a.warmup > 1:
            # the first step alone, without kernel events (on a table that
            # starts empty it inserts every key it sees: the insert-heavy step)
            f0, f1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            f0.record()
            step(0)
            f1.record()
            torch.cuda.synchronize()
            sc0 = (stepscal[0] if ring < nsteps else ctxs[0].scalars()).cpu().numpy()
            first_step = {"ms": f0.elapsed_time(f1), "ids": int(batches[0][2]), "U": int(sc0[0]),
                          "new_keys": int(sc0[1])}
            continue
        evs = {k: (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for k in names}
        for k, (e0, e1) in evs.items():
            table.set_kernel_events(k, e0, e1)
        step(i)
        torch.cuda.synchronize()
        for k, (e0, e1) in evs.items():
            prof[k].append(e0.elapsed_time(e1))
    for k in names:
        table.set_kernel_events(k, None, None)
    # the dominant kernel: the largest of the pool, the short-key backward and
    # the hot-key backward (unit sums + finish) by their median time over the
    # warm-up steps after the first (cold) one
    def wmed(k):
        return float(np.median(prof[k])) if prof[k] else 0.0

    dom = max(("pool", "bwd_short", "bwd_long"), key=wmed)
    cands = (dom,)
    # timed region: K steps, the dominant kernel timed in every 4th step by
    # start / stop events that its launch hands to the dispatch (timestamps
    # of the kernel's own execution on the step's stream)
    sampled = list(range(0, a.steps, 4))
    cand_ev = {k: {j: (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for j in sampled}
               for k in cands}

    def set_events(j):
        for k in cands:
            if j in cand_ev[k]:
                table.set_kernel_events(k, *cand_ev[k][j])
            else:
                table.set_kernel_events(k, None, None)
    for k in cands:  # create the events' handles before the timed region
        for e0, e1 in cand_ev[k].values():
            e0.record()
            e1.record()
    torch.cuda.synchronize()
    e_start, e_stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    # step boundaries (serial schedule): per-step times for the median
    step_ev = [torch.cuda.Event(enable_timing=True) for _ in range(a.steps)] if not a.no_step_events else []
    pipelined = a.pipelined
    caps = [table.capacity()]
    e_start.record()
    if pipelined:
        # the library records the dominant kernel's events at each launch; set
        # them per step just before that step's pool / backward is enqueued
        timed = list(range(a.warmup, a.warmup + a.steps))
        side.wait_event(e_start)
        cur = torch.cuda.current_stream()

        def prep(i):
            v, o, n, g = batches[i]
            table.prepare(v, o, w.mode, pad_len=w.pad_len, ctx=ctxs[i], stream=side)
            ev = torch.cuda.Event()
            ev.record(side)
            return ev

        # host order: prepare(j+1) is enqueued before pool(j) + backward(j),
        # so the side stream works on the next batch while this one runs
        nxt = prep(timed[0])
        for j, i in enumerate(timed):
            ev = nxt
            if j + 1 < len(timed):
                nxt = prep(timed[j + 1])
            _, _, n, g = batches[i]
            cur.wait_event(ev)
            set_events(j)
            ob = out[:g]
            mb = mask[:g] if mask is not None else None
            table.pool(ctxs[i], out=ob, mask=mb)
            if a.unfused:
                table.backward(ctxs[i], grad_of(i), gu)
                table.optimizer_step(ctxs[i], gu, w.lr, w.eps, w.beta1, w.beta2, w.weight_decay)
            else:
                table.backward_optimizer(ctxs[i], grad_of(i), w.lr, w.eps, w.beta1, w.beta2, w.weight_decay)
    else:
        for j in range(a.steps):
            set_events(j)
            step(a.warmup + j)
            if step_ev and j + 1 < a.steps:
                step_ev[j].record()
            # the host grows the IDMap inside the call when it must: its
            # capacity after the call tells whether this step resized it
            caps.append(table.capacity())
    e_stop.record()
    torch.cuda.synchronize()
    for k in cands:
        table.set_kernel_events(k, None, None)
    cand_ms = {k: float(np.mean([e0.elapsed_time(e1) for e0, e1 in cand_ev[k].values()])) for k in cands}
    total_ms = e_start.elapsed_time(e_stop)
    step_ms = None
    if step_ev and not pipelined:
        bounds = [e_start] + step_ev[:a.steps - 1] + [e_stop]
        step_ms = [bounds[j].elapsed_time(bounds[j + 1]) for j in range(a.steps)]
    table.check()
    eviction = None
    if a.evict_age >= 0:
        # one eviction over the whole table, after the timed steps: it reads
        # every allocated row's {key, clock} record (12 bytes) and, per evicted
        # key, writes its row's key, its free-stack entry and its IDMap slot
        rows_before = table.size()
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        ev0.record()
        n_ev = table.evict(a.evict_age)
        ev1.record()
        torch.cuda.synchronize()
        ems = ev0.elapsed_time(ev1)
        # rows allocated = live rows before the last step + the keys it inserted
        # (no row has been freed before this first eviction)
        last = (stepscal[-1] if ring < nsteps else ctxs[nsteps - 1].scalars()).cpu().numpy()
        hw = int(last[3] + last[1])
        ebytes = 12 * hw + n_ev * (8 + 8 + 16)
        eviction = {"max_age": a.evict_age, "ms": ems, "keys_before": rows_before, "evicted": n_ev,
                    "rows_scanned": hw, "bytes_alg": ebytes, "GBps_alg": ebytes / (ems * 1e-3) / 1e9}
        progress(f"evicted {n_ev} of {rows_before} keys in {ems:.3f} ms")
        # then compaction: the live rows above the live count move into the
        # freed rows below it and the Blocks past the live rows are released
        # (host time of the synchronizing call; it reads every row's key
        # record and moves whole rows of row + state + record)
        t0 = time.perf_counter()
        moved, released = table.compact()
        cms = (time.perf_counter() - t0) * 1e3
        live = table.size()
        eviction["compaction"] = {"ms_host": cms, "rows_moved": moved, "bytes_released": released,
                                  "live_rows": live, "rows_before": hw}
        progress(f"compacted: moved {moved} rows, released {released / 2**30:.2f} GiB in {cms:.1f} ms")

    # per-step sizes (read after the timed region)
    tot_ids = tot_bytes = tot_occ = 0
    Us, news, dom_b = [], [], []
    scal = stepscal.cpu().numpy() if ring < nsteps else None
    for j in range(a.steps):
        i = a.warmup + j
        sc = scal[i] if scal is not None else ctxs[i].scalars().cpu().numpy()
        U, Nnew = int(sc[0]), int(sc[1])
        _, _, n, g = batches[i]
        tot_ids += n
        V = host_windows.get(i)
        tot_bytes += b_alg(w, n, g, U, Nnew, V)
        tot_occ += b_occ(w, n, g, U, Nnew, V)
        if i in host_values:  # every timed step, or 5 evenly spaced ones in long runs
            hv, ho, hw = host_values[i]
            dom_b.append(kernel_bytes(w, dom, n, g, key_stats(hv, ho, hw)))
        Us.append(U)
        news.append(Nnew)
    dom_alg = float(np.mean([b[0] for b in dom_b]))
    dom_impl = float(np.mean([b[1] for b in dom_b]))
    dom_ms = cand_ms[dom]
    ms_per_step = total_ms / a.steps
    gbps = tot_bytes / (total_ms * 1e-3) / 1e9
    achieved = dom_alg / (dom_ms * 1e-3) / 1e9

    traffic = None
    tpath = os.path.join(PROFILES, f"traffic_{W.describe(w)['workload']}_{dom}.json")
    if os.path.exists(tpath):
        with open(tpath) as fh:
            tj = json.load(fh)
        if tj.get("kernel_source_hash") == kernel_source_hash(dom):
            traffic = tj.get("bytes_per_launch")

    res = {
        "metric": METRIC,
        "value": tot_ids / (total_ms * 1e-3),
        "unit": "IDs/s",
        "n_gpus": 1,
        "steps": a.steps,
        "warmup": a.warmup,
        "ms_per_step": ms_per_step,
        "ms_per_step_median": float(np.median(step_ms)) if step_ms else None,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32" if w.row_dtype == 0 else "bf16-storage/f32-math",
        "data": "synthetic (seeded Zipf ids, N(0,1) upstream grads from a ring of 4 tensors; inputs resident in HBM)",
        "config": {**W.describe(w), "live_rows_at_start": live0, "U_mean": float(np.mean(Us)),
                   "new_per_step_mean": float(np.mean(news)),
                   "bwd": "unfused" if a.unfused else "fused",
                   "schedule": "pipelined: next batch's lookup_prepare on a 2nd stream" if a.pipelined else "serial"},
        "gbps": gbps,
        "hbm_frac": gbps / HBM_PEAK_GBPS,
        "bytes_alg_per_step": tot_bytes / a.steps,
        "copy_gbps": copy_gbps,
        "frac_of_copy": gbps / copy_gbps,
        "bytes_occ_per_step": tot_occ / a.steps,
        "gbps_effective_occ": tot_occ / (total_ms * 1e-3) / 1e9,
        "roofline": {"bound": "hbm", "kernel": dom, "achieved": achieved, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBPS, "traffic": traffic, "kernel_ms": dom_ms,
                     "kernel_bytes_alg": dom_alg, "kernel_bytes_impl": dom_impl,
                     "kernel_bytes_bookkeeping": dom_impl - dom_alg},
        "idmap_resize": {"capacity_slots_start": caps[0], "capacity_slots_end": caps[-1],
                         "rehashes_in_window": sum(1 for x, y in zip(caps, caps[1:]) if y != x),
                         "resize_in_window": caps[-1] != caps[0],
                         "live_rows_end": table.size()} if not pipelined else None,
        "kernel_ms_warmup": {k: float(np.mean(v)) for k, v in prof.items() if v},
        "first_step": first_step,
        "evictable": evictable,
        "eviction": eviction,
        "setup_s": setup_s,
    }
    if not a.no_cpu_baseline:
        res["cpu_baseline"] = cpu_baseline(w, a.cpu_seconds)
        res["cpu_baseline"]["gpu_speedup"] = res["value"] / res["cpu_baseline"]["value"]
    table.close()
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
