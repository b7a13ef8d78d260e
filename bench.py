"""Benchmark of the whole hot path: one step = forest_predict over one batch of synthetic rows.

Prints ONE JSON line.  With no --workload it measures every configuration: the headline fields
(`value`, `config`, `roofline`, `cpu_baseline`, `parity`) are those of c5, the largest one, and
`per_config` holds the same fields for c4, c3, c2 and, as a latency, c1.  `value` is rows/s with
X already resident in HBM.  The `roofline` object prices the dominant (only) kernel against the
LDS: the walk kernels, which run every configuration here, test the nodes on a row's path, and a
test is two LDS reads, the node and the row's feature.
`cpu_baseline` is the CPU oracle timed on this machine's host cores over all rows of the
configuration (one warm-up pass, median of three timed passes), and `parity` compares every row
of the timed output with it.  The configurations are set up first and timed back to back, so
that none of the short ones starts on a GPU that has idled since the one before.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# MI355X: 256 compute units x 2.4 GHz; a wavefront's LDS read of 4 or 8 bytes per lane takes two
# clocks without bank conflicts, so 64 tests take four.
LDS_PEAK_TESTS = 256 * 2.4e9 * 64 / 4
HBM_PEAK = 8.0e12
ORACLE_THREADS_MAX = 16   # the share of host cores one GPU's job may use on the bench machine

# HBM bytes per launch from rocprofv3 --pmc runs of these workloads (FETCH_SIZE and WRITE_SIZE, each
# scaled by what the same counter reads for a plain copy of known size).  Not taken live: every
# entry names the summary under profiles/ it comes from and the commit whose kernels were
# measured; a workload without an entry reports null.
MEASURED_TRAFFIC = {
    "c2": {"bytes": 1.327e8, "profile": "profiles/forest_walk_kernels.md", "commit": "e207a50"},
    "c3": {"bytes": 2.110e8, "profile": "profiles/forest_walk_kernels.md", "commit": "e207a50"},
    "c4": {"bytes": 2.907e8, "profile": "profiles/forest_walk_kernels.md", "commit": "e207a50"},
    "c5": {"bytes": 4.164e9, "profile": "profiles/forest_walk_kernels.md", "commit": "e207a50"},
    "l2": {"bytes": 1.456e9, "profile": "profiles/linear_kernels.md", "commit": "7dd9b06"},
    "l3": {"bytes": 1.119e9, "profile": "profiles/linear_kernels.md", "commit": "7dd9b06"},
    "l4": {"bytes": 9.600e8, "profile": "profiles/linear_kernels.md", "commit": "7dd9b06"},
}


CLOCK_WARMUP_MS = 60.0  # untimed launches before a linear workload is timed (see bench_linear)


def bench_linear(args) -> int:
    """The linear-model family (one matmul + bias + transform + label): bound by reading X once
    from HBM, so its roofline is the HBM one."""
    import numpy as np
    import torch

    import paper_2301_13441_amd as pk
    from workloads.linear import make_linear_workload

    w = make_linear_workload(args.workload, n_rows=args.rows)
    n_rows, F, K = w.n_rows, w.model.n_features, w.model.n_outputs
    m = pk.linear_load(w.model)
    xd = torch.empty((n_rows, F), dtype=torch.float32, device="cuda")
    sample_rows = min(n_rows, 262144)
    parts = []
    pos = 0
    for chunk in w.x_chunks(n_rows):
        xd[pos:pos + len(chunk)].copy_(torch.from_numpy(chunk))
        if pos < sample_rows:
            parts.append(chunk[:max(0, sample_rows - pos)].copy())
        pos += len(chunk)
    x_sample = np.concatenate(parts)[:sample_rows]
    out = torch.empty(max(m.out_bytes(n_rows), 4), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream()
    # After an idle gap the clocks take about 25 ms of kernel time to come up, and K launches of a
    # kernel of a quarter of a millisecond end before that: untimed launches for CLOCK_WARMUP_MS
    # first, then the W warm-up and K timed ones.
    t_warm = time.perf_counter()
    while (time.perf_counter() - t_warm) * 1e3 < CLOCK_WARMUP_MS:
        for _ in range(10):
            m.predict(xd, out=out)
        torch.cuda.synchronize()
    for _ in range(args.warmup):
        m.predict(xd, out=out)
    torch.cuda.synchronize()
    starts = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    stops = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    t0 = time.perf_counter()
    for i in range(args.steps):
        starts[i].record(stream)
        m.predict(xd, out=out)
        stops[i].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    kernel_ms = [a.elapsed_time(b) for a, b in zip(starts, stops)]
    kernel_s = float(np.mean(kernel_ms)) * 1e-3
    scores, labels = m.predict(xd, out=out)
    torch.cuda.synchronize()
    algo_bytes = n_rows * 4.0 * F + m.out_bytes(n_rows)
    roofline = {
        "bound": "hbm",
        "kernel": "linear_predict (matmul + bias + transform + label, one kernel)",
        "achieved": algo_bytes / kernel_s / 1e9,
        "peak": HBM_PEAK / 1e9,
        "unit": "GB/s",
        "frac": algo_bytes / kernel_s / HBM_PEAK,
        "kernel_ms_avg": kernel_s * 1e3,
        "kernel_ms_min": float(np.min(kernel_ms)),
        "kernel_ms_median": float(np.median(kernel_ms)),
        "clock_warmup_ms": CLOCK_WARMUP_MS,
        "algorithmic_bytes": algo_bytes,
        "flops": 2.0 * F * K * n_rows,
        "traffic": (MEASURED_TRAFFIC.get(args.workload) or {}).get("bytes"),
        "traffic_source": ({k: MEASURED_TRAFFIC[args.workload][k] for k in ("profile", "commit")}
                           if args.workload in MEASURED_TRAFFIC else None),
    }
    cpu_baseline = None
    parity = None
    if not args.no_cpu_baseline:
        from oracle.linear_oracle import predict_linear
        t1 = time.perf_counter()
        ref = predict_linear(w.model, x_sample)
        dt = time.perf_counter() - t1
        cpu_baseline = {"value": sample_rows / dt, "unit": "rows/s", "cores": os.cpu_count() or 1,
                        "kind": "oracle", "sample": f"first {sample_rows} rows of {args.workload}, one pass "
                                                    "(numpy float64 matmul, its BLAS threads)"}
        parity = {"rows_checked": sample_rows}
        if scores is not None:
            got = scores[:sample_rows].cpu().numpy()
            err = np.abs(got - ref.scores)
            parity["scores_within_tol"] = bool((err <= 1e-6 + 1e-5 * np.abs(ref.scores)).all())
            parity["max_abs_err"] = float(err.max())
        if labels is not None:
            parity["labels_equal"] = bool((labels[:sample_rows].cpu().numpy() == ref.labels).all())
    line = {
        "metric": "rows/sec scored (fp32 X), 1 MI355X",
        "value": n_rows * args.steps / wall,
        "unit": "rows/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64 products and sums of f32 inputs, rounded to f32 once",
        "data": "synthetic (seeded; stands in for the paper's linear models on YearPrediction)",
        "config": {"workload": args.workload, "n_rows": n_rows, "n_features": F, "n_outputs": K},
        "roofline": roofline,
        "cpu_baseline": cpu_baseline,
        "parity": parity,
    }
    print(json.dumps(line))
    m.close()
    return 0


def _host_threads() -> int:
    return max(1, min(os.cpu_count() or 1, ORACLE_THREADS_MAX))


def _time_oracle(forest, X, threads: int, passes: int = 3):
    """One warm-up pass, then `passes` timed passes over all of X; returns (median seconds, result)."""
    import oracle
    ref = oracle.predict(forest, X, n_threads=threads)
    times = []
    for _ in range(passes):
        t0 = time.perf_counter()
        ref = oracle.predict(forest, X, n_threads=threads)
        times.append(time.perf_counter() - t0)
    return sorted(times)[len(times) // 2], ref


def hbm_copy_rate() -> float:
    """Bytes moved per second by a plain device-to-device copy of 1 GiB (read + write), the memory
    system's own rate for a streaming kernel on this machine; reported next to the nominal peak."""
    import torch
    n = 1 << 28
    a = torch.empty(n, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    a.fill_(1.0)
    for _ in range(2):
        b.copy_(a)
    torch.cuda.synchronize()
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(5):
        b.copy_(a)
    stop.record()
    torch.cuda.synchronize()
    return 5 * 2 * 4.0 * n / (start.elapsed_time(stop) * 1e-3)


def compare_issue_rate() -> float:
    """(row, node) comparisons per second of a kernel that only issues the rank kernels' packed-f16
    compare instruction (eight wavefronts per SIMD, sixteen independent chains per lane): what the
    chip delivers where the roofline quotes 256 CU x 4 SIMD x 16 lanes x 2.4 GHz x 2."""
    import torch
    from paper_2301_13441_amd import binding
    word = torch.zeros(1, dtype=torch.int32, device="cuda")
    binding.forest_probe_compare_rate(1000, word)
    torch.cuda.synchronize()
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    n = binding.forest_probe_compare_rate(20000, word)
    stop.record()
    torch.cuda.synchronize()
    return n / (start.elapsed_time(stop) * 1e-3)


def _mean_path_tests(forest, leaves) -> float:
    """Tests on a row's paths through all trees, averaged over the rows of `leaves` ([rows, trees])."""
    import numpy as np
    offset = np.asarray(forest.tree_offset)
    depth = np.zeros(int(offset[-1]), np.int64)
    tree_of = np.repeat(np.arange(len(offset) - 1), np.diff(offset))
    at = offset[:-1].copy()
    level = 0
    while len(at):
        depth[at] = level
        at = at[np.asarray(forest.feature)[at] >= 0]
        base = offset[tree_of[at]]
        at = np.concatenate([base + forest.left[at], base + forest.right[at]])
        level += 1
    return float(depth[offset[:-1][None, :] + leaves].sum(axis=1).mean())


class ForestRun:
    """One tree-ensemble configuration, measured in three steps so that the GPU timing of several
    configurations can run back to back: prepare (model and X to the device), time (W warm-up and
    K timed forest_predict calls), finish (oracle baseline, parity, the result fields)."""

    def __init__(self, name: str, args):
        import numpy as np
        import torch

        import paper_2301_13441_amd as pk
        import workloads as wl
        from paper_2301_13441_amd.binding import forest_launch

        self.name, self.args = name, args
        self.w = wl.make_workload(name, n_rows=args.rows)
        self.n_rows, self.F = self.w.n_rows, self.w.forest.n_features
        self.f = pk.forest_load(self.w.forest)
        self.info = self.f.info
        self.launch = forest_launch(self.f, self.n_rows)
        # X: generated on the host in chunks, copied to HBM before the timed region; the host copy
        # is kept for the oracle
        self.want_host = not args.no_cpu_baseline
        self.xd = torch.empty((self.n_rows, self.F), dtype=torch.float32, device="cuda")
        self.xh = np.empty((self.n_rows, self.F), dtype=np.float32) if self.want_host else None
        pos = 0
        for chunk in self.w.x_chunks(self.n_rows):
            self.xd[pos:pos + len(chunk)].copy_(torch.from_numpy(chunk))
            if self.want_host:
                self.xh[pos:pos + len(chunk)] = chunk
            pos += len(chunk)
        self.out = torch.empty(max(self.f.out_bytes(self.n_rows), 4), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()

    def time(self):
        import torch
        args = self.args
        stream = torch.cuda.current_stream()   # forest_predict is enqueued on this stream
        for _ in range(args.warmup):
            self.f.predict(self.xd, out=self.out)
        torch.cuda.synchronize()
        starts = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
        stops = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
        t0 = time.perf_counter()
        for i in range(args.steps):
            starts[i].record(stream)
            self.f.predict(self.xd, out=self.out)
            stops[i].record(stream)
        torch.cuda.synchronize()
        self.wall = time.perf_counter() - t0
        self.kernel_ms = [a.elapsed_time(b) for a, b in zip(starts, stops)]

    def finish(self) -> dict:
        import numpy as np
        import torch
        args, name, info, n_rows, F, f = self.args, self.name, self.info, self.n_rows, self.F, self.f
        kernel_ms, wall = self.kernel_ms, self.wall
        kernel_s = float(np.mean(kernel_ms)) * 1e-3
        scores, labels = f.predict(self.xd, out=self.out)
        torch.cuda.synchronize()

        sample = f.predict_leaves(self.xd[:4096]).cpu().numpy()
        tests = _mean_path_tests(self.w.forest, sample)
        achieved = tests * n_rows / kernel_s
        algo_bytes = n_rows * (4.0 * F) + f.out_bytes(n_rows)
        traffic = MEASURED_TRAFFIC.get(name) if args.rows is None else None
        roofline = {
            "bound": "lds",
            "kernel": "forest_predict (walk of the row's paths + reduction)",
            "achieved": achieved / 1e12,
            "peak": LDS_PEAK_TESTS / 1e12,
            "unit": "Ttest/s",
            "frac": achieved / LDS_PEAK_TESTS,
            "peak_basis": "256 CU x 2.4 GHz x 64 rows per 4 clocks (two LDS reads of 2 clocks per test)",
            "tests_per_row": tests,
            "kernel_ms_avg": kernel_s * 1e3,
            "kernel_ms_min": float(np.min(kernel_ms)),
            "kernel_ms_median": float(np.median(kernel_ms)),
            "algorithmic_bytes": algo_bytes,
            "hbm_GBps": algo_bytes / kernel_s / 1e9,
            "hbm_frac": algo_bytes / kernel_s / HBM_PEAK,
            "traffic": traffic["bytes"] if traffic else None,
            "traffic_source": ({k: traffic[k] for k in ("profile", "commit")} if traffic else None),
        }

        cpu_baseline = None
        parity = None
        if self.want_host:
            threads = _host_threads()
            dt, ref = _time_oracle(self.w.forest, self.xh, threads)
            cpu_baseline = {"value": n_rows / dt, "unit": "rows/s", "cores": threads, "kind": "oracle",
                            "host_cpu_count": os.cpu_count(),
                            "sample": f"all {n_rows} rows of {name}: one warm-up pass, median of 3 timed passes, "
                                      f"{threads} threads over contiguous row blocks"}
            parity = {"rows_checked": n_rows}
            if scores is not None:
                got = scores.cpu().numpy()
                err = np.abs(got - ref.scores)
                parity["scores_within_tol"] = bool((err <= 1e-6 + 1e-5 * np.abs(ref.scores)).all())
                parity["max_abs_err"] = float(err.max())
            if labels is not None:
                parity["labels_equal"] = bool((labels.cpu().numpy() == ref.labels).all())
            if name == "c1":   # the small configuration also on one thread
                dt1, _ = _time_oracle(self.w.forest, self.xh, 1)
                cpu_baseline["one_thread_value"] = n_rows / dt1

        res = {
            "value": n_rows * args.steps / wall,
            "ms_per_step": wall / args.steps * 1e3,
            "dtype": "f32 compare, f64 accumulate",
            "config": {"workload": name, "n_rows": n_rows, "n_features": F,
                       "n_trees": info["n_trees"], "max_depth": info["max_depth"],
                       "n_internal_nodes": info["n_internal"], "n_outputs": info["n_outputs"],
                       "kernel": self.launch["kernel"], "rows_per_workgroup": self.launch["rows_per_workgroup"],
                       "packed_bytes": info["packed_bytes"]},
            "roofline": roofline,
            "cpu_baseline": cpu_baseline,
            "parity": parity,
        }
        f.close()
        self.xd = self.out = self.xh = None
        del scores, labels
        torch.cuda.empty_cache()
        return res


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default=None, choices=["c1", "c2", "c3", "c4", "c5", "l1", "l2", "l3", "l4"],
                    help="one configuration only (c1..c5: tree ensembles; l1..l4: linear models); "
                         "default: c5 as the headline and c4, c3, c2, c1 under per_config")
    ap.add_argument("--rows", type=int, default=None, help="override the row count (testing)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU; --gpus must be 1 "
              "(rows are independent: more GPUs = shard X by rows, replicate the packed model)",
              file=sys.stderr)
        return 2

    import torch

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 2
    torch.cuda.set_device(0)
    if args.workload is not None and args.workload.startswith("l"):
        return bench_linear(args)

    names = [args.workload] if args.workload else ["c5", "c4", "c3", "c2", "c1"]
    # Every configuration is set up first (model and X on the device), then the configurations are
    # timed one right after the other -- W warm-up and K timed calls each, nothing but a
    # synchronisation between them, so the clocks the first one has raised stay up for the short
    # ones (after an idle gap the first 25 ms or so of kernel time run up to 15 % slower) -- and the
    # CPU oracle is timed and compared afterwards.
    runs = []
    for name in names:
        print(f"bench: setting up {name} ...", file=sys.stderr, flush=True)
        runs.append(ForestRun(name, args))
    for r in runs:
        r.time()
    results = {}
    for r in runs:
        print(f"bench: oracle and parity of {r.name} ...", file=sys.stderr, flush=True)
        results[r.name] = r.finish()
    head = results[names[0]]
    line = {
        "metric": "rows/sec scored (fp32 X), 1 MI355X",
        "value": head["value"],
        "unit": "rows/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": head["dtype"],
        "data": "synthetic (seeded; stands in for YearPrediction and the paper's unstated models)",
        "config": head["config"],
        "roofline": head["roofline"],
        "cpu_baseline": head["cpu_baseline"],
        "parity": head["parity"],
    }
    if len(names) > 1:
        per = {}
        for name in names[1:]:
            r = results[name]
            if name == "c1":
                # 1,000 rows: bound by the launch, so a latency and no roofline claim
                per[name] = {"latency_us_per_call": r["roofline"]["kernel_ms_avg"] * 1e3,
                             "latency_us_min": r["roofline"]["kernel_ms_min"] * 1e3,
                             "value": r["value"], "unit": "rows/s", "config": r["config"],
                             "cpu_baseline": r["cpu_baseline"], "parity": r["parity"]}
            else:
                per[name] = {k: r[k] for k in ("value", "ms_per_step", "dtype", "config", "roofline",
                                               "cpu_baseline", "parity")}
                per[name]["unit"] = "rows/s"
        line["per_config"] = per
        line["measured_peaks"] = {"hbm_copy_GBps": hbm_copy_rate() / 1e9,
                                  "packed_f16_compare_Tps": compare_issue_rate() / 1e12,
                                  "note": "device-to-device copy of 1 GiB, bytes read + written; a kernel of "
                                          "nothing but v_pk_fma_f16 ... clamp, two comparisons per lane-op"}
    print(json.dumps(line))
    return 0


if __name__ == "__main__":
    sys.exit(main())
