"""Benchmark: asynchronous SCD epochs on one MI355X, oracle timed beside it.

One step = one epoch of the hot path (permutation, gather-dot, reduction, closed-form step,
atomic scatter) followed by one evaluation of the duality gap, i.e. one iteration of a
train-until-gap loop.  The gap of step k is read on the host while epoch k+1 runs (two
asynchronous evaluation slots), as a training loop that checks convergence every epoch would.
Prints ONE JSON line.

The default workload is the largest single-GPU one: the click-log hinge SVM dual (50 M examples x
75 M features, 1.95 B stored entries, one of four workers' shares of a criteo-like data set).

    python bench.py [--gpus 1] [--steps 20] [--warmup 5] [--workload click_svm]
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "time to duality gap 1e-3 (s); nnz processed/sec per SCD epoch; HBM GB/s, 1 GPU"
HBM_PEAK_GBS = 8000.0

# Workloads (full sizes).  The default bench line is the click-log workload, the largest that one GPU
# holds; the others are measured with --workload NAME.
WORKLOADS = {
    "sparse_ridge": ("sparse_ridge_100000x50000_d1e-3", {}),
    "dense_ridge": ("dense_ridge_2000x200", {}),
    "text_svm": ("text_svm_350000x16600000_3700perrow", {}),
    "text_ridge_csc": ("text_ridge_csc_350000x16600000_3700perrow", {}),
    "click_svm": ("click_svm_50000000x75000000_39perrow", {}),
}


def algorithmic_bytes(prob) -> int:
    """Bytes one epoch must move (the roofline's numerator).  Per stored entry: 4 B index + 4 B
    value read once, a 4 B atomic update of the shared vector, and the gathers the step needs:
    4 B of the shared vector for the duals, 8 B (shared vector and label) for the ridge primal,
    whose step reads y - w at every row.  Per coordinate: 8 B of ptr, 4 B norm, 4 B model read and
    4 B model write, plus a 4 B label for the duals.  So 16 B per entry + 24 B per coordinate for
    the duals, 20 + 20 for the ridge primal."""
    if prob.form == "ridge_primal":
        return 20 * prob.nnz + 20 * prob.C
    return 16 * prob.nnz + 24 * prob.C


def kernel_sources() -> list:
    """Every file the library is compiled from: its sources and their headers."""
    import glob

    from paper_1702_07005_amd import build

    return [*build.SOURCES, *sorted(glob.glob(os.path.join(build.CSRC, "*.h")))]


def kernel_source_hash() -> str:
    h = hashlib.sha256()
    for path in kernel_sources():
        with open(path, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(workload: str):
    """HBM bytes per epoch launch from the committed rocprofv3 counter summary, if it was
    taken on the current kernel sources; else None."""
    path = os.path.join(ROOT, "profiles", f"epoch_{workload}_traffic.json")
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        t = json.load(fh)
    if t.get("kernel_source_hash") != kernel_source_hash():
        return None
    return t.get("hbm_bytes_per_launch")


def device_ceilings(L: int):
    """Live device-wide rates on this GPU (libscdprobe.so): scattered fp32 atomic adds into an array
    the size of the shared vector; independent gathers from and atomic adds into that array (pairs
    per second), packed and with one entry per 64 bytes (the spread copy, for up to 4 M entries);
    and a 1 GiB streaming copy."""
    import ctypes
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_1702_07005_amd", "libscdprobe.so"))
    lib.scd_probe_rate.argtypes = [ctypes.c_int, ctypes.c_uint64, ctypes.c_void_p, ctypes.POINTER(ctypes.c_double)]
    out = {}
    n = max(L, 1024)
    modes = [(0, "atomic_adds_per_s", n), (1, "gather_and_atomic_pairs_per_s", n)]
    if n <= (1 << 22):
        modes.append((3, "gather_and_atomic_pairs_spread_per_s", n))
    modes.append((2, "copy_bytes_per_s", 1 << 28))
    for mode, key, n in modes:
        v = ctypes.c_double()
        rc = lib.scd_probe_rate(mode, n, None, ctypes.byref(v))
        out[key] = v.value if rc == 0 else None
    return out


def cpu_baseline(prob, budget_s: float, seed: int, f32_budget_s: float = 0.0):
    """The fp64 sequential oracle on the host, same workload from the zero state, run for
    whole epochs until about `budget_s` seconds of epoch time have elapsed (at least one
    epoch).  The duality gap after each epoch is evaluated outside the timed epochs.  With
    `f32_budget_s` > 0, the oracle's single-precision copy of the epochs is timed the same way
    and reported as `fp32_sequential`."""
    import numpy as np
    from oracle import oracle as orc

    model = np.zeros(prob.C)
    shared = np.zeros(prob.L)
    epochs = 0
    el = 0.0
    curve = []
    ttg = None
    # One core, pinned: the oracle is sequential by definition.
    allowed = sorted(os.sched_getaffinity(0))
    os.sched_setaffinity(0, {allowed[0]})
    while True:
        t0 = time.perf_counter()
        orc.epochs(prob.form, prob.n_rows, prob.n_cols, prob.ptr, prob.idx, prob.val, prob.y, prob.lam, seed, epochs,
                   1, model, shared)
        el += time.perf_counter() - t0
        epochs += 1
        g = orc.objectives(prob.form, prob.n_rows, prob.n_cols, prob.ptr, prob.idx, prob.val, prob.y, prob.lam,
                           model, shared)[2]
        curve.append(g)
        if ttg is None and g <= 1e-3:
            ttg = (epochs, el)
        if el >= budget_s or epochs >= 1000:
            break
    # The same sequential epochs in single precision, the precision of the paper's one-thread
    # baseline, on the same core and a shorter budget.
    f32 = None
    if f32_budget_s > 0:
        m32 = np.zeros(prob.C, dtype=np.float32)
        s32 = np.zeros(prob.L, dtype=np.float32)
        e32, el32, ttg32, curve32 = 0, 0.0, None, []
        while True:
            t0 = time.perf_counter()
            orc.epochs_f32(prob.form, prob.n_rows, prob.n_cols, prob.ptr, prob.idx, prob.val, prob.y, prob.lam, seed,
                           e32, 1, m32, s32)
            el32 += time.perf_counter() - t0
            e32 += 1
            g = orc.objectives(prob.form, prob.n_rows, prob.n_cols, prob.ptr, prob.idx, prob.val, prob.y, prob.lam,
                               m32.astype(np.float64))[2]
            curve32.append(g)
            if ttg32 is None and g <= 1e-3:
                ttg32 = (e32, el32)
            if el32 >= f32_budget_s or e32 >= 1000:
                break
        f32 = {"value": prob.nnz * e32 / el32, "unit": "nnz/s", "epochs_per_s": e32 / el32,
               "sample": f"{e32} sequential fp32 epochs from the zero state ({el32:.1f} s of epoch time, same core)",
               "time_to_gap_1e-3_s": ttg32[1] if ttg32 else None, "epochs_to_gap_1e-3": ttg32[0] if ttg32 else None,
               "gap_curve": [float(f"{g:.3e}") for g in curve32[:12]]}
    os.sched_setaffinity(0, set(allowed))
    cpu = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            cpu = next((ln.split(":", 1)[1].strip() for ln in fh if ln.startswith("model name")), cpu)
    except OSError:
        pass
    return {"value": prob.nnz * epochs / el, "unit": "nnz/s", "cores": 1, "kind": "oracle",
            "sample": f"{epochs} sequential fp64 epochs of the same workload from the zero state "
                      f"({el:.1f} s of epoch time on one host thread, pinned to core {allowed[0]})",
            "cpu_model": cpu, "host_cores_visible": len(allowed),
            "epochs_per_s": epochs / el,
            "time_to_gap_1e-3_s": ttg[1] if ttg else None, "epochs_to_gap_1e-3": ttg[0] if ttg else None,
            "gap_curve": [float(f"{g:.3e}") for g in curve[:12]], "fp32_sequential": f32}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="click_svm", choices=sorted(WORKLOADS))
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--cpu-f32-seconds", type=float, default=8.0,
                    help="budget of the single-precision sequential epochs timed beside the oracle (0: skip)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--max-gap-epochs", type=int, default=200)
    ap.add_argument("--gap-seconds", type=float, default=10.0,
                    help="after the gap has reached 1e-3, stop the time-to-gap run once this much epoch time "
                         "has been spent (it always stops at gap 1e-6)")
    ap.add_argument("--gap-limit-seconds", type=float, default=120.0,
                    help="stop the time-to-gap run after this much epoch time even if the gap is above 1e-3")
    ap.add_argument("--ablation", action="store_true",
                    help="before the timed steps, run the frozen gather-dot kernel (no scatter) three times, for "
                         "attributing L2 counters: stream only (set-up norms), gathers only, full epoch")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="after the timed steps, run a plain 1 GiB device-to-device copy twice (a kernel of known "
                         "traffic for scaling rocprofv3 FETCH_SIZE/WRITE_SIZE counters)")
    args = ap.parse_args()

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print(f"bench.py measures one GPU only (asked for --gpus {args.gpus}, WORLD_SIZE={world}); "
              "the solver has no multi-GPU path.", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from paper_1702_07005_amd import scd, synth

    name, over = WORKLOADS[args.workload]
    print(f"# generating {name}", file=sys.stderr, flush=True)
    prob = synth.make(args.workload, seed=args.seed, **over)
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    stream = torch.cuda.current_stream()
    solver = scd.solver_for(prob, device=dev)
    info = solver.info()
    # A pipelined plan may run on the spread copy of the shared vector, copied out and back inside each
    # scd_epochs call.
    spread = solver.get_option("next_spread") == 1
    zeros_m = torch.zeros(prob.C, dtype=torch.float32, device=dev)
    zeros_s = torch.zeros(prob.L, dtype=torch.float32, device=dev)

    def reset():
        solver.set_state(zeros_m, zeros_s, 0)

    # --- time to duality gap (epoch kernels only, gap evaluation excluded) ------------------
    # One untimed epoch first: the first launch of a kernel in a process also loads its code
    # object, which is not part of an epoch's cost.
    print("# time to gap", file=sys.stderr, flush=True)
    solver.epochs(args.seed, 1)
    torch.cuda.synchronize()
    reset()
    gap0 = solver.duality_gap()
    P0, _ = solver.objective()
    t_epochs = 0.0
    hits = {}
    curve = []
    for e in range(args.max_gap_epochs):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        solver.epochs(args.seed, 1)
        b.record(stream)
        g = solver.duality_gap()
        t_epochs += a.elapsed_time(b) / 1e3
        curve.append(g)
        print(f"#   epoch {e + 1}: gap {g:.3e}, {t_epochs:.3f} s of epochs", file=sys.stderr, flush=True)
        for thr in (1e-3, 1e-6):
            if thr not in hits and g <= thr:
                hits[thr] = (e + 1, t_epochs)
        if 1e-6 in hits or t_epochs >= args.gap_limit_seconds:
            break
        if 1e-3 in hits and t_epochs >= args.gap_seconds:
            break

    if args.ablation:
        _, shared_now, _ = solver.get_state()
        for _ in range(3):
            solver.gather_dots(shared_now)
        torch.cuda.synchronize()

    # --- timed steps ------------------------------------------------------------------------
    reset()
    for _ in range(args.warmup):
        solver.epochs(args.seed, 1)
        solver.duality_gap()
    starts = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    step_gaps = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        starts[k].record(stream)
        solver.epochs(args.seed, 1)
        ends[k].record(stream)
        solver.duality_gap_async(k % 2)
        if k > 0:
            step_gaps.append(solver.duality_gap_wait((k - 1) % 2)[0])
    step_gaps.append(solver.duality_gap_wait((args.steps - 1) % 2)[0])
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    epoch_s = np.array([s.elapsed_time(e) / 1e3 for s, e in zip(starts, ends)])
    epoch_avg = float(epoch_s.mean())

    alg = algorithmic_bytes(prob)
    achieved = alg / epoch_avg / 1e9
    traffic = measured_traffic(args.workload)
    out = {
        "metric": METRIC,
        "value": prob.nnz * args.steps / wall,
        "unit": "nnz/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": name, "formulation": prob.form, "layout": prob.layout, "n_rows": prob.n_rows,
                   "n_cols": prob.n_cols, "nnz": prob.nnz, "lambda": prob.lam, "seed": args.seed,
                   "group_lanes": info["group_lanes"], "window": info["window"]},
        "epoch_ms": epoch_avg * 1e3,
        "epoch_nnz_per_s": prob.nnz / epoch_avg,
        "epochs_per_s": 1.0 / epoch_avg,
        "gap_eval_ms": (wall / args.steps - epoch_avg) * 1e3,
        "gap_after_timed_steps": step_gaps[-1],
        "time_to_gap_1e-3_s": hits[1e-3][1] if 1e-3 in hits else None,
        "epochs_to_gap_1e-3": hits[1e-3][0] if 1e-3 in hits else None,
        "time_to_gap_1e-6_s": hits[1e-6][1] if 1e-6 in hits else None,
        "epochs_to_gap_1e-6": hits[1e-6][0] if 1e-6 in hits else None,
        "gap_at_zero": gap0,
        "primal_at_zero": P0,
        "gap_curve": [float(f"{g:.3e}") for g in curve[:12]],
        "gap_epochs_run": len(curve),
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "algorithmic_bytes_per_launch": alg,
                     "kernel": f"scd::k_epoch_* ({info['kernel']}); timed: one scd_epochs call of one epoch"
                               + (", with its two k_spread copies" if spread else "")},
    }
    solver.close()
    ceil = device_ceilings(prob.L)
    if traffic is not None:
        # Measured HBM bytes (rocprofv3 counters, copy-calibrated) over the live epoch time.
        tg = traffic / epoch_avg / 1e9
        out["roofline"]["traffic_GBps"] = tg
        out["roofline"]["traffic_frac_of_peak"] = tg / HBM_PEAK_GBS
        if ceil["copy_bytes_per_s"]:
            out["roofline"]["traffic_frac_of_copy"] = tg * 1e9 / ceil["copy_bytes_per_s"]
    if ceil["atomic_adds_per_s"]:
        # The scatter issues one device-scope atomic per stored entry.
        rate = prob.nnz / epoch_avg
        frac = rate / ceil["atomic_adds_per_s"]
        out["atomic_roofline"] = {"bound": "device-scope fp32 atomics", "achieved": rate,
                                  "peak": ceil["atomic_adds_per_s"], "unit": "atomic adds/s",
                                  "frac": frac,
                                  # every atomic is resolved beyond L2 at any scope, so this rate, not
                                  # HBM bandwidth, binds an epoch that runs near it
                                  "binding": frac >= 0.5,
                                  "gather_and_atomic_pairs_per_s": ceil["gather_and_atomic_pairs_per_s"],
                                  "gather_and_atomic_pairs_spread_per_s":
                                      ceil.get("gather_and_atomic_pairs_spread_per_s"),
                                  "copy_GBps": (ceil["copy_bytes_per_s"] or 0) / 1e9}
    if args.calibrate_copy:
        src = torch.ones(1 << 28, dtype=torch.float32, device=dev)  # 1 GiB
        dst = torch.empty_like(src)
        for _ in range(2):
            dst.copy_(src)
        torch.cuda.synchronize()
        out["calibration_copy_bytes"] = src.numel() * 4
        del src, dst
    # Release every device object this process made before the host leg and the exit: the solver is
    # closed above; the state tensors, events and the caching allocator's blocks go here.
    del zeros_m, zeros_s, starts, ends
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    if not args.no_cpu_baseline:
        print("# oracle on the host", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(prob, args.cpu_seconds, args.seed, args.cpu_f32_seconds)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
