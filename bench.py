#!/usr/bin/env python3
"""Truth-table enumeration benchmark on one MI355X.

One step = the whole hot path over one batch of synthetic neurons:
batched enumeration (persistent, autotuned launch: prep + enumeration
kernels, the histogram counted inside the enumeration kernel) followed by
the input support of the packed tables.  The
default workload is 512 neurons with F=8 inputs of b=3 bits (2^24 rows each,
2-bit outputs, 2 GiB of packed tables), the largest single-GPU shape.

Prints ONE JSON line.  `value` is row-evaluations per second of the whole
step with inputs resident in HBM.  `roofline` is the enumeration kernel's
achieved HBM write bandwidth (algorithmic bytes: the packed tables) over its
HIP-event duration.  `cpu_baseline` times the CPU oracle on a bounded sample
of the same neurons and checks the GPU tables of that sample bit for bit.
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

HBM_PEAK_GBS = 8000.0
MFMA_I8_PEAK_TOPS = 5000.0  # dense int8, TOP/s
TUNE_CACHE = os.path.join(ROOT, "paper_2502_08673_amd", "tune_cache.txt")
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "enum_wide_kernel_cfg3_traffic.txt")
ENUM_SRC = os.path.join(ROOT, "paper_2502_08673_amd", "csrc", "tt_enum.hip")
NET_TRAFFIC_FILE = os.path.join(ROOT, "profiles", "lutnet_packed_kernel_cfg1net_traffic.txt")
NET_SQ_FILE = os.path.join(ROOT, "profiles", "lutnet_packed_kernel_cfg1net_sq.txt")
CNF_SQ_FILE = os.path.join(ROOT, "profiles", "cnf_fast_kernel_cnf_sq.txt")
GD_SQ_FILE = os.path.join(ROOT, "profiles", "gd_compiled_kernel_gd_sq.txt")
GD_INTERP_SQ_FILE = os.path.join(ROOT, "profiles", "gd_sample_kernel_gd_sq.txt")
CSRC = os.path.join(ROOT, "paper_2502_08673_amd", "csrc")
# VALU issue peak of MI355X: 256 CUs x 4 SIMDs x 2.4 GHz, one wave64 VALU
# instruction per SIMD every 4 cycles (16 lanes per cycle; packed fp32 is not
# used) = 614.4 G wave instructions/s, i.e. 78.6 TFLOP/s of fp32 FMA.
VALU_PEAK_INSTR_S = 256 * 4 * 2.4e9 / 4
NET_SRC = os.path.join(ROOT, "paper_2502_08673_amd", "csrc", "tt_lutnet.hip")

WORKLOADS = {
    "cfg3": "512 neurons, F=8, b=3 (2^24 rows each), o=2, w=clip(round(N(0,4)),+-15), bias U{-8..8}, "
            "T={4,8,12}, ReLU; 2 GiB packed tables",
    "cfg2": "8192 uneven neurons, F in 3..8, b in 1..3 (F*b<=16), o in 1..3, 30% zero weights",
    "cfg1": "448 neurons (256-128-64 sparse MLP), F=6, b=2, o=2",
    "cfg0": "64 neurons, F=6, b=2, o=2",
}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="cfg3", choices=sorted(WORKLOADS) + ["cfg4", "cfg1net", "cnf", "gd"])
    ap.add_argument("--samples", type=int, default=1 << 18, help="cfg1net: input samples per step")
    ap.add_argument("--batch", type=int, default=1 << 20, help="gd: samples per step")
    ap.add_argument("--instances", type=int, default=32768,
                    help="cnf: CNF instances per step (8192 distinct ones, repeated)")
    ap.add_argument("--epochs", type=int, default=40, help="cfg4: screen training epochs")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=10.0, help="target CPU time of the oracle sample")
    ap.add_argument("--no-tune", action="store_true", help="default launch configuration")
    ap.add_argument("--only", choices=["step", "enumerate", "support-scan"],
                    help="cfg0-cfg3: run only this part (warmup + steps calls) and print its time; for profiles")
    ap.add_argument("--tune-cache", default=TUNE_CACHE, help="autotuner cache file (read, appended to)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain 1 GiB device copy (reference for HBM counters)")
    return ap.parse_args()


def source_hash(path: str) -> str:
    import hashlib
    return hashlib.sha256(open(path, "rb").read()).hexdigest()[:16]


def read_sq(path: str, src: str):
    """Per-dispatch SQ counters of a kernel from its committed rocprofv3
    summary, if it was taken on this kernel source (else None)."""
    if not os.path.exists(path):
        return None
    kv = {}
    for line in open(path):
        if ":" in line and not line.lstrip().startswith("#"):
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    if kv.get("kernel_source_sha256_16") != source_hash(src):
        return None
    return kv


def alu_roofline(kernel: str, kernel_ms: float, sq):
    """Instruction-rate roofline: VALU wave instructions per launch (from the
    counter summary) over the kernel's time, against the VALU issue peak."""
    valu = float(sq["sq_insts_valu_per_dispatch"]) if sq else None
    achieved = valu / (kernel_ms * 1e-3) if valu else None
    return {"bound": "alu", "kernel": kernel, "achieved": achieved, "peak": VALU_PEAK_INSTR_S,
            "unit": "VALU wave instructions/s", "frac": achieved / VALU_PEAK_INSTR_S if achieved else None,
            "traffic": None, "kernel_ms": kernel_ms,
            "salu_per_launch": float(sq["sq_insts_salu_per_dispatch"]) if sq else None,
            "valu_per_launch": valu}


def read_traffic(words_bytes: float, path: str = TRAFFIC_FILE, src: str = ENUM_SRC):
    """Measured HBM bytes per launch of a kernel, from its committed
    rocprofv3 counter summary, if it was taken on this kernel source and on a
    workload with the same algorithmic bytes (else None)."""
    if not os.path.exists(path):
        return None
    kv = {}
    for line in open(path):
        if ":" in line and not line.lstrip().startswith("#"):
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    if kv.get("kernel_source_sha256_16") != source_hash(src):
        return None
    try:
        if int(kv["algorithmic_bytes_per_launch"]) != int(words_bytes):
            return None
        return float(kv["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def main():
    args = parse()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py measures one GPU: the enumeration shards across GPUs without any exchange, "
              "so its throughput is measured on a single MI355X (use --gpus 1).", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2502_08673_amd as tt
    import workloads

    torch.cuda.set_device(0)
    tt.device_check()
    if args.workload == "cfg4":
        print(json.dumps(bench_screen(args)), flush=True)
        return
    if args.workload == "cfg1net":
        print(json.dumps(bench_lutnet(args)), flush=True)
        return
    if args.workload == "cnf":
        print(json.dumps(bench_cnf(args)), flush=True)
        return
    if args.workload == "gd":
        print(json.dumps(bench_gd(args)), flush=True)
        return
    ns = {"cfg0": workloads.cfg0, "cfg1": workloads.cfg1, "cfg2": workloads.cfg2, "cfg3": workloads.cfg3}[
        args.workload]()
    n = len(ns)
    rows = ns.total_rows()
    desc = tt.descriptors(ns)
    total = tt.layout(desc)
    table_bytes = 8.0 * total
    tables = torch.empty(total, dtype=torch.int64, device="cuda")
    hist = torch.zeros(n * 8, dtype=torch.int32, device="cuda")
    sup = torch.zeros(n, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream()

    tune = None if args.no_tune else tt.autotune(desc, tables, cache_path=args.tune_cache)
    plan = tt.Plan(desc, total, tune=tune, flags=tt.TT_PLAN_PERSISTENT | tt.TT_PLAN_TIMING)
    info = plan.info()

    def step():
        # enumeration with the fused histogram, then the support of the plan's
        # own tables (decided from the neurons' parameters, no table read)
        plan.step(tables, hist, sup, stream)

    if args.only:
        fn = {"step": step, "enumerate": lambda: plan.launch(tables, hist, stream),
              "support-scan": lambda: plan.support(tables, support_out=sup, stream=stream)}[args.only]
        for _ in range(args.warmup):
            fn()
        torch.cuda.synchronize()
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        a.record(stream)
        for _ in range(args.steps):
            fn()
        b.record(stream)
        torch.cuda.synchronize()
        plan.close()
        print(json.dumps({"only": args.only, "workload": args.workload, "calls": args.steps,
                          "ms_per_call": a.elapsed_time(b) / args.steps, "tune": info}), flush=True)
        return

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    plan.kernel_times_ms()  # drop warm-up timings
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    wall0 = time.perf_counter()
    e0.record(stream)
    for _ in range(args.steps):
        step()
    e1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - wall0
    step_ms = e0.elapsed_time(e1) / args.steps
    kms = plan.kernel_times_ms()
    kernel_ms = float(np.mean(kms)) if kms else float("nan")

    # enumeration alone (batched, the plan above) and the plain one-shot path
    def timed(fn, reps):
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        fn()
        torch.cuda.synchronize()
        a.record(stream)
        for _ in range(reps):
            fn()
        b.record(stream)
        torch.cuda.synchronize()
        return a.elapsed_time(b) / reps

    def queued(fn, reps):
        # GPU time alone: the launches are queued behind a ~20 ms spin, so the
        # host's issue rate does not gate them
        fn()
        torch.cuda.synchronize()
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        torch.cuda._sleep(50_000_000)
        a.record(stream)
        for _ in range(reps):
            fn()
        b.record(stream)
        torch.cuda.synchronize()
        return a.elapsed_time(b) / reps

    reps = max(3, min(args.steps, 10))
    batched_ms = timed(lambda: plan.launch(tables, None, stream), reps)
    batched_hist_ms = timed(lambda: plan.launch(tables, hist, stream), reps)
    support_only_ms = timed(lambda: plan.support(tables, support_out=sup, stream=stream), reps)
    support_enum_ms = timed(lambda: plan.support_enumerated(tables, support_out=sup, stream=stream), reps)
    plain_ms = timed(lambda: tt.enumerate(desc, tables, total_words=total, stream=stream), reps)
    # the step without the kernel-timing events, eager and replayed from one
    # captured hipGraph; host-paced (as issued) and GPU-only (queued)
    sreps = 200 if step_ms < 0.2 else reps
    with tt.Plan(desc, total, tune=tune, flags=tt.TT_PLAN_PERSISTENT) as eplan:
        step_eager_ms = timed(lambda: eplan.step(tables, hist, sup, stream), sreps)
        step_eager_queued_ms = queued(lambda: eplan.step(tables, hist, sup, stream), sreps)
    with tt.Plan(desc, total, tune=tune, flags=tt.TT_PLAN_PERSISTENT | tt.TT_PLAN_GRAPH) as gplan:
        graph_ms = timed(lambda: gplan.launch(tables, hist, stream), reps)
        step_graph_ms = timed(lambda: gplan.step(tables, hist, sup, stream), sreps)
        step_graph_queued_ms = queued(lambda: gplan.step(tables, hist, sup, stream), sreps)
    support_ms = timed(lambda: plan.support(tables, support_out=sup, hist=hist, stream=stream), reps)
    support_oneshot_ms = timed(lambda: tt.support(desc, tables, support_out=sup, hist=hist, stream=stream), reps)
    # measured store roof: a plain fill of the same table buffer
    fill_ms = timed(lambda: tables.fill_(0), reps)
    # the tables again, for the bit-exact check of the CPU sample below
    plan.launch(tables, hist, stream)
    torch.cuda.synchronize()
    plan.kernel_times_ms()

    issued_ops = _mfma_issued_ops(ns)
    useful_ops = sum(2 * int(f) * (1 << max(0, int(f) * int(b) - 6)) for f, b in zip(ns.F, ns.b))

    achieved = table_bytes / (kernel_ms * 1e-3) / 1e9
    traffic = read_traffic(table_bytes)
    out = {
        "metric": "truth-table rows/sec (neuron-evals/s) + MFMA/HBM % peak, batched vs plain, bit-exact",
        "value": rows / (step_ms * 1e-3),
        "unit": "rows/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": step_ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int8",
        "data": "synthetic",
        "config": {
            "workload": f"{args.workload}: {WORKLOADS[args.workload]}",
            "neurons": n,
            "rows": rows,
            "table_bytes": int(table_bytes),
            "step": "tt_plan_step: persistent enumeration with fused histogram + support of the plan's own "
                    "tables (from the neurons' parameters)",
            "tune": info,
            "parallelism": "single GPU",
        },
        "roofline": {
            "bound": "hbm",
            "kernel": ("enum_wide_kernel" if info["wide_neurons"] == n else
                       "enum_small_kernel" if info["wide_neurons"] == 0 else "enum_wide_kernel + enum_small_kernel"),
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": traffic,
            "kernel_ms": kernel_ms,
        },
        "detail": {
            "enumerate_batched_ms": batched_ms,
            "enumerate_batched_with_hist_ms": batched_hist_ms,
            "support_enumerated_ms": support_enum_ms,
            "support_tables_only_ms": support_only_ms,
            "step_ms_with_table_scan_support": batched_hist_ms + support_only_ms,
            "enumerate_plain_ms": plain_ms,
            "enumerate_graph_with_hist_ms": graph_ms,
            "step_eager_ms": step_eager_ms,
            "step_graph_ms": step_graph_ms,
            "step_eager_queued_ms": step_eager_queued_ms,
            "step_graph_queued_ms": step_graph_queued_ms,
            "support_hist_ms": support_ms,
            "support_hist_oneshot_ms": support_oneshot_ms,
            "store_roof_fill_ms": fill_ms,
            "store_roof_fill_GBps": table_bytes / (fill_ms * 1e-3) / 1e9,
            "enum_frac_of_store_roof": fill_ms / kernel_ms,
            "rows_per_s_enumerate_batched": rows / (batched_ms * 1e-3),
            "rows_per_s_enumerate_plain": rows / (plain_ms * 1e-3),
            "mfma_int8_issued_ops_per_launch": issued_ops,
            "mfma_int8_useful_ops_per_launch": useful_ops,
            "mfma_int8_issued_frac_of_peak": issued_ops / (kernel_ms * 1e-3) / (MFMA_I8_PEAK_TOPS * 1e12),
            "wall_s_timed_region": wall,
        },
    }
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(ns, desc, tables, args.cpu_seconds, rows / n)
    if args.copy_calibration:
        out["detail"]["copy_calibration_bytes"] = copy_calibration(torch)
    plan.close()
    print(json.dumps(out), flush=True)


def bench_lutnet(args):
    """The 256 -> 128 -> 64 network of cfg1 evaluated through its enumerated
    tables (a tt_lutnet handle, lookups only; the one-shot tt_lutnet_eval in
    detail): samples of 256 primary 2-bit
    inputs per second, with the tables resident in HBM; checked against the
    oracle's arithmetic evaluation on a sample."""
    import numpy as np
    import torch

    import paper_2502_08673_amd as tt
    import workloads

    ns = workloads.cfg1()
    fanin = workloads.network_fanin(ns)
    P, n, B = 256, len(ns), int(args.samples)
    desc = tt.descriptors(ns)
    total = tt.layout(desc)
    tables = torch.empty(total, dtype=torch.int64, device="cuda")
    tt.enumerate(desc, tables, total_words=total)
    inputs_h = np.random.Generator(np.random.PCG64(20250212 + 101)).integers(0, 4, size=(B, P)).astype(np.uint8)
    x = torch.from_numpy(inputs_h).cuda()
    out = torch.empty((B, n), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream()

    net = tt.Lutnet(desc, fanin, P, tables, total, stream)

    def step():
        net.run(x, out, stream)

    def oneshot():
        tt.lutnet_eval(desc, fanin, P, tables, total, x, out, stream)

    for _ in range(args.warmup):
        oneshot()
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(args.steps):
        oneshot()
    e1.record(stream)
    torch.cuda.synchronize()
    oneshot_ms = e0.elapsed_time(e1) / args.steps
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(args.steps):
        step()
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / args.steps
    # rejection sampling of the same number of draws (inputs made on the
    # device), kept when three last-layer neurons output the given codes
    # (about 1.1 % of draws)
    targets = {P + 444: 3, P + 439: 3, P + 441: 2}
    found_x = torch.empty((B, P), dtype=torch.uint8, device="cuda")
    found_d = torch.empty(B, dtype=torch.int64, device="cuda")
    count = torch.zeros(1, dtype=torch.int32, device="cuda")
    for _ in range(args.warmup):
        net.sample(targets, 1, 0, B, found_x, found_d, count, stream)
    count.zero_()
    torch.cuda.synchronize()
    e0.record(stream)
    for k in range(args.steps):
        net.sample(targets, 1, k * B, B, found_x, found_d, count, stream)
    e1.record(stream)
    torch.cuda.synchronize()
    sample_ms = e0.elapsed_time(e1) / args.steps
    kept = int(count.item())
    alg_bytes = B * (P + n)  # inputs read once, every output code written once
    res = {
        "metric": "LUT-network samples/s: cfg1 256-128-64 evaluated through its enumerated tables, bit-exact",
        "value": B / (ms * 1e-3), "unit": "samples/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u8",
        "data": "synthetic",
        "config": {"workload": "cfg1net: 448-neuron 256-128-64 network, F=6, b=2, o=2, tables via tt_enumerate",
                   "samples": B, "lookups_per_sample": n},
        # per-(sample, neuron) instructions bound the kernel, not bytes: the
        # instruction-rate roofline, with the HBM view beside it
        "roofline": alu_roofline("lutnet_packed_kernel (one launch)", ms, read_sq(NET_SQ_FILE, NET_SRC)),
        "detail": {"hbm_roofline": {"achieved": alg_bytes / (ms * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                                    "frac": alg_bytes / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                                    "traffic": read_traffic(alg_bytes, NET_TRAFFIC_FILE, NET_SRC)},
                   "lookups_per_s": B * n / (ms * 1e-3), "oneshot_eval_ms": oneshot_ms,
                   "sample_draws_per_s": B / (sample_ms * 1e-3), "sample_ms": sample_ms,
                   "sample_targets": {str(k): v for k, v in targets.items()},
                   "sample_kept_fraction": kept / (B * args.steps)},
    }
    net.close()
    if not args.no_cpu_baseline:
        from oracle import lutnet
        got = out.cpu().numpy()
        f6 = [f[:6] for f in fanin]
        t0 = time.perf_counter()
        lutnet.evaluate(ns, f6, P, inputs_h[:4096])  # pilot: sizes the sample to about --cpu-seconds
        rate = 4096 / (time.perf_counter() - t0)
        m = int(min(B, max(4096, rate * args.cpu_seconds)))
        t0 = time.perf_counter()
        want = lutnet.evaluate(ns, f6, P, inputs_h[:m])
        t_cpu = time.perf_counter() - t0
        res["cpu_baseline"] = {"value": m / t_cpu, "unit": "samples/s", "cores": 1, "kind": "oracle",
                               "sample": f"first {m} of {B} samples, {t_cpu:.1f} s",
                               "bit_exact_vs_gpu": bool(np.array_equal(got[:m], want))}
    return res


def bench_cnf(args):
    """Algorithm 1 on random Tseitin circuits (8 to 64 gates of every kind,
    4 to 12 primary inputs, a unit constraint on the last output): CNF
    instances transformed per second by a staged tt_cnf handle (clauses
    resident in HBM, one wave per instance), checked against the oracle's
    Algorithm 1 on a sample."""
    import numpy as np
    import torch

    import paper_2502_08673_amd as tt
    import workloads

    distinct = workloads.tseitin_instances(20250212 + 201, min(8192, int(args.instances)))
    inst = (distinct * (int(args.instances) // len(distinct) + 1))[: int(args.instances)]
    lits, coff, ioff, nv = tt.cnf_csr(inst)
    n_inst, n_cl = len(inst), int(ioff[-1])
    stream = torch.cuda.current_stream()
    vc = torch.zeros((int((nv + 1).sum()),), dtype=torch.uint8, device="cuda")
    ex = torch.zeros((n_cl * 640,), dtype=torch.uint8, device="cuda")
    ne = torch.zeros((n_inst,), dtype=torch.int32, device="cuda")
    st = torch.zeros((n_inst,), dtype=torch.int32, device="cuda")
    t0 = time.perf_counter()
    tt.cnf_transform(lits, coff, ioff, nv, vc, ex, ne, st, stream)
    torch.cuda.synchronize()
    oneshot_s = time.perf_counter() - t0
    h = tt.Cnf(lits, coff, ioff, nv, stream)
    for _ in range(args.warmup):
        h.run(vc, ex, ne, st, stream)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(args.steps):
        h.run(vc, ex, ne, st, stream)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / args.steps
    h.close()
    n_expr = ne.cpu().numpy()
    status = st.cpu().numpy()
    # clauses, offsets and classes read; expression records and classes written
    alg_bytes = 4 * (len(lits) + 2 * n_cl + 4 * n_inst) + 640 * int(n_expr.sum()) + vc.numel()
    res = {
        "metric": "CNF instances transformed per second (Algorithm 1 on packed truth tables), exact",
        "value": n_inst / (ms * 1e-3), "unit": "instances/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "u64 (bit tables)", "data": "synthetic",
        "config": {"workload": "cnf: random Tseitin circuits, 8-64 gates, 4-12 inputs, unit constraint on the last "
                               "output", "instances": n_inst, "distinct_instances": len(distinct), "clauses": n_cl,
                   "literals": int(len(lits))},
        "roofline": alu_roofline("cnf_fast_kernel", ms, read_sq(CNF_SQ_FILE, os.path.join(CSRC, "tt_cnf.hip"))),
        "detail": {"clauses_per_s": n_cl / (ms * 1e-3), "expressions": int(n_expr.sum()),
                   "algorithmic_bytes": alg_bytes, "hbm_frac_of_algorithmic_bytes": alg_bytes / (ms * 1e-3) / 1e9 /
                   HBM_PEAK_GBS,
                   "instances_stopped": int((status != 0).sum()),
                   "oneshot_wall_ms_incl_host_prep_and_upload": oneshot_s * 1e3},
    }
    if not args.no_cpu_baseline:
        from oracle import transform as T
        recs = ex.cpu().numpy().view(tt.CNF_EXPR_DTYPE)
        t0 = time.perf_counter()
        for k in range(20):
            T.transform(inst[k][1])
        rate = 20 / (time.perf_counter() - t0)
        m = int(min(len(distinct), max(20, rate * args.cpu_seconds)))
        t0 = time.perf_counter()
        got = [T.transform(inst[k][1]) for k in range(m)]
        t_cpu = time.perf_counter() - t0
        exact = True
        for k, (_, _, _, E) in enumerate(got):
            exact &= int(n_expr[k]) == len(E)
            for q, e in enumerate(E[: int(n_expr[k])]):
                r = recs[int(ioff[k]) + q]
                n = int(r["n_vars"])
                words = [int(w) for w in r["table"]]
                table = sum(w << (64 * i) for i, w in enumerate(words)) & ((1 << (1 << n)) - 1)
                sup = [e.vars[j] for j in range(n) if (int(r["support"]) >> j) & 1]
                exact &= (int(r["out"]), int(r["first"]), int(r["last"]), list(r["vars"][:n]), table, sup) == \
                    (e.out, e.first, e.last, e.vars, e.table, e.support)
        res["cpu_baseline"] = {"value": m / t_cpu, "unit": "instances/s", "cores": 1, "kind": "oracle",
                               "sample": f"first {m} of {n_inst} instances, {t_cpu:.1f} s",
                               "bit_exact_vs_gpu": bool(exact)}
    return res


def bench_gd(args):
    """The paper's sampler on a transformed CNF: one random Tseitin circuit
    (48 candidate inputs, 60 gates reading the last 64 signals, the last
    output forced to 1) transformed
    by tt_cnf, then GD (rate 10, 5 iterations) on a batch of random logits,
    hardening, the CNF check and the distinct-solution filter; unique valid
    solutions per second, the paper's throughput metric."""
    import numpy as np
    import torch

    import paper_2502_08673_amd as tt
    import workloads

    n_vars, clauses = workloads.tseitin_instances(20250212 + 301, 1, n_in=(48, 48), n_gates=(60, 60), window=64)[0]
    lits, coff, ioff, nv = tt.cnf_csr([(n_vars, clauses)])
    stream = torch.cuda.current_stream()
    vc = torch.zeros((n_vars + 1,), dtype=torch.uint8, device="cuda")
    ex = torch.zeros((len(clauses) * 640,), dtype=torch.uint8, device="cuda")
    ne = torch.zeros((1,), dtype=torch.int32, device="cuda")
    st = torch.zeros((1,), dtype=torch.int32, device="cuda")
    t0 = time.perf_counter()
    tt.cnf_transform(lits, coff, ioff, nv, vc, ex, ne, st, stream)
    torch.cuda.synchronize()
    transform_ms = (time.perf_counter() - t0) * 1e3
    assert int(st.item()) == 0
    recs = ex.cpu().numpy().view(tt.CNF_EXPR_DTYPE)[: int(ne.item())]
    cls = vc.cpu().numpy()
    gd = tt.GdSampler(clauses, n_vars, recs, cls, stream)
    B = int(args.batch)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(20250212 + 302)
    V0 = torch.randn((B, gd.n_pi), device="cuda", generator=gen)  # the initial logits, read by every step
    V = torch.empty_like(V0)
    valid = torch.empty((B,), dtype=torch.uint8, device="cuda")
    sol = torch.empty((B, gd.words), dtype=torch.int64, device="cuda")
    first = torch.empty((B,), dtype=torch.uint8, device="cuda")
    count = torch.zeros((1,), dtype=torch.int32, device="cuda")

    def step():
        # GD from the initial logits (the final ones are not kept), then the
        # distinct valid solutions; the compiled kernel also does the
        # filter's first pass
        count.zero_()
        gd.sample_unique(V0, None, 10.0, 5, valid, sol, first, count, stream)

    def step_two_calls():
        # the same as tt_gd_run_from, then tt_gd_unique
        count.zero_()
        gd.run_from(V0, None, 10.0, 5, valid, sol, stream)
        gd.unique(valid, sol, first, count, stream)

    def step_in_place():
        # the same through tt_gd_run: the logits restored, updated in place
        V.copy_(V0)
        count.zero_()
        gd.run(V, 10.0, 5, valid, sol, stream)
        gd.unique(valid, sol, first, count, stream)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(args.steps):
        step()
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / args.steps
    uniq = int(count.item())
    n_valid = int(valid.sum().item())
    # the sampling kernel alone (GD from the logits as they stand: the same
    # work), the circuit's compiled kernel and the interpreter; the filter alone
    def timed(fn):
        fn()
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(args.steps):
            fn()
        e1.record(stream)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / args.steps

    kernel = gd.kernel
    run_ms = timed(lambda: gd.run_from(V0, None, 10.0, 5, valid, sol, stream))
    two_calls_ms = timed(step_two_calls)
    in_place_ms = timed(step_in_place)
    gd.kernel = tt.TT_GD_INTERPRETED
    V.copy_(V0)
    interp_ms = timed(lambda: gd.run(V, 10.0, 5, valid, sol, stream))
    gd.kernel = kernel
    unique_ms = timed(lambda: gd.unique(valid, sol, first, count, stream))
    words = gd.words
    alg_bytes = B * (4 * gd.n_pi + 1 + 8 * words)  # initial logits read, validity and solutions written
    res = {
        "metric": "unique valid solutions per second (GD sampling of a transformed CNF)",
        "value": uniq / (ms * 1e-3), "unit": "solutions/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": "gd: random Tseitin circuit, 48 inputs, 60 gates, last output forced to 1; GD rate 10, "
                               "5 iterations", "batch": B, "primary_inputs": gd.n_pi, "expressions": len(recs),
                   "clauses": len(clauses)},
        "roofline": (alu_roofline("tt_gd_compiled (the circuit's own kernel)", run_ms,
                                  read_sq(GD_SQ_FILE, os.path.join(CSRC, "tt_gd_compile.hip")))
                     if kernel == tt.TT_GD_COMPILED else
                     alu_roofline("gd_sample_kernel", run_ms, read_sq(GD_INTERP_SQ_FILE, os.path.join(CSRC, "tt_gd.hip")))),
        "detail": {"valid_fraction": n_valid / B, "unique": uniq, "transform_ms_incl_host": transform_ms,
                   "kernel": "compiled" if kernel == tt.TT_GD_COMPILED else "interpreted",
                   "gd_run_ms": run_ms, "gd_run_interpreted_ms": interp_ms, "unique_filter_ms": unique_ms,
                   "step_two_calls_ms": two_calls_ms, "step_in_place_ms": in_place_ms,
                   "interpreted_roofline": alu_roofline("gd_sample_kernel", interp_ms,
                                                        read_sq(GD_INTERP_SQ_FILE, os.path.join(CSRC, "tt_gd.hip"))),
                   "algorithmic_bytes": alg_bytes,
                   "hbm_frac_of_algorithmic_bytes_whole_step": alg_bytes / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                   "samples_per_s": B / (ms * 1e-3)},
    }
    gd.close()
    if not args.no_cpu_baseline:
        from oracle import gdsample as G
        from oracle import transform as T
        R = T.transform(clauses)
        V0h = V0.cpu().numpy().astype(np.float64)
        t0 = time.perf_counter()
        G.sample(clauses, R, V0h[:1000])
        rate = 1000 / (time.perf_counter() - t0)
        m = int(min(B, max(1000, rate * args.cpu_seconds)))
        t0 = time.perf_counter()
        _, ok, u = G.sample(clauses, R, V0h[:m])
        t_cpu = time.perf_counter() - t0
        res["cpu_baseline"] = {"value": len(u) / t_cpu, "unit": "solutions/s", "cores": 1, "kind": "oracle",
                               "sample": f"first {m} of {B} samples, {t_cpu:.1f} s ({len(u)} unique)",
                               "valid_fraction": float(ok.mean())}
    return res


def bench_screen(args):
    """Learned screen: train on 200k neurons, screen 100k new candidates;
    plain enumeration vs the trivial nonzero-weight screen vs the learned
    screen, all exact (outputs compared bit for bit with plain)."""
    import math

    import numpy as np
    import torch

    import paper_2502_08673_amd as tt
    import workloads
    from paper_2502_08673_amd import screen as sc

    t0 = time.perf_counter()
    tr = sc.candidates(workloads.cfg4_train())
    dtr = sc.exact_labels(tr)
    torch.cuda.synchronize()
    t_labels = time.perf_counter() - t0
    n_hold = 20000
    fit = {k: dtr[k][: tr.n - n_hold] for k in ("X", "y", "m", "h")}
    hold = {k: dtr[k][tr.n - n_hold:] for k in ("X", "y", "m", "h")}
    net = sc.ScreenNet(workloads.mlp_init(20250212 + 42), max_batch=100_000)
    t0 = time.perf_counter()
    losses = sc.train(net, fit, epochs=args.epochs, batch=4096, lr=2e-3, seed=1)
    torch.cuda.synchronize()
    t_train = time.perf_counter() - t0

    # Operating point: among thresholds whose support-bit accuracy on the
    # held-out training neurons that the network screens (the wave-pass
    # candidates) is at least 0.99, the one with the fewest modelled rows.
    hold_ns = workloads.subset(tr.ns, np.arange(tr.n - n_hold, tr.n))
    hc = sc.candidates(hold_ns)
    hl = sc.predict(net, hold["X"], n_hold)
    hg = torch.from_numpy(np.nonzero(sc.wave_pass_candidates(hc.desc))[0]).cuda()
    hr = sc.ScreenRunner(hc)
    search = []
    for tau in (0.5, 0.3, 0.2, 0.1, 0.05, 0.03):
        a = sc.support_accuracy(hl.index_select(0, hg), hold["y"].index_select(0, hg), hold["m"].index_select(0, hg),
                                tau)
        hr.screened(logits=hl, tau=tau)
        cost = sc.row_cost(hc, hr.mask.cpu().numpy(), hr.accept.cpu().numpy())
        search.append({"tau": tau, "holdout_bit_accuracy": a["bit_accuracy"], "holdout_rows": cost})
    ok = [r for r in search if r["holdout_bit_accuracy"] >= 0.99]
    pick = min(ok, key=lambda r: r["holdout_rows"]) if ok else max(search, key=lambda r: r["holdout_bit_accuracy"])
    tau = pick["tau"]

    c = sc.candidates(workloads.cfg4_screen())
    d = sc.exact_labels(c)  # plain reference outputs (full enumeration + support)
    runner = sc.ScreenRunner(c)
    ref_tables = d["tables"]
    ref_sup = d["support"].clone()
    ref_hist = d["hist"].clone()
    full = torch.empty_like(runner.tables)
    gate = sc.wave_pass_candidates(c.desc)
    gi = torch.from_numpy(np.nonzero(gate)[0]).cuda()
    lg_all = torch.empty((c.n, 12), dtype=torch.float32, device="cuda")
    net.infer_desc(c.d_desc, c.n, False, lg_all)  # every candidate: accuracy report only
    acc_screened = sc.support_accuracy(lg_all.index_select(0, gi), d["y"].index_select(0, gi),
                                       d["m"].index_select(0, gi), tau)
    acc_all = sc.support_accuracy(lg_all, d["y"], d["m"], tau)
    trivial = sc.nonzero_weight_mask(c)

    def check():
        torch.cuda.synchronize()
        ok = bool(torch.equal(runner.support, ref_sup)) and bool(torch.equal(runner.hist, ref_hist))
        runner.expand(full)
        torch.cuda.synchronize()
        return ok and bool(torch.equal(full, ref_tables)) and runner.status.item() == 0

    learned = sc.LearnedScreen(net, runner, tau)
    reps = 10
    t_plain = sc.timed(runner.plain, reps)
    ok_plain = bool(torch.equal(runner.support, ref_sup)) and bool(torch.equal(runner.hist, ref_hist))
    t_trivial = sc.timed(lambda: runner.screened(force_mask=trivial), reps)
    ok_trivial = check()
    cost_trivial = sc.row_cost(c, runner.mask.cpu().numpy(), runner.accept.cpu().numpy())
    t_ideal = sc.timed(lambda: runner.screened(force_mask=ref_sup), reps)
    ok_ideal = check()
    cost_ideal = sc.row_cost(c, runner.mask.cpu().numpy(), runner.accept.cpu().numpy())
    t_infer = sc.timed(lambda: net.infer_desc(c.d_desc, c.n, True, learned.logits), reps)
    t_infer_gpu = sc.timed_queued(lambda: net.infer_desc(c.d_desc, c.n, True, learned.logits), reps)
    t_infer_all = sc.timed(lambda: net.infer_desc(c.d_desc, c.n, False, lg_all), reps)
    t_learned = sc.timed(learned, reps)
    ok_learned = check()
    cost_learned = sc.row_cost(c, runner.mask.cpu().numpy(), runner.accept.cpu().numpy())
    accept_rate = float(runner.accept.float().mean().item())

    # The host-built batched plan on the same candidates, plan creation and
    # tuning outside the timed region: enumeration with fused histogram, then
    # the support of the tables as tables; and the whole step, whose support
    # follows from the parameters (plain enumeration at its fastest).
    ptab = torch.empty(c.total_words, dtype=torch.int64, device="cuda")
    psup = torch.zeros(c.n, dtype=torch.uint8, device="cuda")
    phist = torch.zeros(c.n * 8, dtype=torch.int32, device="cuda")
    ptune = tt.autotune(c.desc, ptab, cache_path=args.tune_cache)
    pplan = tt.Plan(c.desc, c.total_words, tune=ptune, flags=tt.TT_PLAN_PERSISTENT)

    def batched():
        pplan.launch(ptab, phist)
        pplan.support(ptab, support_out=psup)

    t_batched = sc.timed(batched, reps)
    torch.cuda.synchronize()
    ok_batched = (bool(torch.equal(psup, ref_sup)) and bool(torch.equal(phist, ref_hist))
                  and bool(torch.equal(ptab, ref_tables)))
    psup.zero_()
    t_step = sc.timed(lambda: pplan.step(ptab, phist, psup), reps)
    torch.cuda.synchronize()
    ok_batched = ok_batched and bool(torch.equal(psup, ref_sup)) and bool(torch.equal(phist, ref_hist))
    pplan.close()
    rows = c.ns.total_rows()
    return {
        "metric": "learned screen: end-to-end screened vs plain enumeration (support + histogram), exact",
        "value": t_plain / t_learned,
        "unit": "speedup",
        "n_gpus": 1,
        "higher_is_better": True,
        "dtype": "bf16 (screen) / int8 (enumeration)",
        "data": "synthetic",
        "config": {"workload": "cfg4: train 200k, screen 100k neurons of the uneven distribution",
                   "train_neurons": tr.n - n_hold, "holdout_neurons": n_hold, "screen_neurons": c.n,
                   "network_screened_candidates": int(gate.sum()), "epochs": args.epochs, "batch": 4096,
                   "tau": tau},
        "detail": {
            "label_generation_s": t_labels, "train_s": t_train, "loss_first_epoch": losses[0],
            "loss_last_epoch": losses[-1], "tau_search": search,
            "support_bit_accuracy": acc_screened["bit_accuracy"],
            "support_exact_neurons": acc_screened["exact_neurons"],
            "support_covered": acc_screened["covers_support"],
            "support_bit_accuracy_all_candidates": acc_all["bit_accuracy"],
            "plain_ms": t_plain, "trivial_screen_ms": t_trivial, "learned_screen_ms": t_learned,
            "ideal_mask_screen_ms": t_ideal, "network_gated_ms": t_infer, "network_gated_gpu_ms": t_infer_gpu,
            "network_all_candidates_ms": t_infer_all,
            "speedup_learned_vs_plain": t_plain / t_learned, "speedup_trivial_vs_plain": t_plain / t_trivial,
            "speedup_learned_vs_trivial": t_trivial / t_learned, "speedup_ideal_vs_trivial": t_trivial / t_ideal,
            "plain_batched_plan_ms": t_batched, "speedup_learned_vs_batched_plan": t_batched / t_learned,
            "plain_plan_step_ms": t_step, "speedup_learned_vs_plan_step": t_step / t_learned,
            "exact_batched_plan": ok_batched,
            "rows_plain": rows, "rows_trivial": cost_trivial, "rows_learned": cost_learned, "rows_ideal": cost_ideal,
            "accept_rate_learned": accept_rate,
            "exact_plain": ok_plain, "exact_trivial": ok_trivial, "exact_learned": ok_learned, "exact_ideal": ok_ideal,
            "final_mismatches": 0 if (ok_learned and ok_trivial and ok_plain) else -1,
        },
    }


def _mfma_issued_ops(ns):
    """int8 MFMA ops issued per launch: one 16x16x32 product per 256 words of
    one neuron, for tables of at least 256 words per plane (shorter ones sum
    per lane)."""
    ops = 0
    for f, b in zip(ns.F, ns.b):
        w = max(1, (1 << (int(f) * int(b))) // 64)
        ops += (w // 256) * 16 * 16 * 32 * 2
    return ops


def cpu_baseline(ns, desc, tables, seconds, rows_per_neuron):
    """The oracle as it stands, on all host cores, over a bounded sample of
    neurons (batches of one neuron per core until `seconds` have passed), and
    a bit-exact comparison of the sample's GPU tables."""
    import numpy as np

    import oracle
    from workloads import subset

    cores = oracle.max_threads()
    done, t_cpu, exact = 0, 0.0, True
    n = len(ns)
    while done < n and t_cpu < seconds:
        idx = list(range(done, min(n, done + cores)))
        sub = subset(ns, idx)
        t0 = time.perf_counter()
        ref = oracle.enumerate(sub, hist=False, support=False, nthreads=cores)
        t_cpu += time.perf_counter() - t0
        for k, i in enumerate(idx):
            W = max(1, (1 << (int(ns.F[i]) * int(ns.b[i]))) // 64)
            o = int(ns.o[i])
            off = int(desc["word_off"][i])
            got = tables[off: off + o * W].cpu().numpy().view(np.uint64)
            ro = int(ref["word_off"][k])
            exact &= bool(np.array_equal(got, ref["planes"][ro: ro + o * W]))
        done += len(idx)
    sample_rows = int(sum(1 << (int(ns.F[i]) * int(ns.b[i])) for i in range(done)))
    return {
        "value": sample_rows / t_cpu,
        "unit": "rows/s",
        "cores": cores,
        "kind": "oracle",
        "sample": f"first {done} of {n} neurons ({sample_rows} rows), planes only, {t_cpu:.1f} s",
        "bit_exact_vs_gpu": exact,
    }


def copy_calibration(torch):
    """A plain device copy of 1 GiB (read 1 GiB, write 1 GiB): the counter
    reference for the HBM traffic of the enumeration kernel."""
    a = torch.empty(1 << 27, dtype=torch.int64, device="cuda")
    b = torch.empty_like(a)
    a.fill_(1)
    torch.cuda.synchronize()
    for _ in range(3):
        b.copy_(a)
    torch.cuda.synchronize()
    return 1 << 30


if __name__ == "__main__":
    main()
