#!/usr/bin/env python3
"""Benchmark of the RSR++ vector x matrix product on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--batch B] [--regime cold|warm]
                    [--workload NAME] [--dtype f32|i8]

A "step" is one pass of the whole hot path (index stream, gather, segmented sums, fold, combine,
store) over one batch: one rsr_matvec call.  The default workload is the binary 16384 x 16384
matrix with block width k = 12 and one float activation vector, i.e. the configuration the
headline metric is quoted on.  Inputs are seeded and synthetic and are resident in device memory
before the timed region starts.

Regimes: "cold" rotates the calls over enough separately allocated copies of the index that the
working set exceeds twice the 256 MB last-level cache, so every call streams its tables from
HBM; "warm" calls one copy back to back (cache-assisted; reported for context).

Prints ONE JSON line: throughput in matvecs/s, the HBM roofline of the kernel, and the CPU oracle
timed on the host cores on a bounded sample (a reported baseline, not a target).  The roofline's
`achieved` counts the bytes of the method itself: the permutations and full segmentations as 16-bit
words, P*nb*rows*2 + P*nb*2^k*2, plus activations in and results out, over the average launch
duration measured with events on the launch stream; `stored_frac` is the same figure on the bytes
of the tables as this library stores them (what a launch really reads).  `launch_us_median` and
`launch_us_min` are taken over groups of ten launches; `warm_launch_us` is the same product called
on one copy of the index back to back (cache-assisted, for context).
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

HBM_PEAK_GBS = 8000.0          # MI355X published peak HBM3E bandwidth

# HBM bytes per launch measured offline with rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE (scaled by a plain
# copy of known size; summaries under profiles/).  Keyed by (workload, batch, dtype, regime); the value
# holds the stored table bytes of the build that was profiled, and the figure is reported only while
# the tables still have that size (any change of the layout makes it null until it is measured again).
PROFILED_TRAFFIC = {
    ("binary_16k", 1, "f32", "cold"): {"table_bytes": 58392380, "traffic_bytes": 60.0e6,
                                       "source": "profiles/rsr_matvec_f32_binary16k_b1_cold.md"},
    ("binary_16k", 8, "f32", "cold"): {"table_bytes": 58392380, "traffic_bytes": 70.6e6,
                                       "source": "profiles/rsr_matvec_f32_binary16k_b8_cold.md"},
}
PRECONDITION_LAUNCHES = 3000   # untimed, before the warm-up steps (see main)
LLC_BYTES = 256 << 20          # last-level (Infinity) cache; the cold regime rotates over > 2x this


def parse_args():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3000)
    ap.add_argument("--warmup", type=int, default=300)
    ap.add_argument("--batch", type=int, default=1)
    ap.add_argument("--regime", choices=("cold", "warm"), default="cold")
    ap.add_argument("--workload", default="binary_16k")
    ap.add_argument("--dtype", choices=("f32", "i8"), default="f32")
    ap.add_argument("--step2", choices=("fold", "plain"), default="fold",
                    help="step 2 as the RSR++ fold (Algorithm 3) or as the plain product of Algorithm 2 (for comparison)")
    ap.add_argument("--comparator", choices=("none", "dense"), default="none",
                    help="dense: time the bit-packed comparator (include/rsr_dense.h) instead of the RSR++ path, same protocol")
    ap.add_argument("--cpu-seconds", type=float, default=10.0, help="budget of the CPU-oracle timing leg")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU-oracle leg and with it the parity check (profiling runs)")
    ap.add_argument("--no-check", action="store_true", help="skip the parity check against the CPU leg's product")
    ap.add_argument("--plain", action="store_true",
                    help="only the W warm-up and K timed steps: no conditioning launches, no per-group spread, no warm figure "
                         "(for runs under a profiler, where every launch of the process is counted)")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="N",
                    help="also run N plain device copies of 256 MiB (a kernel of known traffic, used to "
                         "scale the FETCH_SIZE / WRITE_SIZE counters of a rocprofv3 --pmc run)")
    return ap.parse_args()


def cpu_baseline(A, v, dtype, budget_s):
    """The oracle as it stands, on all host cores (column stripes), for about budget_s seconds.

    Returns the baseline record and the oracle's product of every batch lane (the leg's first call),
    against which the caller checks what the GPU returned for the same inputs.
    """
    from oracle import dense

    threads = dense.host_threads()
    fn = dense.matvec_f32 if dtype == "f32" else dense.matvec_i8
    exact = fn(A, v, threads=threads)
    one = v[:1]
    t0 = time.perf_counter()
    fn(A, one, threads=threads)
    first = time.perf_counter() - t0
    reps = max(1, min(200, int(budget_s / max(first, 1e-4)) - 1))
    t0 = time.perf_counter()
    for _ in range(reps):
        fn(A, one, threads=threads)
    dt = time.perf_counter() - t0
    t1 = time.perf_counter()
    fn(A, one, threads=1)
    single = time.perf_counter() - t1
    return {
        "value": reps / dt,
        "unit": "matvecs/s",
        "cores": threads,
        "kind": "oracle",
        "sample": f"{reps} full products of the same {A.shape[0]}x{A.shape[1]} matrix with one vector, "
                  f"columns striped over {threads} threads",
        "single_thread_matvecs_per_s": 1.0 / single,
    }, exact


def bench_llm_block(args):
    """--workload llm_block: one decode step of the transformer block of configuration 4 as a unit of work.

    The block's seven matrices are four stages (q/k/v one index, attn_o, gate/up one index, mlp_down): a step
    is the four products, (a) as four launches captured in one HIP graph (the stages of a real block depend on
    each other through attention and the activation function, which are not part of this library, so they
    stay separate kernels), (b) as four plain launches, (c) as one launch that carries all four (possible
    only when their inputs are ready together; an upper bound).  `value` is (a)."""
    import numpy as np
    import torch

    import paper_2411_06360_amd as R
    import workloads
    from oracle import dense

    torch.cuda.set_device(0)
    stages = workloads.llm_block_stages()
    mats = [workloads.stage_matrix(members) for _, members in stages]
    k = stages[0][1][0].k
    batch = args.batch
    i8 = args.dtype == "i8"   # the int8 activations of a BitLinear-style layer (Section 5.3), int32 results, exact
    vs = [members[0].activations(batch, args.dtype) for _, members in stages]
    first = [R.rsr_preprocess(A, k) for A in mats]
    infos = [R.rsr_info(h) for h in first]
    table_bytes = sum(int(i.table_bytes) for i in infos)
    ncopies = 1 if args.regime == "warm" else min(32, max(2, -(-2 * LLC_BYTES // table_bytes) + 1))
    copies = [first] + [[R.rsr_preprocess(A, k) for A in mats] for _ in range(ncopies - 1)]
    dv = [torch.from_numpy(v).cuda() for v in vs]
    outs = [torch.zeros((batch, A.shape[1]), dtype=torch.int32 if i8 else torch.float32, device="cuda") for A in mats]
    lib = R.load()
    matvec = lib.rsr_matvec_i8 if i8 else lib.rsr_matvec
    cur = torch.cuda.current_stream().cuda_stream

    def launches(hs, stream):
        for h, v, o in zip(hs, dv, outs):
            if matvec(h, v.data_ptr(), o.data_ptr(), batch, stream) != 0:
                raise RuntimeError(R.rsr_last_error())

    jobs = [R.make_jobs(list(zip(hs, dv, outs))) for hs in copies]

    def fused(c, stream):
        (R.rsr_matvec_multi_i8 if i8 else R.rsr_matvec_multi)(jobs[c], batch, stream)

    launches(copies[-1], cur)
    torch.cuda.synchronize()
    got = [o.cpu().numpy() for o in outs]
    side = torch.cuda.Stream()
    graphs = []
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        launches(copies[0], side.cuda_stream)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for hs in copies:
        gph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(gph, stream=side):
            launches(hs, torch.cuda.current_stream().cuda_stream)
        graphs.append(gph)

    def timed(step_fn, steps, warm):
        for i in range(warm):
            step_fn(i % ncopies)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0 = time.perf_counter()
        e0.record()
        for i in range(steps):
            step_fn((warm + i) % ncopies)
        e1.record()
        torch.cuda.synchronize()
        return time.perf_counter() - t0, e0.elapsed_time(e1) * 1e3 / steps

    for i in range(PRECONDITION_LAUNCHES // 4):
        graphs[i % ncopies].replay()
    torch.cuda.synchronize()
    wall, graph_us = timed(lambda c: graphs[c].replay(), args.steps, args.warmup)
    _, plain_us = timed(lambda c: launches(copies[c], cur), args.steps, args.warmup)
    _, fused_us = timed(lambda c: fused(c, cur), args.steps, args.warmup)
    per_stage = []
    for si in range(len(stages)):
        def one(c, si=si):
            if matvec(copies[c][si], dv[si].data_ptr(), outs[si].data_ptr(), batch, cur) != 0:
                raise RuntimeError(R.rsr_last_error())
        per_stage.append(timed(one, args.steps, args.warmup)[1])

    io_bytes = sum(batch * (A.shape[0] * (1 if i8 else 4) + A.shape[1] * 4) for A in mats)
    method_bytes = sum(int(i.parts) * int(i.nblocks) * (int(i.rows) * 2 + (1 << k) * 2) for i in infos) + io_bytes
    stored_bytes = table_bytes + io_bytes
    result = {
        "metric": "RSR++ transformer-block decode step (7 ternary matrices of a ~2B-parameter 1.58-bit block as 4 products): blocks/s",
        "value": args.steps / wall,
        "unit": "blocks/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": wall * 1e3 / args.steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": args.dtype, "data": "synthetic",
        "config": {
            "workload": f"llm_block: stages {[n for n, _ in stages]} with shapes {[list(A.shape) for A in mats]}, k={k}, batch {batch}, {args.dtype} activations",
            "regime": args.regime, "index_copies_rotated": ncopies, "table_bytes": table_bytes,
            "step": "four launches captured in one HIP graph, one replay per step",
            "us_per_block_graph": graph_us, "us_per_block_four_launches": plain_us, "us_per_block_one_launch": fused_us,
            "us_per_stage_alone": dict(zip([n for n, _ in stages], per_stage)),
            "us_per_block_at_hbm_peak": stored_bytes / HBM_PEAK_GBS * 1e-3,
            "parity_worst_error_over_bound": None,
        },
        "roofline": {
            "bound": "hbm", "achieved": method_bytes / (graph_us * 1e-6) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": method_bytes / (graph_us * 1e-6) / 1e9 / HBM_PEAK_GBS, "traffic": None,
            "algorithmic_bytes_per_launch": method_bytes, "stored_bytes_per_launch": stored_bytes,
            "stored_frac": stored_bytes / (graph_us * 1e-6) / 1e9 / HBM_PEAK_GBS, "launch_us": graph_us,
            "note": "per block (four kernels); the smallest stage alone is bound by what a launch costs before its first sums",
        },
    }
    if not args.no_cpu:
        threads = dense.host_threads()
        oracle_fn = dense.matvec_i8 if i8 else dense.matvec_f32
        exact = [oracle_fn(A, v, threads=threads) for A, v in zip(mats, vs)]
        worst = 0.0
        for g_, e_, v in zip(got, exact, vs):
            if i8:
                if not np.array_equal(g_.astype(np.int64), e_):
                    print("parity FAILED: int8 result differs from the oracle", file=sys.stderr)
                    sys.exit(1)
                continue
            bound = 1e-5 * np.abs(v.astype(np.float64)).sum(axis=1, keepdims=True)
            worst = max(worst, float((np.abs(g_.astype(np.float64) - e_) / bound).max()))
        if not worst <= 1.0:
            print(f"parity FAILED: error is {worst:.3g} x the allowed 1e-5*sum|v|", file=sys.stderr)
            sys.exit(1)
        result["config"]["parity_worst_error_over_bound"] = worst
        t0 = time.perf_counter()
        reps = 0
        while time.perf_counter() - t0 < args.cpu_seconds:
            for A, v in zip(mats, vs):
                oracle_fn(A, v[:1], threads=threads)
            reps += 1
        result["cpu_baseline"] = {
            "value": reps / (time.perf_counter() - t0), "unit": "blocks/s", "cores": threads, "kind": "oracle",
            "sample": f"{reps} passes over the four stage matrices with one vector each, columns striped over {threads} threads",
        }
    torch.cuda.synchronize()
    del graphs
    for hs in copies:
        for h in hs:
            R.rsr_destroy(h)
    print(json.dumps(result), flush=True)


def main():
    args = parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU: --gpus {args.gpus} is not supported (column blocks shard across "
              "GPUs without communication, but this build runs on a single device)", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2411_06360_amd as R
    import workloads

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(2)
    if args.workload == "llm_block":
        bench_llm_block(args)
        return
    torch.cuda.set_device(0)
    w = workloads.get(args.workload)
    A = w.matrix()
    v = w.activations(args.batch, args.dtype)
    rows, cols = A.shape

    # ---- index copies -------------------------------------------------------------------------
    dense_mode = args.comparator == "dense"
    first = R.rsr_preprocess(A, w.k)
    info = R.rsr_info(first)
    table_bytes = int(info.table_bytes)
    if dense_mode:  # the comparator: same inputs, same rotation and timing, other tables and kernels
        R.rsr_destroy(first)
        first = R.rsr_dense_preprocess(A)
        table_bytes = R.rsr_dense_table_bytes(first)
    if args.regime == "cold":
        ncopies = max(2, -(-2 * LLC_BYTES // table_bytes) + 1)
        ncopies = min(ncopies, 64)
    else:
        ncopies = 1
    handles = [first] + [(R.rsr_dense_preprocess(A) if dense_mode else R.rsr_preprocess(A, w.k)) for _ in range(ncopies - 1)]
    if args.step2 == "plain" and not dense_mode:
        for h in handles:
            R.rsr_set_step2(h, R.RSR_STEP2_PLAIN)

    dv = torch.from_numpy(v).cuda()
    out_dtype = torch.float32 if args.dtype == "f32" else torch.int32
    dout = torch.zeros((args.batch, cols), dtype=out_dtype, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    call = R.rsr_matvec if args.dtype == "f32" else R.rsr_matvec_i8
    if dense_mode:
        call = R.rsr_dense_matvec if args.dtype == "f32" else R.rsr_dense_matvec_i8

    # ---- one product at full size, in the launch configuration that is timed: kept for the check
    #      against the oracle's product, which the CPU leg below computes ---------------------------
    call(handles[-1], dv, dout, args.batch, stream)
    torch.cuda.synchronize()
    got = dout.cpu().numpy()

    # ---- timed region -------------------------------------------------------------------------------
    lib = R.load()
    fn = lib.rsr_matvec if args.dtype == "f32" else lib.rsr_matvec_i8
    if dense_mode:
        fn = lib.rsr_dense_matvec if args.dtype == "f32" else lib.rsr_dense_matvec_i8
    pv, po = dv.data_ptr(), dout.data_ptr()

    def run(n, offset=0):
        for i in range(n):
            rc = fn(handles[(offset + i) % ncopies], pv, po, args.batch, stream)
            if rc != 0:
                raise RuntimeError(R.rsr_last_error())

    # Untimed conditioning before the W warm-up steps: the same product for a few tens of milliseconds, so that
    # a short timed region (the default driver run times 20 steps) sees the device at its steady clock.
    if not args.plain:
        run(PRECONDITION_LAUNCHES)
        torch.cuda.synchronize()
    run(args.warmup)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    ev0.record()
    run(args.steps, args.warmup)
    ev1.record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    dev_ms = ev0.elapsed_time(ev1)

    if args.copy_calibration > 0:
        # reads 256 MiB and writes 256 MiB per copy; distinct buffers, larger than the last-level cache
        src = torch.empty(256 << 20, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        for _ in range(args.copy_calibration):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    # ---- spread of the launch duration (groups of ten launches, cold rotation continues) and the warm figure
    per_group, warm_us = [None], None
    if not args.plain:
        group, ngroups = 10, max(5, min(100, args.steps // 10))
        evs = [torch.cuda.Event(enable_timing=True) for _ in range(ngroups + 1)]
        evs[0].record()
        for gi in range(ngroups):
            run(group, args.warmup + args.steps + gi * group)
            evs[gi + 1].record()
        torch.cuda.synchronize()
        per_group = sorted(evs[gi].elapsed_time(evs[gi + 1]) * 1e3 / group for gi in range(ngroups))
        wsteps = max(20, min(args.steps, 1000))
        for _ in range(20):
            fn(handles[0], pv, po, args.batch, stream)
        torch.cuda.synchronize()
        w0, w1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        w0.record()
        for _ in range(wsteps):
            fn(handles[0], pv, po, args.batch, stream)
        w1.record()
        torch.cuda.synchronize()
        warm_us = w0.elapsed_time(w1) * 1e3 / wsteps

    # ---- independent products on two streams (context, never `value`): the start of one launch overlaps the
    #      end of its neighbour, which is what a serving loop with independent requests sees ---------------------
    two_stream_us = None
    pairs = ncopies // 2 * 2  # (an even number of copies: no handle is used on both streams at once)
    if not args.plain and not dense_mode and pairs:
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        dout2 = torch.zeros_like(dout)
        targets = ((s1.cuda_stream, po), (s2.cuda_stream, dout2.data_ptr()))
        tsteps = max(40, min(args.steps, 2000)) // 2 * 2

        def run2(n):
            for i in range(n):   # handle i on stream i % 2
                st_, out_ = targets[i % 2]
                if fn(handles[i % pairs], pv, out_, args.batch, st_) != 0:
                    raise RuntimeError(R.rsr_last_error())

        torch.cuda.synchronize()
        run2(100)
        torch.cuda.synchronize()
        b1, b2, f1, f2 = (torch.cuda.Event(enable_timing=True) for _ in range(4))
        b1.record(s1); b2.record(s2)
        run2(tsteps)
        f1.record(s1); f2.record(s2)
        torch.cuda.synchronize()
        two_stream_us = max(b1.elapsed_time(f1), b1.elapsed_time(f2), b2.elapsed_time(f1), b2.elapsed_time(f2)) * 1e3 / tsteps

    ms_per_step = wall * 1e3 / args.steps
    launch_us = dev_ms * 1e3 / args.steps
    elem = 4 if args.dtype == "f32" else 1
    io_bytes = args.batch * (rows * elem + cols * 4)
    method_bytes = int(info.parts) * int(info.nblocks) * (rows * 2 + (1 << w.k) * 2) + io_bytes
    stored_bytes = table_bytes + io_bytes
    achieved = method_bytes / (launch_us * 1e-6) / 1e9
    prof = PROFILED_TRAFFIC.get((args.workload, args.batch, args.dtype, args.regime))

    result = {
        "metric": "RSR++ v.A matvecs/s at n=16384; achieved HBM GB/s vs peak"
                  if args.workload == "binary_16k" else f"RSR++ v.A matvecs/s ({args.workload})",
        "value": args.batch * args.steps / wall,
        "unit": "matvecs/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": args.dtype,
        "data": "synthetic",
        "config": {
            "workload": f"{w.name}: {w.kind} {rows}x{cols}, k={w.k}, batch {args.batch}, {args.dtype} activations",
            "regime": args.regime,
            "step2": args.step2,
            "index_copies_rotated": ncopies,
            "untimed_conditioning_launches": 0 if args.plain else PRECONDITION_LAUNCHES,
            "working_set_bytes": ncopies * table_bytes,
            "table_bytes": table_bytes,
            "stored_rows": int(info.stored_rows),
            "segments": int(info.segments),
            "work_units": int(info.work_units),
            "parity_worst_error_over_bound": None,
        },
        "roofline": {
            "bound": "hbm",
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": prof["traffic_bytes"] if prof and prof["table_bytes"] == table_bytes else None,
            "traffic_source": (prof["source"] + " (measured offline)") if prof and prof["table_bytes"] == table_bytes else None,
            "algorithmic_bytes_per_launch": method_bytes,
            "stored_bytes_per_launch": stored_bytes,
            "stored_frac": stored_bytes / (launch_us * 1e-6) / 1e9 / HBM_PEAK_GBS,
            "launch_us": launch_us,
            "launch_us_median": per_group[len(per_group) // 2],
            "launch_us_min": per_group[0],
            "warm_launch_us": warm_us,
            "two_stream_us_per_product": two_stream_us,
            "note": "priced against HBM as the metric asks; beside the stream the launch is bound by the LDS of the compute units (a gather "
                    "per row and vector, a store per 64 segments) and by its start",
        },
    }
    if not args.no_cpu:
        result["cpu_baseline"], exact = cpu_baseline(A, v, args.dtype, args.cpu_seconds)
        if not args.no_check:
            if args.dtype == "f32":
                bound = 1e-5 * np.abs(v.astype(np.float64)).sum(axis=1, keepdims=True)
                parity = float((np.abs(got.astype(np.float64) - exact) / bound).max())
                if not parity <= 1.0:
                    print(f"parity FAILED: error is {parity:.3g} x the allowed 1e-5*sum|v|", file=sys.stderr)
                    sys.exit(1)
            else:
                if not np.array_equal(got.astype(np.int64), exact):
                    print("parity FAILED: int8 product is not exact", file=sys.stderr)
                    sys.exit(1)
                parity = 0.0
            result["config"]["parity_worst_error_over_bound"] = parity
    torch.cuda.synchronize()
    for h in handles:
        (R.rsr_dense_destroy if dense_mode else R.rsr_destroy)(h)
    if dense_mode:
        result["metric"] = f"bit-packed comparator v.A matvecs/s ({args.workload})"
        result["config"]["comparator"] = "dense bit-packed matrix with a table of sums per four rows (two kernels per product)"
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
