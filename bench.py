#!/usr/bin/env python3
"""Benchmark of the GCN hot path on one MI355X.

The default run measures three of the benchmark configurations, one after the other, on
synthetic inputs that are resident in HBM before each timed region, and prints ONE JSON line:

  headline   config 4, the largest configuration one GPU holds: one GCN layer 128 -> 128,
             forward + backward, on the power-law graph with N = 1.11e8 nodes and 3.3e9
             stored entries (the three-layer model's activations do not fit 288 GB, the paper
             spreads them over 32 GPUs; one layer at its real shape does).  If it cannot run
             (not enough device memory on this machine), config 3 and then config 2 take its
             place and the line says so.
  secondary  config 2 (3-layer GCN 128-256-256-16, R-MAT scale 20, fp32), one epoch,
             config 5 (3-layer GCN 100-256-256-47, N = 2.45e6, bf16 storage), one epoch, and
             config 3 (one layer 128 -> 1024 on a 128-column slice, R-MAT scale 24, fp32).

`value` is whole-job throughput in edges*feat/s: sum over layers of nnz(A_hat) * d^(l), divided
by the step time.  `roofline` describes the dominant kernel (the aggregation gather): its
algorithmic bytes per launch over its average launch duration, taken from HIP events that the
library records around that kernel on the kernel's own stream inside the timed region.
`cpu_baseline` is the CPU oracle as it stands, timed on this host on a bounded, down-scaled
sample of the headline workload (median of three runs after a warm-up).

`--config c1|c2|c3|c4|c5` runs that configuration alone (the form the profiles under profiles/
were taken with).
"""
from __future__ import annotations

import argparse
import gc
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0       # MI355X published HBM3E bandwidth
MFMA_F32_TFLOPS = 157.3     # published dense fp32 matrix rate
MFMA_BF16_TFLOPS = 2500.0   # published dense bf16 matrix rate
KIND_NAMES = ["agg_g4", "agg_g8", "agg_g16", "agg_g32", "agg_g64", "update_fwd", "update_dgrad",
              "update_wgrad"]
# rocprofv3 --pmc summaries (committed) that hold the HBM traffic of the dominant kernel
TRAFFIC_FILES = {("c2", 256): "c2_aggregate_pmc.txt", ("c3", 128): "c3_aggregate_pmc.txt",
                 ("c4", 128): "c4_aggregate_pmc.txt", ("c5", 256): "c5_aggregate_pmc.txt"}


def measured_traffic(config, width):
    """HBM bytes per launch of the dominant kernel and where the figure comes from: the
    committed rocprofv3 --pmc summary of this same workload.  Hardware counters cannot be read
    from inside the run, so this is NOT measured by the run that prints it."""
    name = TRAFFIC_FILES.get((config, width))
    if name is None:
        return None, None
    path = os.path.join(ROOT, "profiles", name)
    try:
        for line in open(path):
            if line.startswith("traffic_bytes_per_launch"):
                return float(line.split()[1]), (f"profiles/{name} (committed rocprofv3 --pmc summary of "
                                                f"this workload; not re-measured in this run)")
    except OSError:
        pass
    return None, None


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def model_dims(name):
    return {"c1": [64, 32, 8], "c2": [128, 256, 256, 16], "c4": [128, 128, 128, 172],
            "c5": [100, 256, 256, 47]}[name]


def make_inputs(name, scale, seed, scramble=True):
    import graphgen as gg

    dims = model_dims(name)
    src, dst, n = gg.config_graph(name, seed=seed, scale_override=scale, scramble=scramble)
    if name in ("c1", "c5"):
        x = gg.uniform(seed, 1, n, dims[0])
    else:
        x = gg.normal(seed, 1, n, dims[0])
    # weights with a leading dimension of whole 16-byte groups (47 columns -> ld 48)
    ws = [gg.glorot(seed, 10 + l, dims[l], dims[l + 1], ld=(dims[l + 1] + 3) // 4 * 4)[:, :dims[l + 1]]
          for l in range(len(dims) - 1)]
    y = gg.labels(seed, 5, n, dims[-1])
    return src, dst, n, x, ws, y, dims


def timed_median(fn, runs=3):
    """One warm-up call, then `runs` timed calls; returns (median seconds, all timed seconds)."""
    fn()
    ts = []
    for _ in range(runs):
        t0 = time.perf_counter()
        fn()
        ts.append(time.perf_counter() - t0)
    return statistics.median(ts), ts


def cpu_baseline_model(name, scale, seed, single_thread_scale=None):
    """The oracle on the host cores: one forward+backward step of a down-scaled instance of the
    same generator and model (median of 3 after a warm-up); optionally also one thread on a
    smaller instance."""
    import numpy as np

    import oracle

    def prepare(sc):
        src, dst, n, x, ws, y, dims = make_inputs(name, sc, seed)
        g = oracle.transpose(oracle.normalize(oracle.build_csr(src, dst, n)))
        ws = [np.ascontiguousarray(w) for w in ws]
        q = oracle.Q_BF16 if name == "c5" else oracle.Q_NONE
        return g, n, dims, (lambda: oracle.gcn_step(g, x, ws, y, q=q))

    g, n, dims, step = prepare(scale)
    med, ts = timed_median(step)
    work = sum(g.nnz * d for d in dims[:-1])
    out = {
        "value": work / med, "unit": "edges*feat/s", "cores": oracle.num_threads(), "kind": "oracle",
        "cpu_model": cpu_model(), "median_s": med,
        "sample": f"{name} recipe at scale {scale} (N={n}, nnz={g.nnz}), one fwd+bwd step, "
                  f"median of 3 after a warm-up",
    }
    if single_thread_scale:
        g1, n1, dims1, step1 = prepare(single_thread_scale)
        threads = oracle.num_threads()
        oracle.set_num_threads(1)
        try:
            med1, ts1 = timed_median(step1)
        finally:
            oracle.set_num_threads(threads)
        out["single_thread"] = {
            "value": sum(g1.nnz * d for d in dims1[:-1]) / med1, "unit": "edges*feat/s", "cores": 1,
            "median_s": med1,
            "sample": f"{name} recipe at scale {single_thread_scale} (N={n1}, nnz={g1.nnz}), one thread"}
    return out


def cpu_baseline_layer(name, scale, seed, k, m, relu):
    """The oracle on the host cores for the single-layer workloads (configs 3 and 4): Z = A_hat H,
    H' = sigma(Z W), dW = Z^T dP, dZ = dP W^T, dH = A_hat^T dZ on a down-scaled instance of the
    same graph generator, median of 3 after a warm-up."""
    import numpy as np

    import graphgen as gg
    import oracle

    if name == "c3":
        n = 1 << scale
        src, dst = gg.rmat_edges(seed, scale, 8 * n)
    else:
        src, dst, n = gg.config_graph("c4", seed, scale)
    g = oracle.transpose(oracle.normalize(oracle.build_csr(src, dst, n)))
    h = gg.normal(seed, 1, n, k).astype(np.float64)
    w = gg.glorot(seed, 10, k, m).astype(np.float64)
    grad = gg.normal(seed, 3, n, m).astype(np.float64)

    def step():
        z = oracle.spmm(g, h)
        out = oracle.update_fwd(z, w, relu)
        dp = oracle.relu_grad(grad, out if relu else None)
        oracle.update_wgrad(z, dp)
        oracle.spmm(g, oracle.update_dgrad(dp, w), transposed=True)

    med, ts = timed_median(step)
    return {
        "value": g.nnz * k / med, "unit": "edges*feat/s", "cores": oracle.num_threads(),
        "kind": "oracle", "cpu_model": cpu_model(), "median_s": med,
        "sample": f"{name} graph recipe at scale {scale} (N={n}, nnz={g.nnz}), one layer {k}->{m} "
                  f"fwd+bwd, median of 3 after a warm-up",
    }


def read_kinds(pipe):
    kinds = {}
    for i, nm in enumerate(KIND_NAMES):
        ms, cnt = pipe.timing_read(i)
        if cnt:
            kinds[nm] = {"total_ms": ms, "launches": cnt, "avg_ms": ms / cnt}
    return kinds


def kernels_compact(kinds):
    """{kind: [average ms per launch, launches]} for the printed line."""
    return {k: [v["avg_ms"], v["launches"]] for k, v in kinds.items()}


def update_rate(kind, tflops, arith):
    """Rate of an update product of fp32 features against the matrix rate of its arithmetic: the fp32 MFMA
    for the forward product, a sixth of the bf16 MFMA for six products of bf16 terms each."""
    if kind == "update_fwd" and arith == "fp32":
        return {"tflops": tflops, "frac_of_fp32_mfma_peak": tflops / MFMA_F32_TFLOPS}
    return {"tflops": tflops, "frac_of_sixth_of_bf16_mfma_peak": tflops / (MFMA_BF16_TFLOPS / 6.0)}


def aggregation_roofline(config, kinds, nnz, n, esz, chunks=1):
    """Roofline block of the aggregation launch that takes the most time of the step."""
    agg = {k: v for k, v in kinds.items() if k.startswith("agg")}
    if not agg:
        return None
    dom = max(agg, key=lambda k: agg[k]["total_ms"])
    gsz = int(dom.split("g")[-1])
    f = gsz * 16 // esz  # columns of a pass of that width class (16 bytes per lane)
    # algorithmic minimum per full-graph launch: the entry stream (column + value) once, every
    # feature row read once, every output row written once, one row pointer per row
    per_launch = (8.0 * nnz + 2.0 * n * f * esz + 8.0 * n) / max(1, chunks)
    no_reuse = (nnz * (8.0 + f * esz) + n * f * esz) / max(1, chunks)
    avg_s = agg[dom]["avg_ms"] * 1e-3
    achieved = per_launch / avg_s / 1e9
    traffic, source = measured_traffic(config, f) if chunks == 1 else (None, None)
    out = {
        "bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
        "frac": achieved / HBM_PEAK_GBS, "traffic": traffic, "traffic_source": source,
        "kernel": f"aggregate_kernel<8, {gsz}, {1 if esz == 2 else 0}, ...> "
                  f"({f} {'bf16' if esz == 2 else 'fp32'} columns)",
        "avg_launch_ms": agg[dom]["avg_ms"], "launches": agg[dom]["launches"],
        "algorithmic_bytes_per_launch": per_launch,
        "no_reuse_bytes_per_launch": no_reuse,
        "no_reuse_GBps": no_reuse / avg_s / 1e9,
    }
    if traffic:
        out["counter_traffic_GBps"] = traffic / avg_s / 1e9
        out["counter_traffic_frac"] = traffic / avg_s / 1e9 / HBM_PEAK_GBS
    return out


def bench_single_layer(args, mg, dev, config):
    """Configs 3 and 4: one layer forward + backward at the real shape.

    c3: a 128-column slice of a 1024-wide layer, R-MAT scale 24 with 8 N directed edges; H comes
    from the seeded generator, the 68.7 GB upstream gradient G is drawn on the device.
    c4: N = 1.11e8 with 1.6e9 power-law directed edges, one 128 -> 128 layer in the last-layer
    form (no ReLU).  Three N x 128 tensors (56.8 GB each) plus the graph (54 GB) are resident:
    the upstream gradient reuses the layer output's storage and dH is written over H, which the
    backward pass no longer reads.  Tensor values are drawn on the device (they do not matter for
    the timing; parity at this size is covered by the tests)."""
    import numpy as np
    import torch

    import graphgen as gg
    from paper_2501_01951_amd.model import padded_rows

    t_gen = time.perf_counter()
    if config == "c3":
        scale = args.scale or 24
        n, k, m, relu = 1 << scale, 128, 1024, True
        src, dst = gg.rmat_edges(args.seed, scale, 8 * n)
        what = f"c3: one GCN layer 128->1024 fwd+bwd, R-MAT scale {scale}"
    else:
        src, dst, n = gg.config_graph("c4", args.seed, args.scale)
        k, m, relu = 128, 128, False
        what = "c4: one GCN layer 128->128 fwd+bwd (no ReLU), power-law graph"
    t_gen = time.perf_counter() - t_gen
    s_d, d_d = dev(src.view(np.int32)), dev(dst.view(np.int32))
    del src, dst
    torch.cuda.synchronize()
    t_build = time.perf_counter()
    g = mg.build_csr(s_d, d_d, n)
    del s_d, d_d
    torch.cuda.empty_cache()
    mg.normalize(g)
    torch.cuda.synchronize()
    t_build = time.perf_counter() - t_build
    nnz = g.nnz
    hd = padded_rows(n, k, torch.float32, "cuda")
    if config == "c3":
        hd.copy_(torch.from_numpy(gg.normal(args.seed, 1, n, k)))
    else:
        hd.normal_()
    wd = dev(gg.glorot(args.seed, 10, k, m))
    zd = padded_rows(n, k, torch.float32, "cuda")
    outd = padded_rows(n, m, torch.float32, "cuda")
    if config == "c3":
        gd = padded_rows(n, m, torch.float32, "cuda")
        gd.normal_()
        dhd = padded_rows(n, k, torch.float32, "cuda")
    else:
        gd, dhd = outd, hd
    dwd = torch.empty(k, m, device="cuda")
    pipe = mg.Pipeline()

    def step():
        mg.layer_fwd(g, hd, wd, zd, outd, pipe, relu=relu, n_chunks=args.chunks)
        mg.layer_bwd(g, zd, outd, wd, gd, dwd, dhd, pipe, relu=relu, n_chunks=args.chunks)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    pipe.timing(True)
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / args.steps
    kinds = read_kinds(pipe)
    pipe.timing(False)
    # The same layer with the fine-grain pipeline of Sec. 3.2.2 (aggregation of row chunk k on one
    # stream while the update of chunk k - 1 runs on the other), after and outside the timed
    # region above: reported beside the result.
    pipelined = None
    if args.chunks == 1 and not args.no_pipelined:
        nc = 16

        def step_chunked():
            mg.layer_fwd(g, hd, wd, zd, outd, pipe, relu=relu, n_chunks=nc)
            mg.layer_bwd(g, zd, outd, wd, gd, dwd, dhd, pipe, relu=relu, n_chunks=nc)

        step_chunked()
        torch.cuda.synchronize()
        reps = max(1, min(5, args.steps))
        t0 = time.perf_counter()
        for _ in range(reps):
            step_chunked()
        torch.cuda.synchronize()
        dtc = (time.perf_counter() - t0) / reps
        pipelined = {"row_chunks": nc, "steps": reps, "ms_per_step": dtc * 1e3, "value": nnz * k / dtc,
                     "speedup_over_unpipelined": dt / dtc}
    out = {
        "metric": "GCN layer fwd+bwd edges*feat/s", "value": nnz * k / dt, "unit": "edges*feat/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": dt * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": f"{what}, N={n}, nnz(A_hat)={nnz}", "n_nodes": n, "nnz": nnz,
                   "row_chunks": args.chunks, "seed": args.seed, "update_arith": args.update_arith},
        "generate_edges_s": t_gen, "build_csr_normalize_ms": t_build * 1e3,
        "kernels_avg_ms_launches": kernels_compact(kinds),
        "roofline": aggregation_roofline(config, kinds, nnz, n, 4, args.chunks),
        "update_products": {
            kk: update_rate(kk, 2.0 * n * k * m / (kinds[kk]["avg_ms"] * 1e-3) / 1e12, args.update_arith)
            for kk in ("update_fwd", "update_dgrad", "update_wgrad") if kk in kinds},
    }
    if pipelined:
        out["with_row_chunk_pipeline"] = pipelined
    pipe.free()
    g.free()
    del hd, zd, outd, gd, dhd, dwd, wd
    gc.collect()
    torch.cuda.empty_cache()
    return out


def bench_model(args, mg, dev, config, with_bf16x3=True):
    """Configs 1, 2 and 5: one epoch (forward + loss + backward) of the multi-layer GCN."""
    import numpy as np
    import torch

    t_gen = time.perf_counter()
    src, dst, n, x, ws, y, dims = make_inputs(config, args.scale, args.seed, not args.unscrambled)
    t_gen = time.perf_counter() - t_gen
    s_d, d_d = dev(src.view(np.int32)), dev(dst.view(np.int32))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    g = mg.build_csr(s_d, d_d, n)
    mg.normalize(g)
    torch.cuda.synchronize()
    t_build = time.perf_counter() - t0
    nnz = g.nnz
    del s_d, d_d, src, dst

    pipe = mg.Pipeline()
    bf16 = config == "c5"  # config 5 stores features in bf16
    x_d = torch.from_numpy(x).cuda()
    if bf16:
        x_d = x_d.to(torch.bfloat16)
    w_d = [torch.from_numpy(np.ascontiguousarray(w.base if w.base is not None else w)).cuda()[:, :w.shape[1]]
           for w in ws]
    step = mg.GCNStep(g, x_d, w_d, dev(y), n_chunks=args.chunks, pipe=pipe)

    run_step = step.step
    if args.hip_graph:
        assert args.chunks == 1, "--hip-graph times the single-stream schedule"
        step.capture()
        run_step = step.replay
    for _ in range(args.warmup):
        run_step()
    torch.cuda.synchronize()
    timing = not (args.no_event_timing or args.hip_graph)
    pipe.timing(timing)
    t0 = time.perf_counter()
    for _ in range(args.steps):
        run_step()
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / args.steps
    loss = step.loss.item()
    work = sum(nnz * d for d in dims[:-1])  # sum over layers of nnz * d^(l)
    kinds = read_kinds(pipe) if timing else {}
    pipe.timing(False)
    esz = 2 if bf16 else 4
    out = {
        "metric": "GCN layer fwd+bwd edges*feat/s", "value": work / dt, "unit": "edges*feat/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": dt * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16 storage, f32 accumulate" if bf16 else "f32", "data": "synthetic",
        "config": {
            "workload": f"{config}: {len(dims) - 1}-layer GCN {'-'.join(map(str, dims))}, one "
                        f"fwd+bwd epoch, {'Erdos-Renyi' if config == 'c1' else 'R-MAT'} graph "
                        f"N={n}, nnz(A_hat)={nnz}",
            "n_nodes": n, "nnz": nnz, "row_chunks": args.chunks, "seed": args.seed,
            "hip_graph": bool(args.hip_graph), "update_arith": args.update_arith,
            "aggregate_whole_rows": bool(args.whole_rows), "rmat_ids_scrambled": not args.unscrambled,
        },
        "loss": loss, "generate_inputs_s": t_gen, "build_csr_normalize_ms": t_build * 1e3,
        "kernels_avg_ms_launches": kernels_compact(kinds),
        "roofline": aggregation_roofline(config, kinds, nnz, n, esz, args.chunks),
    }
    upd = sum(v["total_ms"] for k, v in kinds.items() if k.startswith("update")) / args.steps
    if kinds:
        out["update_products_ms_per_step"] = upd
        flops = sum(2.0 * n * dims[l] * dims[l + 1] * (3 if l > 0 else 2) for l in range(len(dims) - 1))
        out["update_products_tflops"] = flops / (upd * 1e-3) / 1e12
    # the same steps with the opt-in arithmetic of the forward product (fp32 operands as three bf16 terms
    # on the bf16 matrix cores, as the gradients always have them), after and outside the timed region
    # above: reported beside the result
    if with_bf16x3 and args.update_arith == "fp32" and not bf16 and not args.hip_graph:
        mg.set_update_arith(mg.ARITH_BF16X3)
        try:
            for _ in range(2):
                run_step()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(args.steps):
                run_step()
            torch.cuda.synchronize()
            dt3 = (time.perf_counter() - t0) / args.steps
            out["with_update_arith_bf16x3"] = {"ms_per_step": dt3 * 1e3, "value": work / dt3,
                                               "loss": step.loss.item()}
        finally:
            mg.set_update_arith(mg.ARITH_FP32)
    pipe.free()
    g.free()
    del step, x_d, w_d
    gc.collect()
    torch.cuda.empty_cache()
    return out


def bench_variant(args, mg, dev):
    """--model sage | gin (not the default line): the paper's two other architectures, three
    layers with 128 hidden units, on the graph and features of the chosen configuration."""
    import numpy as np
    import torch

    import graphgen as gg

    src, dst, n = gg.config_graph(args.config, seed=args.seed, scale_override=args.scale)
    d0 = model_dims(args.config)[0]
    classes = model_dims(args.config)[-1]
    dims = [d0, 128, 128, classes]
    x = gg.normal(args.seed, 1, n, d0)
    y = gg.labels(args.seed, 5, n, classes)
    sage = args.model == "sage"
    flags = mg.SYMMETRIZE | (0 if sage else mg.ADD_SELF_LOOPS)
    g = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), n, flags)
    mg.normalize(g, mg.NORM_MEAN if sage else mg.NORM_SUM, eps=0.0 if sage else 0.1)
    nnz = g.nnz
    if sage:
        ws = [dev(gg.glorot(args.seed, 20 + l, 2 * dims[l], dims[l + 1])) for l in range(3)]
        step = mg.SAGEStep(g, dev(x), ws, dev(y))
        agg_in, agg_out = step.xc[1][:, :128], step.xc[1][:, 128:256]
    else:
        w1s = [dev(0.02 * gg.glorot(args.seed, 30 + l, dims[l], 128)) for l in range(3)]
        w2s = [dev(gg.glorot(args.seed, 40 + l, 128, dims[l + 1])) for l in range(3)]
        step = mg.GINStep(g, dev(x), w1s, w2s, dev(y))
        agg_in, agg_out = step.h[1], step.z[1]
    for _ in range(args.warmup):
        step.step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step.step()
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / args.steps
    loss = step.loss.item()
    # the aggregation at the hidden width, timed alone with events on the stream it runs on
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2 * args.steps)]
    for i in range(args.steps):
        ev[2 * i].record()
        mg.aggregate(g, agg_in, agg_out)
        ev[2 * i + 1].record()
    torch.cuda.synchronize()
    agg_ms = sum(ev[2 * i].elapsed_time(ev[2 * i + 1]) for i in range(args.steps)) / args.steps
    per_launch = 8.0 * nnz + 2.0 * n * 128 * 4 + 8.0 * n
    achieved = per_launch / (agg_ms * 1e-3) / 1e9
    name = "GraphSAGE (mean)" if sage else "GIN (eps = 0.1)"
    out = {
        "metric": f"{name} fwd+bwd edges*feat/s", "value": sum(nnz * d for d in dims[:-1]) / dt,
        "unit": "edges*feat/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": dt * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"{args.config} graph: 3-layer {name} {'-'.join(map(str, dims))}, one "
                               f"fwd+bwd epoch, N={n}, nnz(A_hat)={nnz}",
                   "n_nodes": n, "nnz": nnz, "seed": args.seed, "update_arith": args.update_arith},
        "loss": loss,
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": None, "traffic_source": None,
                     "kernel": "aggregate_kernel<8, 32, 0, false, true> (128 fp32 columns)",
                     "avg_launch_ms": agg_ms, "algorithmic_bytes_per_launch": per_launch},
    }
    if not args.no_cpu_baseline:
        import oracle

        s2, d2, n2 = gg.config_graph(args.config, seed=args.seed, scale_override=args.cpu_scale)
        og = oracle.build_csr(s2, d2, n2, True, not sage)
        og = oracle.transpose(oracle.normalize_mean(og) if sage else oracle.normalize_sum(og, 0.1))
        x2, y2 = gg.normal(args.seed, 1, n2, d0), gg.labels(args.seed, 5, n2, classes)
        t0 = time.perf_counter()
        if sage:
            oracle.sage_step(og, x2, [gg.glorot(args.seed, 20 + l, 2 * dims[l], dims[l + 1])
                                      for l in range(3)], y2)
        else:
            oracle.gin_step(og, x2, [0.02 * gg.glorot(args.seed, 30 + l, dims[l], 128) for l in range(3)],
                            [gg.glorot(args.seed, 40 + l, 128, dims[l + 1]) for l in range(3)], y2)
        t = time.perf_counter() - t0
        out["cpu_baseline"] = {
            "value": sum(og.nnz * d for d in dims[:-1]) / t, "unit": "edges*feat/s",
            "cores": oracle.num_threads(), "kind": "oracle", "cpu_model": cpu_model(),
            "sample": f"same generator and model at R-MAT scale {args.cpu_scale} (N={n2}, "
                      f"nnz={og.nnz}), one fwd+bwd step, {t:.1f} s"}
    print(json.dumps(out))


def rounded(obj, digits=6):
    """The record with every float rounded to `digits` significant digits (keeps the line short)."""
    if isinstance(obj, float):
        return float(f"{obj:.{digits}g}")
    if isinstance(obj, dict):
        return {k: rounded(v, digits) for k, v in obj.items()}
    if isinstance(obj, (list, tuple)):
        return [rounded(v, digits) for v in obj]
    return obj


def summary_of(block):
    """The figures of a secondary block that the headline's `config` carries as well."""
    r = block.get("roofline") or {}
    out = {"ms_per_step": block.get("ms_per_step"), "value": block.get("value"),
           "roofline_frac": r.get("frac"), "roofline_achieved_GBps": r.get("achieved"),
           "counter_traffic_frac": r.get("counter_traffic_frac")}
    if "cpu_baseline" in block:
        out["cpu_baseline_value"] = block["cpu_baseline"].get("value")
    return out


def trimmed(block):
    """A secondary block without the fields that repeat the headline's (metric, unit, step
    counts, peaks): what is left is what differs per configuration."""
    drop = {"metric", "unit", "n_gpus", "steps", "warmup", "higher_is_better", "scaling", "vs_baseline",
            "data", "generate_edges_s", "generate_inputs_s", "build_csr_normalize_ms"}
    out = {k: v for k, v in block.items() if k not in drop}
    out["config"] = {"workload": block["config"]["workload"]}
    if out.get("roofline"):
        keep = ("bound", "achieved", "frac", "traffic", "traffic_source", "counter_traffic_frac", "kernel",
                "avg_launch_ms", "launches", "algorithmic_bytes_per_launch")
        out["roofline"] = {k: v for k, v in out["roofline"].items() if k in keep}
        if out["roofline"].get("traffic_source"):
            out["roofline"]["traffic_source"] = out["roofline"]["traffic_source"].split(" ")[0]
    return out


def run_config(args, mg, dev, config):
    if config in ("c3", "c4"):
        return bench_single_layer(args, mg, dev, config)
    return bench_model(args, mg, dev, config)


def baseline_for(args, config):
    """Oracle timing for a headline configuration, on a sample that takes the host cores about
    ten to thirty seconds in all."""
    if config == "c4":
        return cpu_baseline_layer("c4", args.cpu_scale or 21, args.seed, 128, 128, False)
    if config == "c3":
        return cpu_baseline_layer("c3", args.cpu_scale or 18, args.seed, 128, 1024, True)
    if config == "c5":
        return cpu_baseline_model("c5", args.cpu_scale or 18, args.seed)
    if config == "c2":
        return cpu_baseline_model("c2", args.cpu_scale or 18, args.seed, single_thread_scale=14)
    return cpu_baseline_model(config, None, args.seed)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", default=None,
                    help="run one configuration alone (c1..c5); default: c4 as the headline with "
                         "c2 and c5 as secondary blocks")
    ap.add_argument("--scale", type=int, default=None, help="override the graph scale (with --config)")
    ap.add_argument("--chunks", type=int, default=1, help="row chunks of the layer pipeline")
    ap.add_argument("--seed", type=int, default=250101951)
    ap.add_argument("--cpu-scale", type=int, default=None, help="graph scale of the oracle sample")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-secondary", action="store_true",
                    help="default run without the secondary configurations")
    ap.add_argument("--no-event-timing", action="store_true")
    ap.add_argument("--no-pipelined", action="store_true",
                    help="single-layer configurations: skip the extra run with 16 row chunks on two streams")
    ap.add_argument("--no-peaks", action="store_true", help="skip the measured-peaks block")
    ap.add_argument("--model", default="gcn", choices=["gcn", "sage", "gin"],
                    help="gcn: the benchmark line; sage / gin: the two other architectures of the "
                         "paper's experiments on the same graph (3 layers, 128 hidden units)")
    ap.add_argument("--hip-graph", action="store_true",
                    help="record the step into a HIP graph and time its replays (one stream, no "
                         "per-kernel events): for small inputs, where launches dominate")
    ap.add_argument("--unscrambled", action="store_true",
                    help="secondary data point: keep the R-MAT generator's own node numbering "
                         "(hubs at low ids) for configs 2 and 5 instead of the fixed scramble")
    ap.add_argument("--whole-rows", action="store_true",
                    help="measurement aid: aggregations without column slices, the gather a fused "
                         "aggregate->update kernel would do (not the benchmark line)")
    ap.add_argument("--update-arith", default="fp32", choices=["fp32", "bf16x3"],
                    help="matrix-core arithmetic of the forward product of fp32 features: fp32 MFMA "
                         "(the benchmark line) or, for wide layers, three bf16 terms per operand and "
                         "six bf16 MFMAs per product, as the gradients of fp32 features always run")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build runs on exactly one GPU (no collectives are part of it); "
                 "use --gpus 1")

    import numpy as np
    import torch

    import paper_2501_01951_amd as mg

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    mg.load_library()
    torch.cuda.set_device(0)
    mg.set_update_arith(mg.ARITH_BF16X3 if args.update_arith == "bf16x3" else mg.ARITH_FP32)
    mg.set_aggregate_whole_rows(args.whole_rows)

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a)).cuda()

    if args.model != "gcn":
        args.config = args.config or "c2"
        args.cpu_scale = args.cpu_scale or 20
        assert args.config in ("c1", "c2"), "--model sage/gin run on the graphs of c1 and c2"
        return bench_variant(args, mg, dev)

    # A plain copy kernel of known size: its FETCH_SIZE / WRITE_SIZE readings calibrate the
    # counter units when this command runs under rocprofv3 --pmc.
    calib_src = torch.empty(64 * 1024 * 1024, dtype=torch.float32, device="cuda").normal_()
    calib_dst = torch.empty_like(calib_src)
    calib_dst.copy_(calib_src)
    torch.cuda.synchronize()
    del calib_src, calib_dst
    torch.cuda.empty_cache()

    single = args.config is not None
    out, used, fallbacks = None, None, []
    for config in ([args.config] if single else ["c4", "c3", "c2"]):
        try:
            out = run_config(args, mg, dev, config)
            used = config
            break
        except (mg.MixGCNError, torch.OutOfMemoryError, MemoryError) as e:  # too large for this box
            if single:
                raise
            fallbacks.append(f"{config}: {type(e).__name__}: {str(e)[:200]}")
            gc.collect()
            torch.cuda.empty_cache()
    if out is None:
        sys.exit("bench.py: no configuration could run: " + "; ".join(fallbacks))
    if not single:
        out["config"]["headline_choice"] = (
            "largest configuration one GPU holds (config 4, one layer at its real shape); "
            "configs 2, 5 and 3 follow as secondary blocks" if used == "c4" else
            "fallback after: " + "; ".join(fallbacks))
        if not args.no_secondary:
            out["secondary"] = {}
            for config in ("c2", "c5", "c3"):
                if config == used:
                    continue
                try:
                    if config == "c3":
                        out["secondary"][config] = bench_single_layer(args, mg, dev, config)
                    else:
                        out["secondary"][config] = bench_model(args, mg, dev, config,
                                                               with_bf16x3=(config == "c2"))
                except (mg.MixGCNError, torch.OutOfMemoryError, MemoryError) as e:
                    out["secondary"][config] = {"error": f"{type(e).__name__}: {str(e)[:200]}"}
    # what this device sustains on a plain copy and on register-only MFMA chains (outside the
    # timed regions): context for the published peaks the fractions above are quoted against
    if not args.no_peaks:
        try:
            out["measured_peaks"] = mg.measure_peaks()
        except mg.MixGCNError as e:  # needs 8 GiB of free device memory; not part of the result
            out["measured_peaks"] = {"error": str(e)}
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = baseline_for(args, used)
        if not single and not args.no_secondary:
            for config in ("c2", "c5", "c3"):
                blk = out.get("secondary", {}).get(config)
                if blk and "error" not in blk:
                    blk["cpu_baseline"] = baseline_for(args, config)
    try:  # the untrimmed record, for whoever wants every field (best effort, never fatal)
        os.makedirs(os.path.join(ROOT, "gpurun_out"), exist_ok=True)
        with open(os.path.join(ROOT, "gpurun_out", "bench_full.json"), "w") as fh:
            json.dump(out, fh)
    except OSError:
        pass
    if "secondary" in out:
        # the same figures once more inside `config`, for readers that keep only the standard keys
        out["config"]["secondary_configs"] = {k: summary_of(v) for k, v in out["secondary"].items()
                                              if "error" not in v}
        out["secondary"] = {k: (v if "error" in v else trimmed(v)) for k, v in out["secondary"].items()}
    print(json.dumps(rounded(out), separators=(",", ":")))


if __name__ == "__main__":
    main()
