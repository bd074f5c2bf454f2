#!/usr/bin/env python3
"""Benchmark of the MoE-layer hot path on one MI355X.

A step is one call of the fused layer (router, permutation, grouped SwiGLU expert
FFN over paged weights, combine) on one micro-batch of synthetic input that is
already resident in HBM.  Default workload: the Mixtral-8x7B-shaped layer with
4096 tokens, the configuration the headline metric is quoted on.

Prints ONE JSON line: tokens/s of the whole layer, the roofline of the dominant
kernel (the gate/up expert GEMM, measured with HIP events recorded by the
library on the launch stream while the timed steps run again) and the CPU oracle
timed on a bounded sample of the same workload.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0     # MI355X dense bf16 MFMA peak, TFLOP/s
PEAK_HBM_GBS = 8000.0
PEAK_CLOCK_MHZ = 2400.0       # the clock the published peaks are quoted at

# HBM traffic per launch of the gate/up GEMM on the default workload, in bytes, from the
# rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs summarised under profiles/ (None: not measured).
MEASURED_TRAFFIC = {"c3_mixtral8x7b_t4096": 3.416e9, "c2_mixtral8x7b_t256": 1.914e9, "c4_mixtral8x22b_t8192_skew": 2.112e10}


def cpu_model() -> str:
    """The host CPU's model name as the kernel reports it."""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.lower().startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def gate_up_kernel(cfg):
    """The kernel of the gate/up launch: the library's rules (launch_mode in moe_ffn_f32.hip, launch_expert_ffn_bf16 in
    moe_ffn_bf16.hip, thin_takes_gate_up in moe_ffn_thin_bf16.hip)."""
    each = cfg.R // cfg.E
    if cfg.dtype == "f32":
        return "ffn_split_f32<0>" if each > 32 or (each > 16 and cfg.F // 64 * cfg.E >= 256) else "ffn_few_rows_f32<0>"
    if each > 80:
        return "ffn_gemm_bf16<0>"
    experts = cfg.E * (1.0 - (1.0 - cfg.k / cfg.E) ** cfg.T)       # with rows, on average
    return "ffn_thin_bf16<0>" if cfg.T <= 16 and experts * (cfg.F // 64) <= 440 else "ffn_rows_bf16<0>"


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--config", default="c3_mixtral8x7b_t4096")
    ap.add_argument("--cpu-sample-tokens", type=int, default=1024)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--option", action="append", default=[], help="library option name=value")
    ap.add_argument("--shuffle-host-pages", action="store_true",
                    help="streamed workloads: place the pages in pinned host memory in a random order, so that every "
                         "page is a copy of its own (in order, the runs of consecutive pages of an expert go out as one copy)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="instead of the layer, run a plain device copy of 1 GiB ten times (calibrates the "
                         "FETCH_SIZE / WRITE_SIZE counters of rocprofv3 --pmc against known traffic)")
    ap.add_argument("--pipeline", action="store_true",
                    help="instead of the headline step, time the multi-layer weight-paging pipeline (moe_pipeline_run) "
                         "on --config's layer shape: --layers layers (sharing one set of host pages), --micro-batches "
                         "micro-batches of T / micro-batches tokens, --resident-fraction of every expert's pages kept in HBM")
    ap.add_argument("--tasks", action="store_true",
                    help="instead of the headline step, time the post-attention task (O projection, residual + norm, MoE "
                         "layer) and the pre-attention task (residual + norm, QKV projection) on --config's layer shape, "
                         "with attention width H and a QKV width of 1.5 H (32 query and 8 key/value heads of 128)")
    ap.add_argument("--prefill", action="store_true",
                    help="instead of the headline step, time a prefill pass of a request batch through --config's layer "
                         "(weights resident): --requests seeded prompt lengths (average 77, maximum 418) are packed into "
                         "micro-batches of --ubs requests by paper_2411_11217_amd.batching, and a step runs moe_layer once "
                         "per micro-batch on that micro-batch's prompt tokens")
    ap.add_argument("--mu-sweep", action="store_true",
                    help="instead of the headline step, time moe_layer on --config's layer shape (weights resident) for "
                         "micro-batch sizes 32 .. 4096: the memory-bound plateau of the decode stage (the paper's section "
                         "6.2 sweeps 32 .. 256) and the turn to compute bound beyond it")
    ap.add_argument("--vendor-gemm", action="store_true",
                    help="instead of the layer, time the vendor GEMM library (torch.matmul, bf16) and this library's paged linear "
                         "map on three dense shapes, same box, same data, same warm state")
    ap.add_argument("--splits", action="store_true",
                    help="instead of the layer, time the two expert GEMMs (moe_expert_ffn) of the workload's shape for several ways "
                         "of splitting its rows over the experts: what raggedness costs")
    ap.add_argument("--sample-power", action="store_true",
                    help="after the timed steps run the step for a few seconds more while `amd-smi metric --power --clock --json` is "
                         "polled beside it; board power and the XCDs' clocks go into the JSON line")
    ap.add_argument("--two-streams", action="store_true",
                    help="--mu-sweep: also time two micro-batches at a time, each on a stream and a workspace of its own")
    ap.add_argument("--mu-list", default="", help="--mu-sweep: comma-separated micro-batch sizes instead of the default 32 .. 4096")
    ap.add_argument("--rate-probes", action="store_true",
                    help="instead of the layer, measure the three rates the roofline model takes as its inputs, each with a "
                         "probe that is none of the layer runs the model is then asked to predict: the host link with a "
                         "pinned-to-device copy of 1 GiB, the read rate of device memory with a kernel of nothing but loads "
                         "over 4 GiB, and the matrix rate with a dense bf16 product of 2048 x 8192 x 32768 through the paged "
                         "linear map")
    ap.add_argument("--requests", type=int, default=1024)
    ap.add_argument("--ubs", type=int, default=128)
    ap.add_argument("--layers", type=int, default=2)
    ap.add_argument("--micro-batches", type=int, default=4)
    ap.add_argument("--resident-fraction", type=float, default=0.5)
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (no collectives, no sharding); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2411_11217_amd as M
    from moe_workloads import CONFIGS, make_inputs, oracle_view

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    if args.copy_probe:
        n = 1 << 30
        src = torch.empty(n, dtype=torch.uint8, device="cuda").fill_(3)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        for _ in range(10):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes_read": n, "copy_probe_bytes_written": n, "launches": 10}))
        return
    if args.rate_probes:
        return rate_probes(args, M)
    if args.vendor_gemm:
        return vendor_gemm_bench(args, M)
    cfg = CONFIGS[args.config]
    for o in args.option:
        name, val = o.split("=")
        M.set_option(name, int(val))
    if args.pipeline:
        return pipeline_bench(args, cfg, M, make_inputs)
    if args.tasks:
        return tasks_bench(args, cfg, M, make_inputs)
    if args.prefill:
        return prefill_bench(args, cfg, M, make_inputs)
    if args.mu_sweep:
        return mu_sweep_bench(args, cfg, M, make_inputs)
    if args.splits:
        return splits_bench(args, cfg, M, make_inputs)
    s = M.make_shape(cfg.T, cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes)
    t0 = time.time()
    inp = make_inputs(cfg, threads=16)
    order = torch.Generator().manual_seed(1) if (cfg.streamed and args.shuffle_host_pages) else None
    pw = M.PagedWeights(s, inp["W1"], inp["W3"], inp["W2"], pin=cfg.streamed, order=order)
    x, Wr = inp["x"].cuda(), inp["Wr"].cuda()
    bias = None if inp["bias"] is None else inp["bias"].cuda()
    streamer = None
    if cfg.streamed:
        streamer = M.Streamer(s, pw.pages_host, pw.table_host)
    else:
        pw.to_device(keep_host=False)
    ws = M.Workspace(s)
    y = torch.empty((cfg.T, cfg.H), dtype=torch.float32, device="cuda")
    print(f"[bench] inputs ready in {time.time() - t0:.1f}s", file=sys.stderr, flush=True)

    def step():
        if streamer is not None:
            M.moe_layer_streamed(streamer, x, Wr, bias=bias, workspace=ws, y=y)
        else:
            M.moe_layer(s, x, Wr, pw.table_dev, pw.pages_dev, bias=bias, workspace=ws, y=y)

    # part of the set-up, whatever --warmup says: code objects loaded, clocks and power state settled
    for _ in range(10 if streamer is None else 1):
        step()
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_per_step = elapsed * 1e3 / args.steps
    tokens_per_s = cfg.T / (ms_per_step * 1e-3)

    # the spread over single steps (events around every step, outside the timed region above)
    n_ev = min(args.steps, 100)
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(n_ev + 1)]
    evs[0].record()
    for i in range(n_ev):
        step()
        evs[i + 1].record()
    torch.cuda.synchronize()
    per_step = sorted(evs[i].elapsed_time(evs[i + 1]) for i in range(n_ev))
    spread = {"n": n_ev, "median": round(per_step[n_ev // 2], 4), "min": round(per_step[0], 4), "max": round(per_step[-1], 4)}

    # the same steps again with the library's stage events on (HIP events on the launch stream)
    stages, n_prof = {}, 0
    if streamer is None:
        M.set_option("profile", 1)
        for _ in range(min(args.steps, 200)):
            step()
        torch.cuda.synchronize()
        stages, n_prof = M.profile_read()
        M.set_option("profile", 0)
    flops_gu = 4.0 * cfg.R * cfg.H * cfg.F            # gate/up GEMM: 2 * R * H * 2F
    flops_ffn = cfg.ffn_flops
    roofline = None
    if stages:
        t_gu = stages["gemm_gate_up"] * 1e-3
        achieved = flops_gu / t_gu / 1e12
        kernel = gate_up_kernel(cfg)
        roofline = {"bound": "mfma", "kernel": kernel + " (gate/up expert GEMM + SwiGLU epilogue)",
                    "achieved": round(achieved, 2), "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                    "frac": round(achieved / PEAK_BF16_TFLOPS, 4), "traffic": MEASURED_TRAFFIC.get(args.config),
                    "avg_launch_ms": round(stages["gemm_gate_up"], 4), "launches_timed": n_prof}
        # Few rows per expert (at most half a row tile on average): the launch streams the weights once and HBM is its
        # roof.  Algorithmic bytes: both weight matrices of every expert, x, and h written (f32: and the permuted rows).
        esize = 2 if cfg.dtype == "bf16" else 4
        if cfg.R <= 128 * cfg.E:
            gu_bytes = 2.0 * cfg.E * cfg.H * cfg.F * esize + cfg.T * cfg.H * esize + cfg.R * cfg.F * esize
            if cfg.dtype == "f32" and M.get_option("fuse_gather"):
                gu_bytes += cfg.R * cfg.H * esize
            gbs = gu_bytes / t_gu / 1e9
            roofline.update({"bound": "hbm", "achieved": round(gbs, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                             "frac": round(gbs / PEAK_HBM_GBS, 4), "mfma_tflops": round(achieved, 2)})
        # the shader clock a block of the launch saw (the chip is power limited under this kernel; the
        # published peak is for 2400 MHz), and the fraction of the peak at that clock
        st = ws.view("status").cpu().tolist()
        if cfg.dtype == "bf16" and st[2] > 0:
            roofline["clock_mhz"] = {"gate_up": st[2], "down": st[3]}
            if roofline["bound"] == "mfma":
                roofline["frac_at_that_clock"] = round(achieved / (PEAK_BF16_TFLOPS * st[2] / PEAK_CLOCK_MHZ), 4)
    extra = {}
    if stages:
        t_ffn = (stages["gemm_gate_up"] + stages["gemm_down"]) * 1e-3
        R, H, F, T, E, b = cfg.R, cfg.H, cfg.F, cfg.T, cfg.E, (2 if cfg.dtype == "bf16" else 4)
        alg_bytes = {   # algorithmic HBM bytes of the copy-like stages
            "route": T * H * b + E * H * b + 8 * R,
            # index arrays only when the gate/up GEMM gathers the rows of x itself (the default)
            "permute": 12 * R + (0 if M.get_option("fuse_gather") else T * H * b + R * H * b),
            "combine": 4 * R * H + 4 * R + 4 * T * H,
        }
        extra = {
            "stage_ms": {k: round(v, 4) for k, v in stages.items()},
            "stage_hbm_gbs": {k: round(v / (stages[k] * 1e-3) / 1e9, 1) for k, v in alg_bytes.items()},
            "expert_gemms_tflops": round(flops_ffn / t_ffn / 1e12, 2),
            "expert_gemms_frac_of_bf16_peak": round(flops_ffn / t_ffn / 1e12 / PEAK_BF16_TFLOPS, 4),
            "layer_tflops": round((flops_ffn + cfg.router_flops) / (ms_per_step * 1e-3) / 1e12, 2),
        }

    cpu_baseline = None
    sample_failed = None
    if not args.no_cpu_baseline:
        import oracle
        n = min(args.cpu_sample_tokens, cfg.T)
        stride = max(1, cfg.T // n)                        # tokens at a stride over the micro-batch: their rows fall into
        picked = np.arange(0, cfg.T, stride)[:n]           # every row tile of every expert, not only the first ones
        v = {k: oracle_view(t) for k, t in inp.items() if k != "bias"}
        b = None if inp["bias"] is None else inp["bias"].numpy().astype(np.float64)
        xs = np.ascontiguousarray(v["x"][picked])
        t0 = time.perf_counter()
        ref = oracle.layer(xs, v["Wr"], v["W1"], v["W3"], v["W2"], cfg.k, cfg.dtype_code, bias=b)
        dt = time.perf_counter() - t0
        cpu_baseline = {"value": round(len(picked) / dt, 3), "unit": "tokens/s", "cores": oracle.num_threads(), "kind": "oracle",
                        "cpu_model": cpu_model(),
                        "sample": f"{len(picked)} tokens of the workload at a stride of {stride}, whole layer (route, permute, FFN, "
                                  f"combine), {dt:.1f}s"}
        # the sample doubles as a check of the timed output: a step whose result is wrong is not a measurement
        got = y.cpu().numpy()[picked]
        same = (np.sort(ws.view("topk_ids").cpu().numpy()[picked], axis=1) == np.sort(ref["ids"], axis=1)).all(axis=1)
        err = float(np.abs(got[same] - ref["y"][same]).max())
        extra["max_abs_err_vs_oracle_on_sample"] = round(err, 6)
        extra["sample_tokens_compared"] = int(same.sum())
        tol = 2e-2 if cfg.dtype == "bf16" else 1e-5
        if not (err <= tol) or same.sum() < 0.99 * len(picked):
            sample_failed = f"timed output differs from the oracle on the sample: max |err| {err} (bound {tol}), {int(same.sum())} of {len(picked)} tokens with the oracle's experts"

    out = {
        "metric": "MoE layer tokens/s + % bf16 MFMA peak (Mixtral-8x7B shape, 4096 tokens)",
        "value": round(tokens_per_s, 1), "unit": "tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": cfg.dtype, "data": "synthetic",
        "config": {"workload": cfg.name, "T": cfg.T, "H": cfg.H, "F": cfg.F, "E": cfg.E, "k": cfg.k,
                   "page_bytes": cfg.page_bytes, "weights": "pinned host, streamed" if cfg.streamed else "resident in HBM"},
        "roofline": roofline, "cpu_baseline": cpu_baseline, "single_step_ms": spread,
    }
    if streamer is not None:
        link_bytes = pw.pages_host.numel() * pw.pages_host.element_size()
        extra["host_link"] = {"bytes_per_step": link_bytes, "gbs": round(link_bytes / (ms_per_step * 1e-3) / 1e9, 2),
                              "host_pages": "random order, one copy per page" if args.shuffle_host_pages else "in order, one copy per expert",
                              "note": "every weight page crosses the host link once per step; the step is bound by it"}
    out.update(extra)
    if args.sample_power:
        out["power"] = sample_power(step, torch)
    print(json.dumps(out), flush=True)
    if streamer is not None:
        streamer.close()
    if sample_failed:
        print("bench.py: " + sample_failed, file=sys.stderr)
        sys.exit(3)


def sample_power(step, torch, seconds=4.0):
    """Runs `step` back to back for a few seconds while `amd-smi metric --power --clock --json` is polled from a thread:
    the board's socket power and the clock of every XCD under the workload."""
    import subprocess
    import threading
    watts, clocks, stop = [], [], threading.Event()

    def poll():
        while not stop.is_set():
            try:
                r = subprocess.run(["amd-smi", "metric", "--power", "--clock", "--json"], capture_output=True, text=True, timeout=10)
                g = json.loads(r.stdout)["gpu_data"][0]
                watts.append(float(g["power"]["socket_power"]["value"]))
                clocks.append([float(v["clk"]["value"]) for k, v in sorted(g["clock"].items()) if k.startswith("gfx_")])
            except Exception:
                pass
            time.sleep(0.05)

    for _ in range(20):                                   # reach the steady state first
        step()
    torch.cuda.synchronize()
    th = threading.Thread(target=poll)
    th.start()
    t0 = time.perf_counter()
    while time.perf_counter() - t0 < seconds:
        for _ in range(20):
            step()
        torch.cuda.synchronize()
    stop.set()
    th.join()
    if not watts:
        return {"error": "amd-smi gave no reading"}
    watts.sort()
    med = lambda v: sorted(v)[len(v) // 2]
    return {"source": "amd-smi metric --power --clock --json, polled while the step runs back to back", "samples": len(watts),
            "socket_power_w": {"min": watts[0], "median": med(watts), "max": watts[-1]},
            "gfx_clk_mhz_median_per_xcd": [med([c[i] for c in clocks if len(c) > i]) for i in range(max(len(c) for c in clocks))]}


def vendor_gemm_bench(args, M):
    """The vendor GEMM library (torch.matmul on bf16 tensors) and this library's paged linear map (the down-projection
    kernel with one row segment, f32 output) on the same box, the same random data and the same warm state."""
    import torch
    torch.manual_seed(0)

    def timed(fn, warm=60, reps=60):
        for _ in range(warm):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    rows = []
    # the down projection and the gate/up product of the 4096-token Mixtral-8x7B workload as dense products, and the probe shape
    for T, N, K in ((8192, 4096, 14336), (8192, 28672, 4096), (2048, 32768, 8192)):
        a = torch.randn((T, K), device="cuda").to(torch.bfloat16)
        w = (torch.randn((N, K)) * 0.02).to(torch.bfloat16)
        wd = w.cuda()
        ms_v = timed(lambda: a @ wd.T)
        ls = M.make_linear_shape(T, K, N, 4 << 20)
        n = M.linear_pages_required(ls)
        table = torch.arange(n, dtype=torch.int32)
        pages = torch.empty((n, 4 << 20), dtype=torch.uint8)
        M.linear_pack(ls, w, table, pages)
        pd, td = pages.cuda(), table.cuda()
        ms_l = timed(lambda: M.moe_linear(ls, a, td, pd))
        flop = 2.0 * T * N * K
        rows.append({"T": T, "N": N, "K": K, "vendor_ms": round(ms_v, 4), "vendor_tflops": round(flop / ms_v / 1e9, 1),
                     "library_ms": round(ms_l, 4), "library_tflops": round(flop / ms_l / 1e9, 1)})
        del a, wd, pd, td
    print(json.dumps({"metric": "dense bf16 product: vendor GEMM library (bf16 out) against this library's paged linear map (f32 out, "
                                "allocated per call by the binding)", "unit": "TFLOP/s", "dtype": "bf16", "data": "synthetic", "shapes": rows}), flush=True)


def splits_bench(args, cfg, M, make_inputs):
    """moe_expert_ffn (both expert GEMMs) on the workload's layer shape for several splits of its rows over the experts."""
    import torch
    assert cfg.E == 8 and cfg.R == 8192, "the splits are written for 8 experts and 8192 rows"
    s = M.make_shape(cfg.T, cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes)
    inp = make_inputs(cfg, threads=16)
    pw = M.PagedWeights(s, inp["W1"], inp["W3"], inp["W2"])
    pw.to_device(keep_host=False)
    g = torch.Generator().manual_seed(5)
    xp = torch.randn((cfg.R, cfg.H), generator=g).to(torch.bfloat16).cuda()
    rw = torch.rand((cfg.R,), generator=g).cuda()
    status = torch.zeros(4, dtype=torch.int32, device="cuda")
    splits = {
        "equal: 8 x 1024": [1024] * 8,
        "ragged, as the 4096-token workload routes": [1027, 1061, 1029, 995, 1046, 1010, 1014, 1010],
        "all with 16 rows over a tile multiple": [1040] * 7 + [912],
        "multiples of 256, uneven": [768, 1280, 1024, 1024, 512, 1536, 1024, 1024],
    }
    rows = []
    for name, cnt in splits.items():
        assert sum(cnt) == cfg.R
        off = torch.tensor([0] + list(torch.tensor(cnt).cumsum(0)), dtype=torch.int32).cuda()
        for _ in range(max(args.warmup, 10)):
            M.moe_expert_ffn(s, xp, off, pw.table_dev, pw.pages_dev, row_w=rw, status=status)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(args.steps):
            M.moe_expert_ffn(s, xp, off, pw.table_dev, pw.pages_dev, row_w=rw, status=status)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / args.steps
        rows.append({"split": name, "rows": cnt, "ms": round(ms, 4), "tflops": round(6.0 * cfg.R * cfg.H * cfg.F / ms / 1e9, 1)})
    print(json.dumps({"metric": "both expert GEMMs (moe_expert_ffn, outputs allocated per call by the binding) against the split of "
                                "the rows over the experts", "unit": "ms", "steps": args.steps, "dtype": "bf16", "data": "synthetic",
                      "config": {"workload": cfg.name + " (layer shape)"}, "splits": rows}), flush=True)


def rate_probes(args, M):
    """The inputs of the roofline model (paper_2411_11217_amd.hrm.MI355X_PROBED), measured apart from the layer."""
    import torch

    def timed(fn, reps):
        fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e-3 / reps

    out = {"metric": "rates for the roofline model, measured by probes", "n_gpus": 1, "data": "synthetic"}
    # host link: pinned host memory -> device, one copy of 1 GiB
    n = 1 << 30
    host = torch.empty(n, dtype=torch.uint8).pin_memory()
    dev = torch.empty(n, dtype=torch.uint8, device="cuda")
    t = timed(lambda: dev.copy_(host, non_blocking=True), 5)
    out["host_link_gbs"] = round(n / t / 1e9, 2)
    del host, dev
    # device memory: a kernel of nothing but loads over 4 GiB (larger than every cache), 8 blocks per compute unit
    buf = torch.empty(4 << 30, dtype=torch.uint8, device="cuda").fill_(1)
    rates = {}
    for blocks in (1024, 2048, 4096):
        t = timed(lambda: M.probe_stream_read(buf, blocks=blocks), 10)
        rates[blocks] = round(buf.numel() / t / 1e12, 3)
    out["hbm_read_tbs"] = max(rates.values())
    out["hbm_read_tbs_by_blocks"] = rates
    # the same with the non-temporal hint, as the weight loads of launches with few rows per expert carry it
    rates = {}
    for blocks in (1024, 2048, 4096):
        t = timed(lambda: M.probe_stream_read(buf, blocks=blocks, non_temporal=True), 10)
        rates[blocks] = round(buf.numel() / t / 1e12, 3)
    out["hbm_read_nt_tbs"] = max(rates.values())
    out["hbm_read_nt_tbs_by_blocks"] = rates
    del buf
    # matrix rate: a dense bf16 product of 2048 x 8192 x 32768 through the paged linear map (the down-projection kernel on
    # full, equal tiles: eight row tiles, 128 column tiles, a reduction twice as long as the layer's gate/up product)
    T, K, N = 2048, 8192, 32768
    page_bytes = 2 << 20
    ls = M.make_linear_shape(T, K, N, page_bytes)
    pages = M.linear_pages_required(ls)
    g = torch.Generator().manual_seed(3)
    W = (torch.randn((N, K), generator=g) * 0.02).to(torch.bfloat16)
    pool = torch.empty((pages, page_bytes), dtype=torch.uint8)
    table = torch.arange(pages, dtype=torch.int32)
    M.linear_pack(ls, W, table, pool)
    pool, table = pool.cuda(), table.cuda()
    x = torch.randn((T, K), generator=g).to(torch.bfloat16).cuda()
    for _ in range(5):
        M.moe_linear(ls, x, table, pool)
    t = timed(lambda: M.moe_linear(ls, x, table, pool), 20)
    out["dense_gemm_tflops"] = round(2.0 * T * K * N / t / 1e12, 1)
    out["dense_gemm_shape"] = [T, K, N]
    print(json.dumps(out), flush=True)


def tasks_bench(args, cfg, M, make_inputs):
    """Times the two GPU tasks of the paper's pipeline (its section 4.1) and their stages on one micro-batch."""
    import torch
    s = M.make_shape(cfg.T, cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes)
    inp = make_inputs(cfg, threads=16)
    pw = M.PagedWeights(s, inp["W1"], inp["W3"], inp["W2"])
    T, H, Nq = cfg.T, cfg.H, cfg.H * 3 // 2
    o_shape, q_shape = M.make_linear_shape(T, H, H, cfg.page_bytes), M.make_linear_shape(T, H, Nq, cfg.page_bytes)
    n_exp, n_o, n_q = pw.pool_pages, M.linear_pages_required(o_shape), M.linear_pages_required(q_shape)
    g = torch.Generator().manual_seed(1)
    pool = torch.empty((n_exp + n_o + n_q, cfg.page_bytes), dtype=torch.uint8)
    pool[:n_exp] = pw.pages_host
    o_table = torch.arange(n_exp, n_exp + n_o, dtype=torch.int32)
    q_table = torch.arange(n_exp + n_o, n_exp + n_o + n_q, dtype=torch.int32)
    M.linear_pack(o_shape, (torch.randn((H, H), generator=g) * 0.02).to(torch.bfloat16), o_table, pool)
    M.linear_pack(q_shape, (torch.randn((Nq, H), generator=g) * 0.02).to(torch.bfloat16), q_table, pool)
    pool, o_table, q_table, table = pool.cuda(), o_table.cuda(), q_table.cuda(), pw.table_host.cuda()
    attn = torch.randn((T, H), generator=g).to(torch.bfloat16).cuda()
    hidden = torch.randn((T, H), generator=g).cuda()
    gamma = torch.ones(H).cuda()
    Wr = inp["Wr"].cuda()

    def timed(fn):
        for _ in range(args.warmup):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(args.steps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / args.steps

    hm, x_moe, y, _ws = M.moe_post_attention(s, o_shape, attn, hidden, o_table, gamma, 1e-5, Wr, table, pool)
    o = M.moe_linear(o_shape, attn, o_table, pool)
    ms = {
        "post_attention_task": timed(lambda: M.moe_post_attention(s, o_shape, attn, hidden, o_table, gamma, 1e-5, Wr, table, pool)),
        "pre_attention_task": timed(lambda: M.moe_pre_attention(q_shape, hm, y, gamma, 1e-5, q_table, pool)),
        "o_projection": timed(lambda: M.moe_linear(o_shape, attn, o_table, pool)),
        "qkv_projection": timed(lambda: M.moe_linear(q_shape, x_moe, q_table, pool)),
        "add_rmsnorm": timed(lambda: M.moe_add_rmsnorm(hidden, o, gamma, 1e-5)),
        "cast_bf16_qkv": timed(lambda: M.moe_cast_bf16(torch.empty((T, Nq), dtype=torch.float32, device="cuda"))),
    }
    out = {"metric": "GPU tasks around the MoE layer, ms per micro-batch (includes the binding's output allocations)",
           "config": {"workload": cfg.name + " (layer shape)", "T": T, "H": H, "qkv_width": Nq},
           "ms": {k: round(v, 4) for k, v in ms.items()},
           "tflops": {"o_projection": round(2.0 * T * H * H / ms["o_projection"] / 1e9, 1),
                      "qkv_projection": round(2.0 * T * H * Nq / ms["qkv_projection"] / 1e9, 1)},
           "add_rmsnorm_gbs": round((2 * T * H * 4 + T * H * 4 + T * H * 2) / ms["add_rmsnorm"] / 1e6, 1)}
    print(json.dumps(out), flush=True)


def mu_sweep_bench(args, cfg, M, make_inputs):
    """Layer latency against the micro-batch size mu on one layer shape; the model's prediction beside it."""
    import torch
    from paper_2411_11217_amd import hrm
    inp = make_inputs(cfg, threads=16)
    mus = [int(v) for v in args.mu_list.split(",")] if args.mu_list else [32, 64, 128, 256, 512, 1024, 2048, 4096]
    s_max = M.make_shape(max(mus), cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes)
    pw = M.PagedWeights(s_max, inp["W1"], inp["W3"], inp["W2"])
    pw.to_device(keep_host=False)
    Wr = inp["Wr"].cuda()
    g = torch.Generator().manual_seed(cfg.seed)
    x_all = torch.randn((max(mus), cfg.H), generator=g).to(cfg.torch_dtype).cuda()
    layer = hrm.Layer(cfg.H, cfg.F, cfg.E, cfg.k, 2 if cfg.dtype == "bf16" else 4)
    weight_bytes = 3.0 * cfg.E * cfg.H * cfg.F * (2 if cfg.dtype == "bf16" else 4)
    rows = []
    for mu in mus:
        sh = M.make_shape(mu, cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes)
        x, ws = x_all[:mu].contiguous(), M.Workspace(sh)
        y = torch.empty((mu, cfg.H), dtype=torch.float32, device="cuda")
        for _ in range(args.warmup):
            M.moe_layer(sh, x, Wr, pw.table_dev, pw.pages_dev, workspace=ws, y=y)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            M.moe_layer(sh, x, Wr, pw.table_dev, pw.pages_dev, workspace=ws, y=y)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / args.steps
        model = hrm.layer_latency(layer, hrm.MI355X_PROBED, mu, mu, 1.0, hidden_from_host=False)
        rows.append({"mu": mu, "ms": round(ms, 4), "tokens_per_s": round(mu / (ms * 1e-3), 1),
                     "weight_tb_per_s": round(weight_bytes / (ms * 1e-3) / 1e12, 2),
                     "tflops": round(6.0 * mu * cfg.k * cfg.H * cfg.F / (ms * 1e-3) / 1e12, 1),
                     "model_ms": round(model["T"] * 1e3, 4)})
        if args.two_streams:
            # two micro-batches of the layer at a time, each on a stream and a workspace of its own: the blocks of one fill
            # the partly filled rounds of the other
            streams = [torch.cuda.Stream(), torch.cuda.Stream()]
            ws2, y2 = [ws, M.Workspace(sh)], [y, torch.empty_like(y)]
            torch.cuda.synchronize()

            def pair(n):
                for i in range(n):
                    M.moe_layer(sh, x, Wr, pw.table_dev, pw.pages_dev, workspace=ws2[i & 1], y=y2[i & 1], stream=streams[i & 1])
            pair(2 * args.warmup)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            pair(2 * args.steps)
            torch.cuda.synchronize()
            rows[-1]["ms_per_micro_batch_on_two_streams"] = round((time.perf_counter() - t0) * 1e3 / (2 * args.steps), 4)
    print(json.dumps({"metric": "MoE layer latency against the micro-batch size (weights resident)", "unit": "ms",
                      "steps": args.steps, "warmup": args.warmup, "dtype": cfg.dtype, "data": "synthetic",
                      "config": {"workload": cfg.name + " (layer shape), micro-batch sweep"}, "sweep": rows}), flush=True)


def prefill_bench(args, cfg, M, make_inputs):
    """A prefill pass: variable-length requests -> balanced micro-batches (the paper's appendix A.2) -> the layer once
    per micro-batch on its prompt tokens (in prefill the whole layer runs on the GPU, the paper's section 3.2)."""
    import torch
    from moe_workloads import prompt_lengths
    from paper_2411_11217_amd.batching import Request, batch_requests
    lens = prompt_lengths(args.requests, seed=cfg.seed)
    n_ub = (args.requests + args.ubs - 1) // args.ubs
    mbs, aborted = batch_requests([Request(i, int(v)) for i, v in enumerate(lens)], n_ub, args.ubs, gen_len=128,
                                  cache_size=1 << 40)
    assert not aborted
    tokens = [mb.prompt_tokens for mb in mbs]
    inp = make_inputs(cfg, threads=16)
    s_max = M.make_shape(max(tokens), cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes)
    pw = M.PagedWeights(s_max, inp["W1"], inp["W3"], inp["W2"])
    pw.to_device(keep_host=False)
    Wr = inp["Wr"].cuda()
    g = torch.Generator().manual_seed(cfg.seed)
    shapes = [M.make_shape(t, cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes) for t in tokens]
    xs = [torch.randn((t, cfg.H), generator=g).to(cfg.torch_dtype).cuda() for t in tokens]
    ys = [torch.empty((t, cfg.H), dtype=torch.float32, device="cuda") for t in tokens]
    wss = [M.Workspace(sh) for sh in shapes]

    def step():
        for sh, x, y, ws in zip(shapes, xs, ys, wss):
            M.moe_layer(sh, x, Wr, pw.table_dev, pw.pages_dev, workspace=ws, y=y)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    total = sum(tokens)
    flops = 6.0 * total * cfg.k * cfg.H * cfg.F
    print(json.dumps({
        "metric": "prefill pass of a request batch through one MoE layer, prompt tokens/s", "value": round(total / (ms * 1e-3), 1),
        "unit": "tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 4),
        "dtype": cfg.dtype, "data": "synthetic",
        "config": {"workload": cfg.name + " (layer shape), prefill", "requests": args.requests, "ubs": args.ubs,
                   "prompt_len_avg": round(float(lens.mean()), 2), "prompt_len_max": int(lens.max()),
                   "micro_batch_tokens": tokens},
        "expert_gemms_tflops_lower_bound": round(flops / (ms * 1e-3) / 1e12, 1)}), flush=True)


def pipeline_bench(args, cfg, M, make_inputs):
    """Times passes of moe_pipeline_run: per layer, n micro-batches are computed while the non-resident pages of
    the next layer cross the host link.  Reported next to the paper's per-layer latency model
    T = max(comm_cpu_to_gpu, T_gpu) (its section 4.2; no CPU work here), with T_gpu measured by the same
    pipeline holding every page resident."""
    import torch
    n, L = args.micro_batches, args.layers
    mu = cfg.T // n
    s = M.make_shape(mu, cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes)
    inp = make_inputs(cfg, threads=16)
    host = M.PagedWeights(s, inp["W1"], inp["W3"], inp["W2"], pin=True)
    del inp["W1"], inp["W3"], inp["W2"]
    ppe = host.ppe
    x_host = [[inp["x"][j * mu:(j + 1) * mu].contiguous().pin_memory() for j in range(n)] for _ in range(L)]
    Wr = [inp["Wr"].cuda()] * L
    bias = None if inp["bias"] is None else [inp["bias"].cuda()] * L
    y = [[torch.empty((mu, cfg.H), dtype=torch.float32, device="cuda")] * n for _ in range(L)]   # results overwrite each other
    layers = [(host.pages_host, host.table_host)] * L

    def timed(n_res):
        pipe = M.Pipeline(s, layers, n_res, max_micro_batches=n)
        ws = None
        for _ in range(max(args.warmup // 5, 1)):
            ws = pipe.run(x_host, Wr, y, bias=bias, workspace=ws)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        reps = max(args.steps // 10, 2)
        for _ in range(reps):
            pipe.run(x_host, Wr, y, bias=bias, workspace=ws)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / (reps * L)
        pipe.close()
        del pipe
        torch.cuda.empty_cache()
        return ms

    n_res = int(round(args.resident_fraction * ppe))
    gpu_ms = timed(ppe)
    ms = timed(n_res)
    link_bytes = cfg.E * (ppe - n_res) * cfg.page_bytes
    out = {
        "metric": "MoE layer pipeline tokens/s per layer (weights paged from pinned host memory)",
        "value": round(cfg.T / (ms * 1e-3), 1), "unit": "tokens/s", "n_gpus": 1, "higher_is_better": True,
        "ms_per_layer": round(ms, 3), "dtype": cfg.dtype, "data": "synthetic",
        "config": {"workload": cfg.name + " (layer shape)", "layers": L, "micro_batches": n, "micro_tokens": mu,
                   "resident_pages_per_expert": n_res, "pages_per_expert": ppe, "resident_fraction": round(n_res / ppe, 4)},
        "host_link": {"bytes_per_layer": link_bytes, "gbs": round(link_bytes / (ms * 1e-3) / 1e9, 2)},
        "model": {"gpu_ms_per_layer_all_resident": round(gpu_ms, 3),
                  "note": "per-layer latency = max(link bytes / link rate, gpu_ms); link rate ~55.7 GB/s measured on the "
                          "fully streamed workload"},
    }
    out["model"]["predicted_ms"] = round(max(link_bytes / 55.7e9 * 1e3, gpu_ms), 3)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
