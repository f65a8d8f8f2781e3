"""Throughput of one skip-collocated Pulse stage (forward + backward) on one
MI355X, through the C ABI.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload l64]

A step is one pass of the whole hot path over one microbatch of synthetic
input already resident in HBM: encoder forward (skips cached in HBM),
decoder forward (reading [upstream || skip] from the cache), decoder
backward (skip gradient buffered), encoder backward (skip gradient added).
The ``wave`` workload's step is one wave iteration of the four SD levels
with 4 microbatches in flight (all forwards, then backwards in reverse).
``wave-sched`` runs the same four levels as the four devices of a 4-device
pipeline: each level's stage executes its device's row of the collocated
wave schedule for 4 microbatches (pulse_sched_run_device), one row after
another on this GPU.

Prints ONE JSON line (rank 0): stage fwd+bwd TFLOP/s with the fraction of
the bf16 MFMA peak, microbatches/s, the roofline of the implicit-GEMM conv
kernel (its launches bracketed by HIP events on the stage stream during the
timed steps) and the CPU oracle timed on a bounded sample of the same
workload.
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

PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA
# Overlapped decoder backward, measured per workload (same box, alternating
# runs): 64x64x320 778 against 764 TFLOP/s; 32x32x640 725-728 against
# 709-711 (since the timestep weight gradient takes less of the second
# stream); 16x16x1280 840-841 against 844-847 and 8x8x1280 469 against
# 471-474; the four-level wave 625 either way; the transformer stages 372
# against 371 (768 wide) and 665 against 657 (1408 wide).
OVERLAP_BWD_AUTO = ("l64", "l32", "t768", "t1408")
PEAK_FP32_TFLOPS = 157.3    # MI355X fp32 vector (the fp32 stage)
METRIC = "stage fwd+bwd TFLOP/s (% bf16 MFMA peak) and microbatches/s, 64x64x320 stage"


def workload_desc(name):
    from paper_2606_19163_amd import configs
    if name in ("wave", "wave-sched"):
        return configs.wave_levels()
    return [configs.get(name)]


def describe(name, descs):
    d = descs[0]
    if name == "wave":
        return {"workload": "wave: 4 collocated stages (64x64x320, 32x32x640, 16x16x1280, "
                            "8x8x1280) at batch 8, 4 microbatches in flight, all forwards "
                            "then backwards in reverse",
                "batch": 8, "microbatches": 4, "levels": 4}
    if name == "wave-sched":
        return {"workload": "wave-sched: 4 collocated stages (64x64x320, 32x32x640, "
                            "16x16x1280, 8x8x1280) at batch 8 as devices 0-3 of a 4-device "
                            "pipeline, each running its row of the wave schedule for 4 "
                            "microbatches",
                "batch": 8, "microbatches": 4, "levels": 4, "devices": 4}
    chans = sorted({b["c_out"] for b in d["enc"]} | {b["c_in"] for b in d["enc"]})
    return {"workload": f"{name}: one collocated stage, batch {d['batch']}, "
                        f"{d['height']}x{d['width']}, channels {chans}, "
                        f"{len(d['enc'])} encoder + {len(d['dec'])} decoder ResBlocks, "
                        f"GroupNorm {d['groups']} groups, t-emb {d['temb_dim']}",
            "batch": d["batch"], "height": d["height"], "width": d["width"],
            "enc_blocks": [[b["c_in"], b["c_out"]] for b in d["enc"]],
            "dec_blocks": [[b["c_up"], b["c_skip"], b["c_out"]] for b in d["dec"]]}


# committed FETCH_SIZE/WRITE_SIZE summaries of the conv-mode GEMM launches,
# each valid for the kernel and planning sources it was taken on
TRAFFIC_WORKLOADS = {
    "l64": ["igemm2.hip", "kernels.hpp", "common.hpp", "kpos.hpp", "plan.hpp", "stage.cpp"],
    "l32": ["igemm2.hip", "kernels.hpp", "common.hpp", "kpos.hpp", "plan.hpp", "stage.cpp"],
    "t768": ["igemm2.hip", "kernels.hpp", "common.hpp", "kpos.hpp", "plan.hpp", "tstage.cpp"],
    "t1408": ["igemm2.hip", "kernels.hpp", "common.hpp", "kpos.hpp", "plan.hpp", "tstage.cpp"],
}


def traffic_profile(name):
    return os.path.join(ROOT, "profiles", f"igemm2_conv_{name}_traffic.md")


def kernel_sources_sha256(name="l64"):
    import hashlib
    h = hashlib.sha256()
    for f in TRAFFIC_WORKLOADS[name]:
        with open(os.path.join(ROOT, "paper_2606_19163_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def measured_traffic(name):
    """HBM bytes per conv-mode launch from the committed FETCH_SIZE/WRITE_SIZE
    summary of the workload; None when that summary was taken on other
    kernel sources than the ones built here, or when there is none."""
    path = traffic_profile(name) if name in TRAFFIC_WORKLOADS else None
    if path is None or not os.path.exists(path):
        return None
    vals = {}
    with open(path) as fh:
        for line in fh:
            if line.startswith("- ") and ": " in line:
                k, v = line[2:].strip().split(": ", 1)
                vals[k.strip("`")] = v.strip().strip("`")
    if vals.get("kernel_sources_sha256") != kernel_sources_sha256(name):
        return None
    try:
        return int(vals["traffic_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def mfma_probe_tflops():
    """Sustained bf16 MFMA rate of the GPU: register-operand MFMA chains with
    no memory traffic (2048 workgroups of 4 waves, 400 iterations), timed with
    HIP events; the median of 5 launches per shape."""
    import torch
    from paper_2606_19163_amd import stage as S
    out = torch.empty(2048 * 256, dtype=torch.float32, device="cuda")
    res = {}
    for shape, name in ((32, "32x32x16"), (16, "16x16x32")):
        S.mfma_probe(shape, 2048, 50, out)  # warm up
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fl = S.mfma_probe(shape, 2048, 400, out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        times.sort()
        res[name] = round(fl / (times[2] * 1e-3) / 1e12, 1)
    return res


def library_gemm_tflops():
    """The vendor GEMM (torch.matmul, bf16) on plain GEMMs of the stage's
    shapes and on large squares, median of 5 timed runs of 20 calls each:
    the conv forward of the 64x64x320 stage (M = 32768 pixels, N = 320,
    K = 2880 or 5760), its weight gradient (M = 320, N = 2880, K = 32768,
    A transposed), and 8192^3 / 16384^2 x 8192."""
    import torch
    shapes = [("conv 32768x320x2880", 32768, 320, 2880, False),
              ("conv 32768x320x5760", 32768, 320, 5760, False),
              ("wgrad 320x2880x32768", 320, 2880, 32768, True),
              ("square 8192^3", 8192, 8192, 8192, False),
              ("16384x16384x8192", 16384, 16384, 8192, False)]
    res = {}
    for name, M, N, K, ta in shapes:
        a = (torch.randn(K, M, device="cuda", dtype=torch.bfloat16).t() if ta else
             torch.randn(M, K, device="cuda", dtype=torch.bfloat16))
        b = torch.randn(K, N, device="cuda", dtype=torch.bfloat16)
        for _ in range(3):
            a @ b
        times = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                a @ b
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1) / 20)
        times.sort()
        res[name] = round(2.0 * M * N * K / (times[2] * 1e-3) / 1e12, 1)
        del a, b
    return res


def cpu_baseline(name, descs, seed, sample_batch, min_seconds=10.0):
    """The oracle, as it stands, on `sample_batch` images of the workload's
    first stage (forward + backward), repeated until at least `min_seconds`
    have passed, scaled to TFLOP/s."""
    import numpy as np
    from oracle import pulse_oracle as O
    from paper_2606_19163_amd import configs, synth
    from paper_2606_19163_amd import stage as S
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        threads = os.cpu_count() or 1
    d = configs.shrink(descs[0], batch=sample_batch)
    params, b = synth.make_all(d, seed)
    f = lambda x: {k: np.asarray(v, np.float64) for k, v in x.items()}
    p64, b64 = f(params), f(b)
    flops = S.Stage(d, dry_run=True).flops()
    runs, t0 = 0, time.perf_counter()
    while runs == 0 or time.perf_counter() - t0 < min_seconds:
        O.stage_run(d, p64, b64["x"], b64["u"], b64["temb"], b64["g_enc"], b64["g_dec"])
        runs += 1
    dt = time.perf_counter() - t0
    return {"value": runs * flops / dt / 1e12, "unit": "TFLOP/s", "cores": int(threads),
            "kind": "oracle",
            "sample": f"{runs} x {sample_batch} of {descs[0]['batch']} images of one microbatch of "
                      f"the first stage ({d['height']}x{d['width']}), forward + backward, numpy "
                      f"fp64; {dt:.2f} s", **host_info()}


def host_info():
    """CPU model, logical CPU count and OMP thread setting of the host."""
    model = None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"cpu_model": model, "cpu_count": os.cpu_count(),
            "omp_num_threads": os.environ.get("OMP_NUM_THREADS")}


def timed_steps(step, steps):
    """Run `steps` steps between two device synchronisations; returns the
    wall time and the per-step times from HIP events recorded on the
    current stream between steps (the stages join their side stream into it
    at the end of every backward)."""
    import torch
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ev[0].record()
    for i in range(steps):
        step()
        ev[i + 1].record()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    per = sorted(ev[i].elapsed_time(ev[i + 1]) for i in range(steps))
    return elapsed, per


def step_stats(per):
    n = len(per)
    med = per[n // 2] if n % 2 else 0.5 * (per[n // 2 - 1] + per[n // 2])
    return {"step_ms_median": round(med, 4), "step_ms_min": round(per[0], 4)}


def tstage_cpu_baseline(desc, seed, sample_batch, min_seconds=10.0):
    """The transformer-stage oracle, as it stands, on `sample_batch` images of
    the workload (forward + backward), repeated until `min_seconds` have
    passed, scaled to TFLOP/s."""
    from oracle import transformer_oracle as TO
    from paper_2606_19163_amd import synth
    from paper_2606_19163_amd import tstage as TS
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        threads = os.cpu_count() or 1
    d = dict(desc, batch=sample_batch)
    params, b = synth.make_tstage(d, seed)
    flops = TS.TStage(d, dry_run=True).flops()
    runs, t0 = 0, time.perf_counter()
    while runs == 0 or time.perf_counter() - t0 < min_seconds:
        TO.tstage_run(d, params, b["x"], b["u"], b["g_enc"], b["g_dec"])
        runs += 1
    dt = time.perf_counter() - t0
    return {"value": runs * flops / dt / 1e12, "unit": "TFLOP/s", "cores": int(threads),
            "kind": "oracle",
            "sample": f"{runs} x {sample_batch} of {desc['batch']} images of one microbatch, "
                      f"forward + backward, numpy fp64; {dt:.2f} s", **host_info()}


def bench_tstage(args):
    """One transformer-block stage (t768: UViT-like, 256 tokens of 768
    channels, 12 heads, 2 + 2 blocks, batch 16; t1408: Hunyuan-DiT-like, 1024
    tokens of 1408 channels, 22 heads, 1 + 1 blocks, batch 8): the same step
    and JSON line as the ResBlock stages, with the roofline of the
    token-major GEMM launches."""
    import torch
    from paper_2606_19163_amd import configs, synth
    from paper_2606_19163_amd import tstage as TS

    torch.cuda.set_device(0)
    d = configs.get(args.workload)
    seed = configs.SEEDS[args.workload]
    params, b = synth.make_tstage(d, seed)
    st = TS.TStage(d)
    st.set_params(params)
    overlap_on = args.overlap_bwd == "on" or (args.overlap_bwd == "auto" and
                                              args.workload in OVERLAP_BWD_AUTO)
    st.overlap_bwd(overlap_on)
    dev = {k: st.to_dev(v) for k, v in b.items()}
    outs = {k: st.act() for k in ("y_enc", "y_dec", "dx", "du")}
    if args.copy_calibration_mib > 0:
        # one plain device copy of known size: the scale for HBM counters
        src = torch.ones(args.copy_calibration_mib << 20, dtype=torch.uint8, device="cuda")
        torch.empty_like(src).copy_(src)
        torch.cuda.synchronize()
        del src

    def step():
        st.forward(TS.ENC, 0, dev["x"], out=outs["y_enc"])
        st.forward(TS.DEC, 0, dev["u"], out=outs["y_dec"])
        st.backward(TS.DEC, 0, dev["g_dec"], din=outs["du"])
        st.backward(TS.ENC, 0, dev["g_enc"], din=outs["dx"])

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    elapsed, per = timed_steps(step, args.steps)
    launches, kms, kflops, kbytes = 0, 0.0, 0.0, 0.0
    if not args.no_kernel_events:
        st.timing(True)
        for _ in range(args.steps):
            step()
        torch.cuda.synchronize()
        launches, kms, kflops, kbytes = st.timing_read()
        st.timing(False)
    flops_step = st.flops()
    tflops = flops_step * args.steps / elapsed / 1e12
    line = {
        "metric": "transformer stage fwd+bwd TFLOP/s (% bf16 MFMA peak) and microbatches/s",
        "value": round(tflops, 3), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(elapsed * 1e3 / args.steps, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
        "data": "synthetic (seeded N(0,1) tokens, N(0,1/fan_in) weights)",
        "config": {"workload": f"{args.workload}: one collocated transformer stage, batch "
                               f"{d['batch']}, {d['tokens']} tokens of {d['width']} channels, "
                               f"{d['heads']} heads of 64, MLP x{d['mlp']}, {d['n_enc']} "
                               f"encoder + {d['n_dec']} decoder blocks",
                   "batch": d["batch"], "tokens": d["tokens"], "width": d["width"],
                   "heads": d["heads"], "blocks": [d["n_enc"], d["n_dec"]]},
        "pct_bf16_peak": round(100.0 * tflops / PEAK_BF16_TFLOPS, 2),
        "microbatches_per_s": round(args.steps / elapsed, 2),
        "gflop_per_step": round(flops_step / 1e9, 2),
        **step_stats(per),
        "overlap_bwd": overlap_on,
    }
    if launches:
        achieved = kflops / (kms * 1e-3) / 1e12
        line["roofline"] = {
            "kernel": "igemm_conv in its token-major 1x1 form (linear forward / data gradient)",
            "bound": "mfma", "achieved": round(achieved, 2), "peak": PEAK_BF16_TFLOPS,
            "unit": "TFLOP/s", "frac": round(achieved / PEAK_BF16_TFLOPS, 4),
            "traffic": measured_traffic(args.workload),
            "algorithmic_bytes_per_launch": round(kbytes / launches), "launches": launches,
            "avg_launch_us": round(kms * 1e3 / launches, 2),
            "avg_gflop_per_launch": round(kflops / launches / 1e9, 3)}
    if not args.no_cpu_baseline:
        sample = 1 if d["tokens"] >= 1024 else min(args.cpu_sample_batch, 2)
        line["cpu_baseline"] = tstage_cpu_baseline(d, seed, sample)
    print(json.dumps(line), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="l64",
                    choices=["l64", "l32", "l16", "l8", "tiny", "wave", "wave-sched",
                             "t768", "t1408", "t_tiny"])
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-sample-batch", type=int, default=8)
    ap.add_argument("--serial", action="store_true",
                    help="keep the whole backward on the stage stream (no side stream)")
    ap.add_argument("--overlap-bwd", choices=("auto", "on", "off"), default="auto",
                    help="start a microbatch's encoder backward beside the parameter-gradient "
                         "tail of its decoder backward (auto: on for the workloads where "
                         "that measured faster)")
    ap.add_argument("--no-kernel-events", action="store_true",
                    help="do not bracket the conv launches with HIP events")
    ap.add_argument("--library-gemm", action="store_true",
                    help="also time the vendor GEMM on plain GEMMs of the stage's shapes")
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="run one plain device-to-device copy of this many MiB before "
                         "the warmup (the known-size kernel that scales HBM counters)")
    args = ap.parse_args()

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU: the stage's multi-GPU sharding (pipeline "
              "neighbours over xGMI, data-parallel all-reduce) is not built here; "
              "run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    if args.workload in ("t768", "t1408", "t_tiny"):
        return bench_tstage(args)
    if args.serial:
        os.environ["PULSE_SERIAL"] = "1"
    import numpy as np
    import torch
    from paper_2606_19163_amd import configs, synth
    from paper_2606_19163_amd import stage as S

    torch.cuda.set_device(0)
    descs = workload_desc(args.workload)
    multi = args.workload in ("wave", "wave-sched")
    n_mb = 4 if multi else 1
    seed = configs.SEEDS["wave" if multi else args.workload]
    sched = None
    if args.workload == "wave-sched":
        sched, sched_exact = S.sched_build(len(descs), n_mb)
        for d, need in zip(descs, S.sched_inflight(len(descs), n_mb, sched)):
            d["max_inflight"] = need
    if multi:
        params, bounds = synth.make_wave(descs, seed, n_mb)
    else:
        p0, b0 = synth.make_all(descs[0], seed)
        params, bounds = [p0], [[b0]]
    stages, dev = [], []
    overlap_on = args.overlap_bwd == "on" or (args.overlap_bwd == "auto" and
                                              args.workload in OVERLAP_BWD_AUTO)
    for i, d in enumerate(descs):
        st = S.Stage(d)
        st.set_params(params[i])
        # a microbatch's encoder backward starts beside the parameter-gradient
        # tail of its decoder backward (bitwise the same results); it pays
        # where the side stream is not the backward's bottleneck
        st.overlap_bwd(overlap_on)
        stages.append(st)
        dev.append([{k: st.to_dev(v) for k, v in bb.items()} for bb in bounds[i]])
    dtembs = [torch.zeros((d["batch"], d["temb_dim"]), device="cuda") for d in descs]
    outs = [[{} for _ in range(n_mb)] for _ in descs]
    for i, d in enumerate(descs):
        for m in range(n_mb):
            outs[i][m]["y_enc"] = stages[i].act(d["enc"][-1]["c_out"])
            outs[i][m]["y_dec"] = stages[i].act(d["dec"][-1]["c_out"])
            outs[i][m]["dx"] = stages[i].act(d["enc"][0]["c_in"])
            outs[i][m]["du"] = stages[i].act(d["dec"][0]["c_up"])
    flops_step = sum(st.flops() for st in stages) * n_mb
    if args.copy_calibration_mib > 0:
        nbytes = args.copy_calibration_mib << 20
        src = torch.ones(nbytes, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    io = [[dict(dev[i][m], **outs[i][m], dtemb=dtembs[i]) for m in range(n_mb)]
          for i in range(len(descs))]

    def step_sched():
        for i, st in enumerate(stages):
            S.sched_run_device(st, len(stages), i, n_mb, sched, io[i])

    def step():
        if sched is not None:
            return step_sched()
        for i, st in enumerate(stages):
            for m in range(n_mb):
                b = dev[i][m]
                o = outs[i][m]
                st.forward(S.ENC, m, b["x"], b["temb"], out=o["y_enc"])
                st.forward(S.DEC, m, b["u"], b["temb"], out=o["y_dec"])
            for m in reversed(range(n_mb)):
                b = dev[i][m]
                o = outs[i][m]
                st.backward(S.DEC, m, b["g_dec"], din=o["du"], dtemb=dtembs[i])
                st.backward(S.ENC, m, b["g_enc"], din=o["dx"], dtemb=dtembs[i])

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    # the timed steps: the stage as it runs in production
    elapsed, per = timed_steps(step, args.steps)
    # the conv kernel's roofline: the same steps again with every conv launch
    # bracketed by HIP events on the stage stream (the backward then keeps
    # its weight-gradient GEMMs on that stream, so each event pair times the
    # kernel alone)
    events = not args.no_kernel_events
    launches, kms, kflops, kbytes = 0, 0.0, 0.0, 0.0
    if events:
        for st in stages:
            st.timing(True)
        torch.cuda.synchronize()
        for _ in range(args.steps):
            step()
        torch.cuda.synchronize()
        for st in stages:
            n, ms, fl, by = st.timing_read()
            launches += n
            kms += ms
            kflops += fl
            kbytes += by
            st.timing(False)

    ms_step = elapsed * 1e3 / args.steps
    tflops = flops_step * args.steps / elapsed / 1e12
    bf16 = descs[0]["dtype"] == configs.BF16
    peak = PEAK_BF16_TFLOPS if bf16 else PEAK_FP32_TFLOPS
    line = {
        "metric": METRIC,
        "value": round(tflops, 3),
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16" if bf16 else "f32",
        "data": "synthetic (seeded N(0,1) activations, N(0,1/fan_in) weights)",
        "config": describe(args.workload, descs),
        "pct_bf16_peak": round(100.0 * tflops / PEAK_BF16_TFLOPS, 2),
        "microbatches_per_s": round(n_mb * args.steps / elapsed, 2),
        "gflop_per_step": round(flops_step / 1e9, 2),
        **step_stats(per),
        "overlap_bwd": overlap_on,
    }
    if events and launches:
        achieved = kflops / (kms * 1e-3) / 1e12
        line["roofline"] = {
            "kernel": "igemm_conv (implicit-GEMM conv forward / data gradient)",
            "bound": "mfma", "achieved": round(achieved, 2), "peak": peak,
            "unit": "TFLOP/s", "frac": round(achieved / peak, 4),
            "traffic": measured_traffic(args.workload),
            "traffic_unit": "HBM bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, "
                            "copy-calibrated)",
            "algorithmic_bytes_per_launch": round(kbytes / launches),
            "launches": launches, "avg_launch_us": round(kms * 1e3 / launches, 2),
            "avg_gflop_per_launch": round(kflops / launches / 1e9, 3),
        }
    if sched is not None:
        T = len(sched[0])
        line["schedule"] = {"devices": len(stages), "microbatches": n_mb, "steps": T,
                            "exact_minimum": bool(sched_exact),
                            "device_busy_frac": round(4 * n_mb / T, 4)}
    # the paper's own end-to-end figures, on its hardware: context, not a target
    line["paper_context"] = {
        "communication_volume_reduction": "89% (2 nodes x 8 V100 32 GB), 90% (8 x 8 Ascend 910A)",
        "training_throughput": "up to 2.3x vs pipeline baselines (Ascend 910A cluster)",
        "per_stage_compute": "not reported"}
    if bf16:
        line["mfma_probe_tflops"] = mfma_probe_tflops()
    if args.library_gemm:
        line["library_gemm_tflops"] = library_gemm_tflops()
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline(args.workload, descs, seed,
                                            min(args.cpu_sample_batch, descs[0]["batch"]))
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
