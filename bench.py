#!/usr/bin/env python3
"""Throughput of the CDP hot path on one MI355X.

A "step" is one training step of Cyclic Data Parallelism: 2S ticks, in which every one of
the N micro-batches of a mini-batch runs the forward and backward of every stage with the
weight versions of the chosen update rule, all N gradients are accumulated per stage and
every stage is updated once (Eq. (CDP), Sec. 3.2).  Inputs are synthetic (N(0,1) features,
uniform labels) and already resident in HBM when the timed region starts.

Prints ONE JSON line.  `--gpus` above 1 is refused: this build runs on one GPU.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import cdp_workloads as wl  # noqa: E402

HBM_PEAK_GBS = 8000.0           # MI355X HBM3E
MFMA_PEAK_TFLOPS = {wl.BF16: 2500.0, wl.F32: 157.3}
WORKLOAD_TEXT = {
    "cfg1": "Tiny MLP: 4 stages Linear(64->64)+ReLU + 10-class head, N=4 micro-batches of 8, fp32",
    "cfg2": "CIFAR-shaped MLP: 3072->1024 stem, 8 stages Linear(1024->1024)+ReLU, 10-class head, N=8 micro-batches of 32, bf16",
    "cfg3": "CIFAR-shaped ResNet-18: 8 BasicBlock stages, N=4 micro-batches of 32, bf16",
    "cfg4": "ImageNet-shaped ResNet-50: 16 bottleneck stages, N=8 micro-batches of 32, bf16",
    "cfg5": "Deep wide MLP: 24 stages Linear(4096->4096)+ReLU, 1000-class head, N=16 micro-batches of 64, bf16",
    "vit_b16": "ViT-B/16-shaped: 12 transformer-block stages on 196 tokens of width 768, N=8 micro-batches of 32, bf16",
}


KERNELS = {"cfg1": "linear_tick_kernel<float>", "cfg2": "linear_tick_kernel_bf16<64>", "cfg5": "linear_tick_kernel_bf16<128>",
           "cfg3": "conv_gemm_kernel, conv_gemm_dl_kernel, conv_gemm_run_kernel + conv_wgrad_mixed_kernel + wgrad_reduce_kernel (+ linear_tick_kernel for the classifier)",
           "cfg4": "conv_gemm_kernel, conv_gemm_dl_kernel, conv_gemm_run_kernel + conv_wgrad_mixed_kernel + wgrad_reduce_kernel (+ linear_tick_kernel for the classifier)",
           "vit_b16": "conv_gemm_kernel, conv_gemm_dl_kernel, conv_gemm_run_kernel, conv_gelu_kernel, conv_gelu_dl_kernel + conv_wgrad_mixed_kernel + wgrad_fold_rows_kernel on the token-wise linear maps (attention and LayerNorm kernels are not in this figure)"}


def measured_traffic(workload):
    """HBM bytes per contraction launch from the committed rocprofv3 --pmc summary of this
    workload (profiles/hbm_traffic_<workload>.txt: FETCH_SIZE and WRITE_SIZE, each scaled by
    what the counter reads for a plain 1 GiB copy), or None when no summary is committed."""
    path = os.path.join(ROOT, "profiles", "hbm_traffic_%s.txt" % workload)
    if not os.path.exists(path):
        return None
    for line in open(path):
        if line.startswith("traffic_bytes_per_launch"):
            return float(line.split("=", 1)[1])
    return None


def gpu_run(cfg, rule, steps, warmup, n_batches=4, dp_batched=False, reps=1, dw_group=1):
    import torch
    from paper_2403_08837_amd import binding as b

    if not torch.cuda.is_available():
        raise SystemExit("bench.py needs a GPU; libcdp has no CPU path")
    tr = b.Trainer(cfg.stages, cfg.in_shape, cfg.N, cfg.B, cfg.lr, rule, cfg.dtype, dp_batched=dp_batched, dw_group=dw_group)
    tr.set_weights(wl.init_params(cfg, 0))
    data = []
    for t in range(n_batches):
        x, y = wl.make_batch(cfg, t, 0)
        data.append((torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()))
    torch.cuda.synchronize()
    # warm-up: fills the cycle (the first d*(N-1) ticks run fewer than N micro-batches)
    for t in range(max(warmup, 1)):
        tr.step(*data[t % n_batches])
    torch.cuda.synchronize()
    # pass 1, the throughput figure: `reps` repetitions of exactly `steps` steps, nothing recorded per
    # launch; the median repetition is reported
    walls, gpu_mss = [], []
    k = 0
    for _ in range(reps):
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ev0.record()
        for t in range(steps):
            tr.step(*data[(warmup + k) % n_batches])
            k += 1
        ev1.record()
        torch.cuda.synchronize()
        walls.append(time.perf_counter() - t0)
        gpu_mss.append(ev0.elapsed_time(ev1))
    order = sorted(range(reps), key=lambda r: walls[r])
    med = order[len(order) // 2]
    wall, gpu_ms = walls[med], gpu_mss[med]
    # pass 2, the roofline figure: the same steps again with a HIP event pair around every
    # contraction launch (the events cost a few microseconds per launch, so this pass is slower)
    tr.profile_gemm(True)
    pv0, pv1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    pv0.record()
    for t in range(steps):
        tr.step(*data[(warmup + k + t) % n_batches])
    pv1.record()
    torch.cuda.synchronize()
    prof = tr.gemm_profile()
    prof["pass_ms"] = pv0.elapsed_time(pv1)
    tr.profile_gemm(False)
    tr.drain()
    torch.cuda.synchronize()
    stats = tr.stats()
    losses = tr.losses(max(warmup, 1) + (reps + 1) * steps - 1)
    # in-tick activation bytes over the ticks in which all N micro-batches are in flight
    d = 0 if rule == wl.RULE_DP else cfg.delay
    n_steps = max(warmup, 1) + (reps + 1) * steps
    steady = slice(d * (cfg.N - 1), 2 * cfg.S * n_steps)
    kept, held = tr.live_bytes(0)[steady], tr.live_bytes(1)[steady]
    act = {"retained_for_backward": {"min": min(kept), "max": max(kept), "distinct_values": len(set(kept))},
           "pool_in_tick": {"min": min(held), "max": max(held), "distinct_values": len(set(held))},
           "steady_state_ticks": len(kept)}
    tr.close()
    return dict(wall=wall, gpu_ms=gpu_ms, walls=walls, prof=prof, stats=stats, act=act, last_losses=[float(v) for v in losses])


def cpu_baseline(cfg, rule, budget_s=15.0, threads=None):
    """The oracle as it stands, timed on this host on a bounded number of steps of the same
    workload (fp64 numpy; it is a reported baseline, never a target).  threads: limit of the
    BLAS thread pool (None: whatever the host gives it)."""
    from oracle import cdp_oracle as O
    from threadpoolctl import threadpool_info, threadpool_limits
    with threadpool_limits(limits=threads):
        cores = max([p.get("num_threads", 1) for p in threadpool_info()] or [os.cpu_count() or 1])
        p0 = wl.init_params(cfg, 0)
        xs, ys = wl.make_data(cfg, 1, 0)
        t0 = time.perf_counter()
        O.train_schedule(cfg, p0, xs, ys, rule, keep_versions=False)
        one = time.perf_counter() - t0
        steps = int(max(1, min(512, budget_s // max(one, 1e-3))))
        if steps > 1:
            xs, ys = wl.make_data(cfg, steps, 0)
            t0 = time.perf_counter()
            O.train_schedule(cfg, p0, xs, ys, rule, keep_versions=False)
            total = time.perf_counter() - t0
        else:
            total = one
    return {"value": cfg.N * cfg.B * steps / total, "unit": "samples/s", "cores": int(cores), "kind": "oracle",
            "sample": "%d full training step(s) of %s under the same rule, fp64 numpy timeline oracle, %.1f s"
                      % (steps, cfg.name, total)}


def run_workload(name, rule, steps, warmup, n_batches=4, dp_batched=False, reps=1, dw_group=1):
    cfg = wl.get_config(name)
    r = gpu_run(cfg, rule, steps, warmup, n_batches, dp_batched, reps, dw_group)
    samples = cfg.N * cfg.B * steps
    prof = r["prof"]
    # event-to-event times minus what an empty event pair reads: the kernels' own durations
    raw_ms = prof["total_ms"]
    prof["total_ms"] = max(raw_ms - prof["launches"] * prof["empty_pair_ms"], 0.25 * raw_ms)
    sec = prof["total_ms"] * 1e-3
    ai = prof["flops"] / max(prof["bytes"], 1.0)
    ridge = MFMA_PEAK_TFLOPS[cfg.dtype] * 1e12 / (HBM_PEAK_GBS * 1e9)
    if ai < ridge:
        roof = {"bound": "hbm", "achieved": prof["bytes"] / sec / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s"}
    else:
        roof = {"bound": "mfma", "achieved": prof["flops"] / sec / 1e12, "peak": MFMA_PEAK_TFLOPS[cfg.dtype], "unit": "TFLOP/s"}
    roof["frac"] = roof["achieved"] / roof["peak"]
    roof["traffic"] = measured_traffic(name)
    roof["kernel"] = KERNELS[name]
    roof["launches"] = prof["launches"]
    roof["avg_launch_us"] = prof["total_ms"] * 1e3 / max(1, prof["launches"])
    roof["algorithmic_bytes_per_launch"] = prof["bytes"] / max(1, prof["launches"])
    roof["algorithmic_flops_per_launch"] = prof["flops"] / max(1, prof["launches"])
    roof["arithmetic_intensity_flop_per_byte"] = ai
    roof["mfma_tflops"] = prof["flops"] / sec / 1e12
    roof["mfma_frac"] = roof["mfma_tflops"] / MFMA_PEAK_TFLOPS[cfg.dtype]
    roof["contraction_time_share"] = prof["total_ms"] / prof["pass_ms"]
    roof["event_pair_overhead_us"] = prof["empty_pair_ms"] * 1e3
    roof["avg_launch_us_with_event_overhead"] = raw_ms * 1e3 / max(1, prof["launches"])
    roof["timed_in"] = "a second pass over the same %d steps with a HIP event pair around every contraction launch " \
                       "(%.3f ms/step with the events, %.3f without)" % (steps, prof["pass_ms"] / steps, r["gpu_ms"] / steps)
    return {
        "metric": "CDP training samples/sec on 1 MI355X",
        "value": samples / r["wall"],
        "unit": "samples/s",
        "n_gpus": 1,
        "steps": steps,
        "warmup": warmup,
        "ms_per_step": r["wall"] * 1e3 / steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16" if cfg.dtype == wl.BF16 else "f32",
        "data": "synthetic",
        "config": {"workload": "%s: %s" % (name, WORKLOAD_TEXT[name]),
                   "rule": wl.RULE_NAMES[rule] + ("_batched" if dp_batched else ""),
                   "S": cfg.S, "N": cfg.N, "B": cfg.B, "delay_ticks": cfg.delay if rule != wl.RULE_DP else 0,
                   "dw_group": dw_group},
        "gpu_ms_per_step": r["gpu_ms"] / steps,
        "repetitions": {"n": reps, "ms_per_step": [w * 1e3 / steps for w in r["walls"]], "reported": "median"},
        "activation_bytes_per_tick": r["act"],
        "peak_activation_bytes": r["stats"]["peak_activation_bytes"],
        "dp_activation_bytes": r["stats"]["dp_activation_bytes"],
        "tick_workspace_bytes": r["stats"]["scratch_bytes"],
        "peak_live_stage_inputs": r["stats"]["peak_live_stage_inputs"],
        "kernel_launches_per_step": r["stats"]["kernel_launches"] / max(1, r["stats"]["steps_enqueued"]),
        "last_step_mean_loss": float(np.mean(r["last_losses"])),
        "roofline": roof,
    }


def lockstep_summary(name, steps):
    """The same workload under the lock-step DP timeline with one batched pass per stage: what
    the cyclic schedule trades (weights re-read per micro-batch) for its smaller activation
    footprint (Table 1, single-GPU rows)."""
    w = run_workload(name, wl.RULE_DP, steps, 2, n_batches=2, dp_batched=True)
    return {"value": w["value"], "unit": w["unit"], "ms_per_step": w["ms_per_step"], "steps": steps,
            "peak_activation_bytes": w["peak_activation_bytes"], "peak_live_stage_inputs": w["peak_live_stage_inputs"]}


def grouped_summary(name, rule, steps, g):
    """The same workload with the weight gradients of g consecutive micro-batches of a stage taken in one
    pass over the accumulator (cdp_opts.dw_group): a g-th of the accumulator traffic, paid in activation memory."""
    w = run_workload(name, rule, steps, 3, n_batches=2, reps=3, dw_group=g)
    return {"value": w["value"], "unit": w["unit"], "ms_per_step": w["ms_per_step"], "steps": steps,
            "peak_activation_bytes": w["peak_activation_bytes"], "activation_bytes_per_tick": w["activation_bytes_per_tick"],
            "roofline_frac": w["roofline"]["frac"], "algorithmic_bytes_per_launch": w["roofline"]["algorithmic_bytes_per_launch"]}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None)
    ap.add_argument("--warmup", type=int, default=None)
    ap.add_argument("--reps", type=int, default=5, help="repetitions of the timed pass of the headline workload (median reported)")
    ap.add_argument("--workload", default="cfg5", choices=sorted(WORKLOAD_TEXT),
                    help="headline workload; default: the largest configuration (cfg5, 407 M parameters)")
    ap.add_argument("--rule", default="v2", choices=["dp", "dp_batched", "v1", "v2"],
                    help="dp: lock-step timeline pass by pass; dp_batched: lock-step with the N micro-batches of a "
                         "step as one batch per stage pass (the throughput baseline of the cyclic rules v1 / v2)")
    ap.add_argument("--no-dp-baseline", action="store_true",
                    help="skip the short lock-step (dp_batched) run of the same workload reported under \"lockstep_dp\"")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--also", default="cfg4,cfg2",
                    help="comma-separated further workloads summarised under \"workloads\" (short runs); empty for none")
    ap.add_argument("--dw-group", type=int, default=1,
                    help="weight gradients of this many consecutive micro-batches of a stage in one accumulator pass (Linear layers)")
    ap.add_argument("--no-dw-group-rows", action="store_true",
                    help="skip the short dw_group = 2 / 4 runs of the headline workload reported under \"dw_group_rows\"")
    ap.add_argument("--calib-copy", action="store_true",
                    help="also run one plain 1 GiB device copy (reference for scaling rocprofv3 FETCH_SIZE / WRITE_SIZE)")
    args = ap.parse_args()
    if args.gpus != 1:
        raise SystemExit("bench.py: this build runs the CDP hot path on ONE GPU; --gpus %d is not supported "
                         "(no collectives or sharding are part of it)" % args.gpus)
    cfg = wl.get_config(args.workload)
    rule = {"dp": wl.RULE_DP, "dp_batched": wl.RULE_DP, "v1": wl.RULE_V1, "v2": wl.RULE_V2}[args.rule]
    batched = args.rule == "dp_batched"
    default_steps = {"cfg1": 200, "cfg2": 200, "cfg3": 20, "cfg4": 5, "cfg5": 20, "vit_b16": 5}[args.workload]
    steps = args.steps if args.steps is not None else default_steps
    warmup = args.warmup if args.warmup is not None else 3
    if args.calib_copy:
        import torch
        src = torch.ones(1 << 28, dtype=torch.float32, device="cuda")   # 1 GiB read + 1 GiB written
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    out = run_workload(args.workload, rule, steps, warmup, dp_batched=batched, reps=max(1, args.reps), dw_group=args.dw_group)
    if args.also:
        out["workloads"] = {}
        for name in args.also.split(","):
            name = name.strip()
            if name and name != args.workload:
                short = {"cfg1": 100, "cfg2": 100, "cfg3": 10, "cfg4": 3, "cfg5": 10, "vit_b16": 3}[name]
                w = run_workload(name, rule, short, 2, n_batches=2, dp_batched=batched, reps=3)
                out["workloads"][name] = {k: w[k] for k in ("value", "unit", "ms_per_step", "steps", "dtype", "config", "repetitions",
                                                            "peak_activation_bytes", "dp_activation_bytes",
                                                            "activation_bytes_per_tick", "roofline")}
                if not args.no_dp_baseline and not batched:
                    out["workloads"][name]["lockstep_dp"] = lockstep_summary(name, short)
    if not args.no_dp_baseline and not batched:
        out["lockstep_dp"] = lockstep_summary(args.workload, max(2, steps // 4))
    if not args.no_dw_group_rows and not batched and rule != wl.RULE_DP and args.dw_group == 1 and args.workload in ("cfg1", "cfg2", "cfg5"):
        out["dw_group_rows"] = {str(g): grouped_summary(args.workload, rule, max(2, steps // 2), g) for g in (2, 4) if cfg.N % g == 0}
    # The stated target of the build: the grouped contraction of a tick at >= 50 % of the bf16 MFMA peak.  The
    # Linear workloads sit far below the MFMA / HBM ridge (arithmetic intensity ~ micro-batch rows), so for
    # them the HBM fraction is the bound; the convolution workload is where the MFMA fraction is meaningful.
    tgt = out if args.workload == "cfg4" else out.get("workloads", {}).get("cfg4")
    out["target"] = {"statement": "tick grouped contraction at >= 50 % of the bf16 MFMA peak", "target_frac": 0.5,
                     "headline_workload_mfma_frac": out["roofline"]["mfma_frac"],
                     "headline_workload_bound": out["roofline"]["bound"], "headline_workload_roof_frac": out["roofline"]["frac"],
                     "cfg4_mfma_frac": tgt["roofline"]["mfma_frac"] if tgt else None,
                     "met": bool(max(out["roofline"]["mfma_frac"], tgt["roofline"]["mfma_frac"] if tgt else 0.0) >= 0.5)}
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cfg, rule)
        # single-thread figures for the two small configurations
        out["cpu_baseline_single_thread"] = {n: cpu_baseline(wl.get_config(n), rule, budget_s=4.0, threads=1) for n in ("cfg1", "cfg2")}
    print(json.dumps(out))


if __name__ == "__main__":
    main()
