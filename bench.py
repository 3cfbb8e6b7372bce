#!/usr/bin/env python3
"""Benchmark of the hot path on one MI355X.

A step is one full LM train step (embedding .. loss, backward, Adam) on the 12-layer bf16 workload
("cfg3": d_model 2048, 16 heads, FFN 8192, vocab 32768, seq 1024, batch 8) with synthetic seeded
inputs already resident in HBM.  Prints ONE JSON line: whole-step tokens/s, the MFMA roofline of
the GEMM kernel (HIP-event timing of every GEMM launch inside the timed steps), the chained-dispatch
cost per function, and the CPU oracle timed on a bounded sample of the same workload.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload cfg3|cfg5|cfg4|cfg1|ed3|ed1] [--no-cpu-baseline]

Workloads "ed*" are the encoder-decoder step (the second workload: one step = one source batch through the
encoder plus one target batch through the decoder, tokens counted on both sides); the default stays the
decoder-only step the headline metric is quoted on.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0     # MI355X dense bf16 MFMA, published
# The two optional fusions of the LM step (pw_lm_config.fused_update / fused_head_loss) as this benchmark runs them;
# both settings compute the same step, the choice is the faster one as measured on cfg3.
DEFAULT_FUSED_UPDATE = True     # cfg3: 37.45 -> 36.36 ms per step
DEFAULT_FUSED_HEAD_LOSS = False  # cfg3: + 0.78 ms per step (the head GEMM runs twice)


def fill_model_on_device(model, cfg, torch, seed: int):
    """The workload's initial weights - the seeded counter-based generator of inputs.py (N(0, init_std),
    bf16-representable; biases 0, gains 1), evaluated on the GPU - imported tensor by tensor."""
    from paper_2203_12533_amd import binding as pwb
    from paper_2203_12533_amd import inputs as I
    shapes = I.encdec_param_shapes(cfg) if isinstance(cfg, I.EncDecConfig) else I.param_shapes(cfg)
    for name, shape, kind in shapes:
        t = I.param_torch(cfg, name, shape, kind, "cuda", seed)
        torch.cuda.synchronize()      # torch filled t on its own stream; the import runs on the executor stream
        model.import_device(pwb.PW_PARAMS, name, t.data_ptr())
        del t


def recorded_gemm_traffic(workload: str):
    """HBM-side bytes per GEMM launch as measured with rocprofv3 counters (two --pmc runs, scaled by a plain
    copy kernel; see the summary under profiles/).  Counters cannot be collected from inside this process, so
    the recorded figure is reported; None for workloads that were not profiled."""
    path = os.path.join(ROOT, "profiles", f"{workload}_train_step_hbm_traffic.txt")
    try:
        for line in open(path):
            if line.startswith("# all MFMA GEMM launches"):
                return float(line.split("=")[1].split()[0])
    except OSError:
        pass
    return None


def dispatch_bench(ctx, pwb, I, reps: int = 200):
    """Chained dispatch cost (Section 5.1 analogue on one GPU): chains of L trivial functions on a
    128-float buffer.  host = time for the enqueue call to return; wall = until the result is ready.  Busy functions of no
    duration keep a launch each in every mode, so these are costs per dispatched function; the additions of a chain share
    launches, which "additions_stream" shows as a whole."""
    busy = ctx.compile_scalar_fn(pwb.PW_FN_BUSY, 128, 1.0, busy_us=0.0)
    add1 = ctx.compile_scalar_fn(pwb.PW_FN_ADD_CONST, 128, 1.0)
    x = I.dispatch_input()
    out = {}

    def chained(fn, L, mode):
        f_in = ctx.future_from_host(x)
        host_t, wall_t = [], []
        for r in range(reps + 20):
            ctx.synchronize()
            t0 = time.perf_counter()
            (f,) = ctx.chain([fn] * L, [f_in], 1, mode)
            t1 = time.perf_counter()
            ctx.await_(f, fetch=False)
            t2 = time.perf_counter()
            ctx.future_release(f)
            if r >= 20:
                host_t.append(t1 - t0)
                wall_t.append(t2 - t0)
        ctx.future_release(f_in)
        return float(np.median(host_t)) * 1e6, float(np.median(wall_t)) * 1e6

    for L in (1, 8, 32, 128):
        for mode, mname in ((pwb.PW_STREAM, "stream"), (pwb.PW_GRAPH, "graph")):
            host, wall = chained(busy, L, mode)
            out[f"L{L}_{mname}"] = {"host_us_per_fn": round(host / L, 3), "wall_us_per_fn": round(wall / L, 3)}
    out["additions_stream"] = {f"L{L}_wall_us_per_chain": round(chained(add1, L, pwb.PW_STREAM)[1], 2) for L in (1, 8, 32, 128)}
    # op-by-op: one client call per function, each awaited (the stress case of Section 5.1)
    f = ctx.future_from_host(x)
    ctx.synchronize()
    t0 = time.perf_counter()
    for _ in range(128):
        (g,) = ctx.run_fn(busy, [f])
        ctx.await_(g, fetch=False)
        ctx.future_release(f)
        f = g
    out["L128_opbyop"] = {"wall_us_per_fn": round((time.perf_counter() - t0) * 1e6 / 128, 3)}
    ctx.future_release(f)
    return out


def dispatch_bench_c_abi():
    """The pure C++ run of the two dispatch experiments of Section 5.1 (tools/dispatch_bench, built by build()),
    as a child process in its quick mode; returns its summary figures or None if the binary is not there."""
    import subprocess
    exe = os.path.join(ROOT, "paper_2203_12533_amd", "tools", "dispatch_bench")
    if not os.path.exists(exe):
        return None
    try:
        r = subprocess.run([exe, "--quick"], capture_output=True, text=True, timeout=120)
    except (OSError, subprocess.TimeoutExpired):
        return None
    if r.returncode != 0:
        return {"error": r.stderr.strip()[-200:]}
    rows = [json.loads(l) for l in r.stdout.splitlines() if l.startswith("{")]
    out = {}
    for row in rows:
        if row["bench"] == "overhead_masking" and row["computation_us"] == 0:
            out["us_per_computation_at_0us"] = {k: round(1e6 / v, 3) for k, v in row["computations_per_s"].items()}
        if row["bench"] == "overhead_masking_summary":
            out["smallest_computation_us_masking_dispatch"] = row["smallest_computation_us_for_chained_to_reach"]
        if row["bench"] == "parallel_vs_sequential" and row["stages"] == 64:
            out[f"parallel_over_sequential_64_stages_comp{row['computation_us']:g}us_prep{row['host_prep_us']}us"] = \
                row["parallel_over_sequential"]
        if row["bench"] == "proportional_share":
            out["device_time_share_weights_" + "_".join(f"{w:g}" for w in row["weights"])] = row["device_time_share"]
        if row["bench"] == "multi_tenancy" and row["clients"] == 16 and row["computation_us"] > 0:
            out[f"aggregate_over_single_client_16_clients_comp{row['computation_us']:g}us"] = \
                round(row["aggregate_computations_per_s"] / row["one_client_without_scheduler"], 4)
    return out


def cpu_baseline_encdec(cfg, pwb, I, budget_tokens: int = 512):
    """The CPU oracle on a bounded sample of the encoder-decoder workload: one layer each, one sequence pair of
    `budget_tokens` source and target tokens, the workload's widths.  Extrapolated by model-FLOP ratio."""
    from oracle import oracle
    sample = cfg.with_(n_enc_layer=1, n_dec_layer=1, batch=1, src_len=min(cfg.src_len, budget_tokens),
                       tgt_len=min(cfg.tgt_len, budget_tokens))
    params = I.encdec_params(sample)
    src, tgt = I.encdec_tokens(sample)
    secs = oracle.encdec_train_step(sample, params, src, tgt)["seconds"]
    flops_sample = pwb.encdec_step_flops(sample)
    flops_full_per_token = pwb.encdec_step_flops(cfg) / cfg.n_tokens
    return {"value": (flops_sample / secs) / flops_full_per_token, "unit": "tokens/s", "cores": oracle.threads(),
            "kind": "oracle",
            "sample": f"one full oracle encoder-decoder train step (fp64, plain loops) on 1 + 1 layers, batch 1, "
                      f"{sample.src_len} source and {sample.tgt_len} target tokens with the workload's d_model/d_ff/vocab "
                      f"took {secs:.2f} s = {flops_sample / secs / 1e9:.2f} GFLOP/s; tokens/s extrapolated to the full "
                      f"workload by model-FLOP ratio"}


def cpu_baseline(cfg, pwb, budget_flops: float = 0.8e12):
    """The CPU oracle, as it stands, on a bounded sample: same layer / head shapes, one layer, one sequence cut to
    as many tokens (a multiple of 8, at most the workload's) as keep the step near `budget_flops` - about 10 s on
    the host cores.  Extrapolated to the full workload by model-FLOP ratio."""
    if not cfg.has_head:
        return None
    from oracle import oracle
    seq = cfg.seq
    while seq > 8 and pwb.step_flops(cfg.with_(n_layer=1, batch=1, seq=seq)) > budget_flops:
        seq = max(8, (seq * 3 // 4) // 8 * 8)
    sample = cfg.with_(n_layer=1, batch=1, seq=seq)
    secs = oracle.time_train_step(sample)
    flops_sample = pwb.step_flops(sample)
    flops_full_per_token = pwb.step_flops(cfg) / cfg.n_tokens
    tokens_per_s = (flops_sample / secs) / flops_full_per_token
    return {"value": tokens_per_s, "unit": "tokens/s", "cores": oracle.threads(), "kind": "oracle",
            "sample": f"one full oracle train step (fp64, plain loops) on n_layer=1, batch=1, seq={sample.seq} with the "
                      f"workload's d_model/d_ff/vocab took {secs:.2f} s = {flops_sample / secs / 1e9:.2f} GFLOP/s; "
                      f"tokens/s extrapolated to the full workload by model-FLOP ratio"}


class ClockPowerSampler:
    """Reads the engine clock level and the board power from sysfs every 50 ms on a host thread while the timed
    steps run (host reads only; nothing is sent to the GPU).  The step is power-limited on this chip, so the clock
    it actually ran at belongs next to a fraction of a peak that is quoted at the nominal clock."""

    def __init__(self):
        import glob
        self.sclk = sorted(glob.glob("/sys/class/drm/card*/device/pp_dpm_sclk"))[:1]
        hw = sorted(glob.glob("/sys/class/drm/card*/device/hwmon/hwmon*"))[:1]
        self.power = [h + "/power1_input" for h in hw if os.path.exists(h + "/power1_input")] + \
                     [h + "/power1_average" for h in hw if os.path.exists(h + "/power1_average")]
        self.cap = [h + "/power1_cap" for h in hw if os.path.exists(h + "/power1_cap")]
        self.mhz, self.watts = [], []
        self._stop = False
        self._thread = None

    @staticmethod
    def _read(path):
        try:
            with open(path) as f:
                return f.read()
        except OSError:
            return ""

    def _loop(self):
        import re
        while not self._stop:
            for p in self.sclk:
                m = re.search(r"(\d+)\s*Mhz\s*\*", self._read(p))
                if m:
                    self.mhz.append(int(m.group(1)))
            for p in self.power[:1]:
                t = self._read(p).strip()
                if t.isdigit():
                    self.watts.append(int(t) / 1e6)
            time.sleep(0.05)

    def start(self):
        import threading
        self._thread = threading.Thread(target=self._loop, daemon=True)
        self._thread.start()

    def stop(self):
        self._stop = True
        if self._thread is not None:
            self._thread.join()
        note = {}
        if self.mhz:
            note["sclk_mhz_during_timed_steps"] = {"mean": round(sum(self.mhz) / len(self.mhz)), "min": min(self.mhz),
                                                   "max": max(self.mhz), "samples": len(self.mhz)}
        if self.watts:
            note["board_power_w_during_timed_steps"] = {"mean": round(sum(self.watts) / len(self.watts)),
                                                        "max": round(max(self.watts))}
        for p in self.cap:
            t = self._read(p).strip()
            if t.isdigit():
                note["board_power_cap_w"] = round(int(t) / 1e6)
        return note


def device_note(torch, sampled):
    """What the numbers were taken on: device name, compute units, the peak used as the denominator (nominal
    clock), and what the sampler saw of clock and power during the timed steps."""
    prop = torch.cuda.get_device_properties(0)
    note = {"name": prop.name, "arch": getattr(prop, "gcnArchName", ""), "compute_units": prop.multi_processor_count,
            "peak_used_tflops": PEAK_BF16_TFLOPS, "nominal_clock_mhz": 2400}
    note.update(sampled)
    return note


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="cfg3")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-dispatch", action="store_true")
    ap.add_argument("--no-other-workloads", action="store_true",
                    help="with the default workload: skip the short runs of cfg4, cfg5 and ed3 appended under other_workloads")
    ap.add_argument("--graph", action="store_true",
                    help="run the step as one HIP-graph replay (PW_GRAPH); the per-GEMM event timing is then off")
    ap.add_argument("--fused-update", type=int, default=None,
                    help="1: Adam inside the weight-gradient epilogues (LM workloads); default: the build's choice")
    ap.add_argument("--fused-head-loss", type=int, default=None,
                    help="1: LM head fused with the loss, logits never stored; default: the build's choice")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run a plain 1 GiB device copy three times (reference for HBM traffic counters)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on ONE GPU only (no collectives, no sharding); run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2203_12533_amd import binding as pwb
    from paper_2203_12533_amd import inputs as I

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the HIP path has no CPU fallback", file=sys.stderr)
        sys.exit(2)
    torch.cuda.set_device(0)
    result = measure(args, args.workload, args.steps, args.warmup, torch, pwb, I)
    if args.workload == "cfg3" and not args.no_other_workloads:
        # The other workloads of this build, briefly (5 timed steps each), so that one default run shows them all;
        # the headline above stays the cfg3 step.
        result["other_workloads"] = {}
        for w in ("cfg4", "cfg5", "ed3"):
            r = measure(args, w, 5, 2, torch, pwb, I)
            result["other_workloads"][w] = {
                "workload": r["config"]["workload"], "tokens_per_s": r["value"], "ms_per_step": r["ms_per_step"],
                "steps": 5, "warmup": 2, "model_tflop_per_step": r["config"]["model_tflop_per_step"],
                "pct_peak_bf16_mfma": r["pct_peak_bf16_mfma"], "gemm_frac_of_peak": r["roofline"]["frac"],
                "gemm_ms_per_step": r["roofline"]["gemm_ms_per_step"],
                "fused_update_gemm_ms_per_step": r["roofline"].get("fused_update_gemms", {}).get("ms_per_step", 0.0)}
    if not args.no_dispatch:
        with pwb.Context(0) as ctx:
            result["dispatch_us_per_fn"] = dispatch_bench(ctx, pwb, I)
        cabi = dispatch_bench_c_abi()
        if cabi is not None:
            result["dispatch_c_abi"] = cabi
    if not args.no_cpu_baseline:
        encdec = args.workload.startswith("ed")
        cfg = I.encdec_workload(args.workload) if encdec else I.workload(args.workload)
        cb = cpu_baseline_encdec(cfg, pwb, I) if encdec else cpu_baseline(cfg, pwb)
        if cb is not None:
            result["cpu_baseline"] = cb
    print(json.dumps(result))


def measure(args, workload, steps, warmup, torch, pwb, I):
    """Times `steps` steps of one workload (after `warmup` untimed ones) on a context and model of its own; returns
    the result object of the JSON line (without the dispatch and CPU-baseline parts)."""
    encdec = workload.startswith("ed")
    cfg = I.encdec_workload(workload) if encdec else I.workload(workload)
    ctx = pwb.Context(0)
    fused_update = DEFAULT_FUSED_UPDATE if args.fused_update is None else bool(args.fused_update)
    fused_head_loss = DEFAULT_FUSED_HEAD_LOSS if args.fused_head_loss is None else bool(args.fused_head_loss)
    model = ctx.encdec(cfg, fused_update=fused_update) if encdec else ctx.model(cfg, fused_update=fused_update, fused_head_loss=fused_head_loss)
    fill_model_on_device(model, cfg, torch, seed=1234)
    if encdec:
        src_np, tgt_np = I.encdec_tokens(cfg, seed=1234)
        src, tgt = torch.from_numpy(src_np).cuda(), torch.from_numpy(tgt_np).cuda()
        torch.cuda.synchronize()
        f_src = ctx.future_wrap_device(src.data_ptr(), pwb.PW_I32, tuple(src.shape))
        f_tgt = ctx.future_wrap_device(tgt.data_ptr(), pwb.PW_I32, tuple(tgt.shape))
        step = model.compile_train_step()

        def one_step():
            return ctx.run_fn(step, [f_src, f_tgt], 1)[0]
    elif cfg.has_head:
        tok = torch.from_numpy(I.lm_tokens(cfg, seed=1234)).cuda()
        torch.cuda.synchronize()
        f_tok = ctx.future_wrap_device(tok.data_ptr(), pwb.PW_I32, tuple(tok.shape))
        step = model.compile_train_step()

        def one_step():
            if args.graph:
                return ctx.chain([step], [f_tok], 1, pwb.PW_GRAPH)[0]
            return ctx.train_step(step, f_tok)
    else:
        # One pipeline stage under the GPipe-like schedule: forward for every micro-batch, then backward in
        # reverse order with weight gradients summed, then Adam.  The 2 x n_microbatch calls are one chain of
        # compiled functions consuming futures; a step returns the future of the last input gradient.
        gen = torch.Generator(device="cuda")
        gen.manual_seed(4321)
        nmb, shape = cfg.n_microbatch, (cfg.n_tokens, cfg.d_model)
        xs = [torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16).float() for _ in range(nmb)]
        dys = [torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16).float() for _ in range(nmb)]
        torch.cuda.synchronize()
        fx = [ctx.future_wrap_device(t.data_ptr(), pwb.PW_F32, shape) for t in xs]
        fdy = [ctx.future_wrap_device(t.data_ptr(), pwb.PW_F32, shape) for t in dys]
        fwd = [model.compile_stage(pwb.PW_FN_STAGE_FWD, mb) for mb in range(nmb)]
        bwd = [model.compile_stage(pwb.PW_FN_STAGE_BWD, mb) for mb in range(nmb)]

        def one_step():
            model.zero_grads()
            last = None
            for mb in range(nmb):
                (fy,) = ctx.run_fn(fwd[mb], [fx[mb]])
                ctx.future_release(fy)
            for mb in reversed(range(nmb)):
                (fdx,) = ctx.run_fn(bwd[mb], [fdy[mb]])
                if last is not None:
                    ctx.future_release(last)
                last = fdx
            model.apply_optimizer()
            return last

    losses = []
    for _ in range(warmup):
        f = one_step()
        losses.append(float(ctx.await_(f).reshape(-1)[0]))
        ctx.future_release(f)
    ctx.synchronize()
    torch.cuda.synchronize()
    # The GEMM launches of the first `profiled_steps` timed steps are bracketed by HIP events (the roofline
    # figure); each pair costs a few microseconds of stream time, ~2 % of a step if left on throughout.
    profiled_steps = 0 if args.graph else min(2, steps)
    if profiled_steps:
        ctx.profile_begin()
    # per-step durations as well: HIP events on the executor stream between the steps (no synchronisation)
    ext = torch.cuda.ExternalStream(ctx.stream_ptr())
    marks = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    t0 = time.perf_counter()
    pending = []
    sampler = ClockPowerSampler()
    sampler.start()
    marks[0].record(ext)
    for i in range(steps):
        if profiled_steps and i == profiled_steps:
            ctx.profile_pause()
        pending.append(one_step())
        marks[i + 1].record(ext)
    ctx.synchronize()
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    sampled = sampler.stop()
    per_step = sorted(marks[i].elapsed_time(marks[i + 1]) for i in range(steps))
    n_gemm, gemm_ms, gemm_flops = ctx.profile_end() if profiled_steps else (0, 0.0, 0.0)
    n_fu, fu_ms, fu_flops = ctx.profile_fused_update() if profiled_steps else (0, 0.0, 0.0)
    shape_rows = ctx.profile_gemm_shapes() if profiled_steps else []
    for f in pending:
        losses.append(float(ctx.await_(f).reshape(-1)[0]))
        ctx.future_release(f)
    if not all(math.isfinite(l) for l in losses):
        print(f"bench.py: non-finite loss {losses}", file=sys.stderr)
        sys.exit(1)

    if args.calibrate_copy:
        src = torch.empty(1 << 28, dtype=torch.float32, device="cuda").normal_()
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    ms_per_step = dt * 1e3 / steps
    tokens_per_step = cfg.n_tokens * (1 if encdec else cfg.n_microbatch)
    tokens_per_s = tokens_per_step * steps / dt
    flops = pwb.encdec_step_flops(cfg) if encdec else pwb.step_flops(cfg)
    if encdec:
        what = (f"{workload}: encoder-decoder train step, {cfg.n_enc_layer} encoder + {cfg.n_dec_layer} decoder layers, "
                f"d_model {cfg.d_model}, {cfg.n_head} heads, FFN {cfg.d_ff}, vocab {cfg.vocab}, {cfg.src_len} source + "
                f"{cfg.tgt_len} target positions, batch {cfg.batch}, "
                f"{'bf16 compute / fp32 master' if cfg.bf16 else 'fp32'} + {cfg.optimizer}")
        loss_key = "loss_first_last"
    else:
        what = (f"{workload}: {cfg.n_layer}-layer decoder-only LM "
                f"{'train step' if cfg.has_head else f'pipeline stage, {cfg.n_microbatch} micro-batches fwd-all/bwd-all'}, "
                f"d_model {cfg.d_model}, {cfg.n_head} heads, FFN {cfg.d_ff}, vocab {cfg.vocab}, seq {cfg.seq}, "
                f"batch {cfg.batch}, {'bf16 compute / fp32 master' if cfg.bf16 else 'fp32'} + {cfg.optimizer}")
        loss_key = "loss_first_last" if cfg.has_head else "dx0_first_last"
    achieved = flops / (dt / steps) / 1e12
    gemm_tflops = gemm_flops / (gemm_ms * 1e-3) / 1e12 if gemm_ms > 0 else 0.0
    result = {
        "metric": "train tokens/sec/GPU", "value": round(tokens_per_s, 1), "unit": "tokens/s", "n_gpus": 1,
        "steps": steps, "warmup": warmup, "ms_per_step": round(ms_per_step, 3), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "bf16" if cfg.bf16 else "f32", "data": "synthetic",
        "config": {"workload": what, "tokens_per_step": tokens_per_step, "model_tflop_per_step": round(flops / 1e12, 3),
                   "fused_update": bool(fused_update), "fused_head_loss": bool(fused_head_loss and not encdec)},
        "pct_peak_bf16_mfma": round(100.0 * achieved / PEAK_BF16_TFLOPS, 2),
        "step_tflops": round(achieved, 1),
        "ms_per_step_device": {"median": round(per_step[len(per_step) // 2], 3), "min": round(per_step[0], 3),
                               "max": round(per_step[-1], 3)},
        loss_key: [round(losses[0], 4), round(losses[-1], 4)],
        "roofline": {"bound": "mfma", "kernel": "bf16 MFMA GEMM (gemm_ring_kernel, gemm_ring_group_kernel, gemm_tile_kernel; all layouts, general epilogues)", "achieved": round(gemm_tflops, 1),
                     "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s", "frac": round(gemm_tflops / PEAK_BF16_TFLOPS, 4),
                     "traffic": recorded_gemm_traffic(workload), "launches_per_step": n_gemm // max(1, profiled_steps), "steps_with_events": profiled_steps,
                     "avg_launch_ms": round(gemm_ms / max(1, n_gemm), 4),
                     "avg_launch_gflop": round(gemm_flops / max(1, n_gemm) / 1e9, 2),
                     "gemm_ms_per_step": round(gemm_ms / max(1, profiled_steps), 3)},
    }
    if n_fu:
        # The weight-gradient GEMMs that apply Adam in their epilogue are a kernel instantiation of their own: MFMA work
        # plus 26 bytes of optimizer traffic per parameter.  They are priced on both rooflines, next to the GEMM figure.
        shapes = I.encdec_param_shapes(cfg) if encdec else I.param_shapes(cfg)
        fused_params = sum(int(np.prod(sh)) for nm, sh, kind in shapes
                           if nm.split(".")[-1] in ("wqkv", "wo", "wq", "wkv", "wox", "w1", "w2", "wh"))
        result["roofline"]["fused_update_gemms"] = {
            "kernel": "gemm_ring_kernel / gemm_ring_group_kernel with the Adam epilogue (weight-gradient layout)",
            "launches_per_step": n_fu // profiled_steps, "ms_per_step": round(fu_ms / profiled_steps, 3),
            "tflops": round(fu_flops / (fu_ms * 1e-3) / 1e12, 1),
            "optimizer_gb_per_step": round(26.0 * fused_params / 1e9, 2),
            "note": "the same launches without the epilogue's optimizer traffic take about the GEMM family's rate; "
                    "the separate Adam launch they replace moved 30 B/param at 5.5 TB/s"}
        result["roofline"]["gemm_ms_per_step_incl_fused_update"] = round((gemm_ms + fu_ms) / profiled_steps, 3)
    if shape_rows:
        # every GEMM launch of the bracketed steps by (shape, operand layouts, epilogue): which instantiation runs
        # at what rate.  layout "tn" = A k-major, B row-major, and so on; members > 1 = one launch shared by several GEMMs.
        epi_names = ["store", "bias", "bias_residual", "bias_gelu", "gelu_bwd", "adam", "xent_stats", "xent_grad"]
        result["roofline"]["by_shape"] = [
            {"M": r["M"], "N": r["N"], "K": r["K"], "layout": ("t" if r["a_kmajor"] else "n") + ("n" if r["b_kmajor"] else "t"),
             "epilogue": epi_names[r["epilogue"]], "members": r["members"], "launches_per_step": r["launches"] // profiled_steps,
             "avg_us": round(1e3 * r["total_ms"] / r["launches"], 1),
             "tflops": round(r["total_flops"] / (r["total_ms"] * 1e-3) / 1e12, 1)} for r in shape_rows]
    result["device"] = device_note(torch, sampled)
    clk = sampled.get("sclk_mhz_during_timed_steps", {}).get("mean")
    if clk:
        # context, not the headline: the same achieved rate against the matrix peak at the clock the power limit
        # left the chip during the timed steps (published peak x sampled clock / nominal 2400 MHz)
        peak_at_clk = PEAK_BF16_TFLOPS * clk / 2400.0
        result["roofline"]["peak_at_sampled_clock"] = round(peak_at_clk, 1)
        result["roofline"]["frac_at_sampled_clock"] = round(gemm_tflops / peak_at_clk, 4)
    model.close()
    ctx.close()
    return result


if __name__ == "__main__":
    main()
