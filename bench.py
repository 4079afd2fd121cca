#!/usr/bin/env python3
"""Benchmark: Natural GaLore optimizer steps/s on one MI355X.

One step = one pass of the whole hot path (project, Gram row, s x s solve,
transform + Adam, back-project + weight write) over every matrix of a synthetic
Llama-shaped layer set, gradients and weights resident in HBM.  Prints ONE JSON
line.  `--gpus` above 1 is refused: this build is single-GPU.
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

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E
MFMA_PEAK_TFLOPS = {"bf16": 2500.0, "f32": 157.3}


def algorithmic_work(cfg, mats, hist_dtype="f32"):
    """Bytes and flops per step and phase (algorithmic: every operand moved once)."""
    s, r = cfg.s, cfg.r
    e = 2 if cfg.dtype == "bf16" else 4          # gradient / weight / GEMM-operand element size
    hb = 2.0 if hist_dtype == "bf16" else 4.0    # history element size
    w = {k: {"bytes": 0.0, "flops": 0.0} for k in ("project", "gram", "solve", "adam", "update")}
    for (m, n) in mats:
        rn, mn, mr = r * n, m * n, m * r
        w["project"]["bytes"] += e * mn + e * mr + hb * rn
        w["project"]["flops"] += 2.0 * mn * r
        w["gram"]["bytes"] += hb * s * rn
        w["gram"]["flops"] += 2.0 * s * rn
        w["adam"]["bytes"] += hb * s * rn + 16 * rn + e * rn
        w["adam"]["flops"] += 2.0 * s * rn + 12 * rn
        w["update"]["bytes"] += e * mr + e * rn + 2 * e * mn
        w["update"]["flops"] += 2.0 * mn * r
        w["solve"]["bytes"] += 8.0 * s * s
    return w


def cpu_baseline(cfg, ls, grads_pool, weights, per_shape_s=5.0):
    """The float64 oracle timed on the host cores: one matrix of each distinct shape,
    one warm + one timed step each, scaled by the shape's multiplicity."""
    import numpy as np
    import torch

    import oracle

    def to_f64(t):
        return t.detach().to(torch.float64).cpu().numpy()

    try:
        from threadpoolctl import threadpool_info
        threads = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:
        threads = len(os.sched_getaffinity(0))
    hp = oracle.HParams(s=cfg.s, lam=cfg.lam, beta1=cfg.beta1, beta2=cfg.beta2, eps=cfg.eps, weight_dtype=cfg.dtype)
    mats = cfg.matrices()
    total = 0.0
    parts = []
    for (m, n, mult) in cfg.distinct_shapes():
        i = mats.index((m, n))
        st = oracle.init_state(m, n, cfg.r, cfg.s, "right" if ls.descs[i].side == 1 else "left")
        st.P = to_f64(ls.P(i))
        W = to_f64(weights[i])
        G0 = to_f64(grads_pool[0][i])
        G1 = to_f64(grads_pool[1 % len(grads_pool)][i])
        W = oracle.step(st, G0, W, cfg.lr, hp)          # warm (allocations, BLAS threads)
        reps, spent = 0, 0.0
        while reps < 2 or (spent < per_shape_s and reps < 50):
            G = to_f64(grads_pool[(reps + 1) % len(grads_pool)][i])
            t0 = time.perf_counter()
            W = oracle.step(st, G, W, cfg.lr, hp)
            spent += time.perf_counter() - t0
            reps += 1
        dt = spent / reps
        total += dt * mult
        parts.append("%dx%d: %d steps, %.3f s/step" % (m, n, reps, dt))
    return {"value": 1.0 / total, "unit": "steps/s", "cores": int(threads), "kind": "oracle",
            "sample": "1 matrix of each distinct shape stepped for about %.0f s (%s), mean step time scaled by "
                      "the shape's multiplicity to the %d-matrix set; numpy float64"
                      % (per_shape_s, "; ".join(parts), len(mats))}


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--config", default="c5")
    ap.add_argument("--pool", type=int, default=4, help="pre-generated gradient sets cycled through")
    ap.add_argument("--dtype", default=None, choices=["f32", "bf16"],
                    help="override the configuration's gradient / weight type")
    ap.add_argument("--hist-dtype", default="f32", choices=["f32", "bf16"],
                    help="storage type of the history ring (the benchmark configurations fix f32)")
    ap.add_argument("--sides", default="left", choices=["left", "auto"],
                    help="auto: right-side projection where m > n (the benchmark configurations fix left)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-phase-events", action="store_true")
    ap.add_argument("--no-microbench", action="store_true")
    ap.add_argument("--refresh-in-loop", type=int, default=None,
                    help="refresh every this many timed steps (0 = never); default: 200 for c4, whose "
                         "definition counts one refresh per 200 timed steps (run it with --steps 400), else 0")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="MIB",
                    help="instead of the benchmark, run 10 plain device-to-device copies of MIB MiB "
                         "(calibration of the rocprofv3 FETCH_SIZE / WRITE_SIZE counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on exactly one GPU (matrices are independent; sharding by "
              "matrix is a design note, not built). Re-run with --gpus 1.", file=sys.stderr)
        return 2

    import torch

    from paper_2410_16029_amd import binding as B
    from paper_2410_16029_amd import workloads

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = "cuda:0"
    torch.cuda.set_device(0)
    if args.calibrate_copy:
        n = args.calibrate_copy * (1 << 20) // 4
        src = torch.ones(n, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        for _ in range(10):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"calibrate_copy_bytes_read": n * 4, "calibrate_copy_bytes_written": n * 4, "copies": 10}))
        return 0
    cfg = workloads.CONFIGS[args.config]
    if args.refresh_in_loop is None:
        args.refresh_in_loop = 200 if args.config == "c4" else 0
    if args.dtype is not None:
        import dataclasses
        cfg = dataclasses.replace(cfg, dtype=args.dtype)
    mats = cfg.matrices()

    stream = workloads.TorchGradientStream(mats, cfg.k, cfg.noise, cfg.seed, cfg.dtype, dev)
    pool = [stream.next_set() for _ in range(max(1, args.pool))]
    weights = workloads.torch_weights(mats, cfg.seed, cfg.dtype, dev)
    ls = B.LayerSet(mats, cfg.r, s=cfg.s, lam=cfg.lam, beta1=cfg.beta1, beta2=cfg.beta2, eps=cfg.eps,
                    dtype=cfg.dtype, device=dev, hist_dtype=args.hist_dtype,
                    sides=None if args.sides == "left" else args.sides)
    torch.cuda.synchronize()

    # projector refresh at step 0 (timed separately, not part of `value`)
    t0 = time.perf_counter()
    ls.refresh(pool[0])
    torch.cuda.synchronize()
    refresh_ms = (time.perf_counter() - t0) * 1e3
    assert ls.status() == B.NG_OK, "refresh reported a numeric failure"

    gptr = [B._ptr_array([g.data_ptr() for g in gs]) for gs in pool]
    wptr = B._ptr_array([w.data_ptr() for w in weights])
    st, cur = ls.st, ls.stream()

    # the timed steps must find the history ring full (steady state): at least s warm-up steps
    if args.warmup < cfg.s:
        print("bench.py: warm-up raised from %d to %d steps (the history ring holds s = %d slots)"
              % (args.warmup, cfg.s, cfg.s), file=sys.stderr)
        args.warmup = cfg.s
    for k in range(args.warmup):
        B.ng_step(st, gptr[k % len(pool)], wptr, cfg.lr, cur)
    torch.cuda.synchronize()
    if not args.no_phase_events:
        B.ng_set_profiling(st, True)
        B.ng_get_phase_ms(st, reset=True)

    n_refresh = 0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        if args.refresh_in_loop and k > 0 and k % args.refresh_in_loop == 0:
            ls.refresh(pool[k % len(pool)])
            n_refresh += 1
        B.ng_step(st, gptr[k % len(pool)], wptr, cfg.lr, cur)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    assert ls.status() == B.NG_OK, "a step reported a numeric failure"

    ms_per_step = elapsed * 1e3 / args.steps
    work = algorithmic_work(cfg, mats, args.hist_dtype)
    # Matrices whose two history passes are one launch have their share of the Gram row and the solve in the
    # phase "adam", with the history read once.
    separate = [x for i, x in enumerate(mats) if B._lib.ng_debug_history_tiles(st, i) == 0]
    for name in ("gram", "solve"):
        work[name] = algorithmic_work(cfg, separate, args.hist_dtype)[name]
    phases = {}
    if not args.no_phase_events:
        ms, nsteps = B.ng_get_phase_ms(st, reset=True)
        B.ng_set_profiling(st, False)
        for name, total_ms in zip(B.PHASE_NAMES, ms):
            avg = total_ms / max(nsteps, 1)
            ph = {"ms": round(avg, 4)}
            if avg > 0:
                ph["GB/s"] = round(work[name]["bytes"] / (avg * 1e-3) / 1e9, 1)
                ph["frac_hbm"] = round(ph["GB/s"] / HBM_PEAK_GBS, 4)
                if name in ("project", "update"):
                    ph["TFLOP/s"] = round(work[name]["flops"] / (avg * 1e-3) / 1e12, 1)
                    ph["frac_mfma"] = round(ph["TFLOP/s"] / MFMA_PEAK_TFLOPS[cfg.dtype], 4)
            phases[name] = ph

    from paper_2410_16029_amd import build as ngbuild

    def measured_traffic(kernel):
        """HBM bytes per launch of `kernel` from the committed rocprofv3 counter summary -- only if that
        summary was taken on a library built from the very sources the loaded one was built from."""
        path = os.path.join(ROOT, "profiles", "%s_%s_hbm_traffic.txt" % (kernel, args.config))
        if args.hist_dtype != "f32" or args.sides != "left" or args.dtype is not None:
            return None   # the committed counter summaries cover the default configuration (f32 history, left side, bf16)
        have = ngbuild.built_hash()
        if have is None or have != ngbuild.source_hash():
            return None
        traffic, recorded = None, None
        try:
            for line in open(path):
                if line.startswith("traffic_bytes_per_launch:"):
                    traffic = float(line.split(":")[1])
                if line.startswith("kernel_source_hash:"):
                    recorded = line.split(":")[1].strip()
        except OSError:
            return None
        return traffic if recorded == have else None

    def microbench():
        """Measured ceilings on this GPU: plain streaming copy and read of 1 GiB (beyond the 256 MB
        memory-side cache) and a bare bf16 MFMA loop, on constant operands (the nominal rate) and on
        pseudo-random operands that change with every MFMA (the clock the chip holds on real data)."""
        n = 1 << 30
        a = torch.ones(n // 4, dtype=torch.float32, device=dev)
        b = torch.empty_like(a)
        torch.cuda.synchronize()
        out = {}
        ms, work = B.ng_microbench(B.NG_MB_COPY, a.data_ptr(), b.data_ptr(), n, 20, cur)
        out["stream_copy_GB/s"] = round(work / (ms * 1e-3) / 1e9, 1)
        ms, work = B.ng_microbench(B.NG_MB_READ, a.data_ptr(), b.data_ptr(), n, 20, cur)
        out["stream_read_GB/s"] = round(work / (ms * 1e-3) / 1e9, 1)
        ms, work = B.ng_microbench(B.NG_MB_MFMA_BF16, 0, b.data_ptr(), 8192, 20, cur)
        out["mfma_bf16_TFLOP/s"] = round(work / (ms * 1e-3) / 1e12, 1)
        ms, work = B.ng_microbench(B.NG_MB_MFMA_BF16_RANDOM, 0, b.data_ptr(), 8192, 20, cur)
        out["mfma_bf16_random_operands_TFLOP/s"] = round(work / (ms * 1e-3) / 1e12, 1)
        del a, b
        return out

    roofline = None
    if phases:
        dom = max(phases, key=lambda k: phases[k]["ms"])
        if dom in ("project", "update") and cfg.dtype == "bf16" and args.config == "c5":
            # at the 1.1B shapes the two GEMMs sit at the MFMA/HBM ridge; price them against MFMA
            roofline = {"kernel": dom, "bound": "mfma", "achieved": phases[dom]["TFLOP/s"],
                        "peak": MFMA_PEAK_TFLOPS[cfg.dtype], "unit": "TFLOP/s",
                        "frac": phases[dom]["frac_mfma"], "traffic": measured_traffic(dom)}
        else:
            roofline = {"kernel": dom, "bound": "hbm", "achieved": phases[dom].get("GB/s"),
                        "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": phases[dom].get("frac_hbm"),
                        "traffic": measured_traffic(dom)}

    out = {
        "metric": "natural_galore_optimizer_steps_per_s",
        "value": round(args.steps / elapsed, 3),
        "unit": "steps/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": cfg.dtype if cfg.dtype != "f32" else "f32", "data": "synthetic",
        "config": {"workload": "%s: %d matrices, rank %d, history s=%d, %s gradients/weights, fp32 moments, %s history"
                               % (cfg.name, len(mats), cfg.r, cfg.s, cfg.dtype, args.hist_dtype)
                               + ("" if args.sides == "left" else ", right-side projection where m > n"),
                   "config_key": args.config, "refreshes_in_timed_region": n_refresh,
                   "gradient_pool": len(pool)},
        "roofline": roofline,
        "phases": phases,
        "step_total": {"GB": round(sum(p["bytes"] for p in work.values()) / 1e9, 3),
                       "GFLOP_gemm": round((work["project"]["flops"] + work["update"]["flops"]) / 1e9, 1),
                       "frac_hbm_whole_step": round(sum(p["bytes"] for p in work.values()) / 1e9
                                                    / (ms_per_step * 1e-3) / HBM_PEAK_GBS, 4)},
        "refresh_ms": round(refresh_ms, 2),
    }
    if phases and cfg.dtype == "bf16":
        fr = {k: phases[k].get("frac_mfma") for k in ("project", "update")}
        out["gemm_mfma_target"] = {"target_frac": 0.6, "project": fr["project"], "update": fr["update"],
                                   "met": all(v is not None and v >= 0.6 for v in fr.values())}
    if not args.no_microbench:
        out["microbench"] = microbench()
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cfg, ls, pool, weights)
    print(json.dumps(out))
    return 0


if __name__ == "__main__":
    sys.exit(main())
