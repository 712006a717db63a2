"""Benchmark of the QR-Orth calibration step (the loop body of Alg. 1 of DartQuant) on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config 7b|13b|70b|tiny|heads]

A "step" is one dq_calib_step: QR of the latent Z, Y = X R, fused Whip loss/gradient, G = X^T dY,
the derivative through the QR and the SGD update, on one synthetic activation block that is already
resident in HBM.  Prints ONE JSON line (metric: steps per second).

Without --config the line covers both sizes the metric is quoted on: the headline fields are those of the 7b shape
(n = 4096, T = 8192) and `also` holds the same measurement of the 70b shape (n = 8192, T = 16384), each with
 * `roofline`: the kernel class that takes most of the step, algorithmic work over the summed duration of its
   launches (HIP events around every launch inside a repeat of the timed steps, minus the calibrated cost of an
   event bracket),
 * `stage_roofline`: every stage entry point timed on its own after the timed region (share of the fp32 / bf16
   matrix-core peak and, for the Whip pass, of the HBM peak).
`cpu_baseline` is the fp64 oracle timed on the host on a bounded sample.
"""

from __future__ import annotations

import argparse
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# MI355X published peaks.  The vector-ALU figure is 256 CUs x 4 SIMDs x 16 lanes x 2 flop x 2.4 GHz without packed
# fp32 instructions, which this build keeps the compiler from forming.
PEAK = {"fp32_mfma_tflops": 157.3, "bf16_mfma_tflops": 2500.0, "hbm_gbs": 8000.0, "fp32_valu_tflops": 78.6}

# kernel that takes most of the time of each bracketed class (as named in the rocprofv3 summaries under profiles/)
CLASS_KERNEL = {"gemm_f32": "gemm_f32x3_kernel", "gemm_bf16": "gemm_bf16_nt_big_kernel", "whip": "whip_kernel"}


def flops_per_step(n: int, T: int, b: int = 1, optimizer: str = "sgd") -> float:
    """Dense flop model of one step: two T x n x n products plus (4/3 + 4/3 + 4) n^3 for QR, forming R and
    the derivative through the QR; with the Cayley optimiser (Alg. 3) six n x n products instead of the QR side."""
    side = 12.0 if optimizer == "cayley" else 20.0 / 3.0
    return b * (4.0 * T * n * n + side * n ** 3)


def measured_traffic(cfg_name: str, kernel: str | None):
    """HBM bytes per launch (fetch + write) of `kernel` from the committed counter summary of this workload
    (profiles/calib_step_<workload>_hbm_traffic.txt, written from two rocprofv3 --pmc passes); None if there is none.
    Counters cannot be read from inside this script."""
    if kernel is None:
        return None, None
    path = os.path.join(ROOT, "profiles", f"calib_step_{cfg_name}_hbm_traffic.txt")
    if not os.path.exists(path):
        return None, None
    for line in open(path):
        m = re.match(r"\s*(\S+)\s+([\d.]+)\s+([\d.]+)\s+([\d.]+)\s+([\d.]+)\s+([\d.]+)\s*$", line)
        if m and m.group(1) == kernel:
            return (float(m.group(5)) + float(m.group(6))) * 1024.0, os.path.relpath(path, ROOT)
    return None, None


def cpu_baseline(cfg_name: str, n: int, T: int):
    """Time the oracle as it stands on a bounded sample (a smaller problem with the same value recipe and
    T/n ratio, about 10-30 s of host work) and scale to the benchmark's step with the flop model."""
    from oracle import dartqr_oracle as orc
    from paper_2511_04063_amd import synth

    ns = min(n, 2048)
    Ts = max(1, int(round(T * ns / n)))
    base = cfg_name if cfg_name in ("7b", "13b", "70b") else "7b"
    inp = synth.make_inputs(synth.scaled_config(base, n=ns, T=Ts, b=1), seed=11)
    t0 = time.perf_counter()
    orc.calib_step(inp["X"][0], inp["Z0"][0], 1e-2)
    dt = time.perf_counter() - t0
    scale = flops_per_step(ns, Ts) / flops_per_step(n, T)
    try:
        from threadpoolctl import threadpool_info
        cores = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:
        cores = os.cpu_count() or 1
    return {
        "value": (1.0 / dt) * scale, "unit": "steps/s", "cores": int(cores), "kind": "oracle",
        "sample": (f"one fp64 NumPy oracle step at n={ns}, T={Ts} ({dt:.2f} s), scaled to n={n}, T={T} "
                   f"with the flop model 4Tn^2 + 20/3 n^3 (extrapolated)"),
        "sample_seconds": dt,
    }


def run_config(cfg_name: str, args):
    """Everything measured on one workload; returns the fields of the JSON line that belong to it."""
    import torch

    from paper_2511_04063_amd import binding as B
    from paper_2511_04063_amd import synth

    cfg = synth.CONFIGS[cfg_name]
    inp = synth.make_inputs(cfg)
    bf16 = cfg.x_dtype == "bf16"
    xdt = B.DQ_BF16 if bf16 else B.DQ_F32
    X = torch.from_numpy(inp["X"])
    if bf16:
        X = X.to(torch.bfloat16)
    Xd = X.cuda()
    Z0 = torch.from_numpy(inp["Z0"]).cuda()
    if cfg.b == 1:
        Xd, Z0 = Xd[0], Z0[0]
    del X, inp
    Zd = Z0.clone()
    Z_latent = Z0                      # the initial latent, also what the stage timings factor
    loss = torch.zeros(cfg.b, device="cuda")

    ctx = B.Context()
    ctx.ensure_workspace(cfg.b, cfg.n, cfg.T, xdt)
    red = B.DQ_REDUCE_TOKEN_MEAN
    objectives = {"whip": B.DQ_OBJ_WHIP, "variance": B.DQ_OBJ_VARIANCE, "kurtosis": B.DQ_OBJ_KURTOSIS,
                  "quant": B.DQ_OBJ_QUANT}
    ctx.dq_set_objective(objectives[args.objective], 4)

    if args.optimizer == "cayley":
        # Alg. 3 moves the rotation itself: it starts from the rotation of the initial latent
        Rc = torch.empty_like(Zd)
        ctx.dq_qr_orth(Z0, Rc)
        R_start = Rc.clone()
        Zd = Rc                                   # what the timed loop resets between its phases
        Z0 = R_start
        m_state = torch.zeros_like(Rc)

        def step():
            ctx.dq_cayley_step(Xd, xdt, Rc, m_state, cfg.lr, red, loss, beta=0.9)
    elif args.optimizer == "adam":
        m_state = torch.zeros_like(Zd)
        v_state = torch.zeros_like(Zd)
        counter = [0]

        def step():
            counter[0] += 1
            ctx.dq_calib_step_adam(Xd, xdt, Zd, m_state, v_state, counter[0], cfg.lr, red, loss)
    else:
        def step():
            ctx.dq_calib_step(Xd, xdt, Zd, cfg.lr, red, loss)

    # warm-up, with every kernel class bracketed once to find where the step's time goes
    for _ in range(max(0, args.warmup - 1)):
        step()
    torch.cuda.synchronize()
    ctx.dq_profile_enable((1 << B.DQ_K_COUNT) - 1)
    step()
    names = {B.DQ_K_GEMM_F32: "gemm_f32", B.DQ_K_GEMM_BF16: "gemm_bf16", B.DQ_K_WHIP: "whip",
             B.DQ_K_PANEL: "qr_panel", B.DQ_K_SMALL: "small"}
    breakdown = {names[k]: ctx.dq_profile_read(k) for k in names}
    dominant = max(names, key=lambda k: breakdown[names[k]]["ms"])
    first_loss = float(loss[0].item())

    # timed region: exactly K steps, no event bracketing
    Zd.copy_(Z0)
    ctx.dq_profile_enable(0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    last_loss = float(loss[0].item())

    # the same K steps again with HIP events around every launch of the dominant class (roofline figures) ...
    Zd.copy_(Z0)
    ctx.dq_profile_enable(1 << dominant)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    dt_bracketed = time.perf_counter() - t1
    dom = ctx.dq_profile_read(dominant)
    # ... and what an event bracket costs by itself: the same brackets around a kernel that does next to nothing (one
    # update of a 4 x 4 matrix).  A bracket spans the dispatch of its kernel as well as the kernel, so this figure is
    # taken off every bracket of the class to obtain kernel time, which is what a kernel trace reports.
    tiny_z = torch.zeros((4, 4), device="cuda")
    tiny_d = torch.zeros((4, 4), device="cuda")
    ctx.dq_profile_enable(1 << B.DQ_K_SMALL)
    for _ in range(256):
        ctx.dq_sgd_update(tiny_z, tiny_d, 0.0)
    cal = ctx.dq_profile_read(B.DQ_K_SMALL)
    bracket_ms = cal["ms"] / max(1, cal["launches"])
    ctx.dq_profile_enable(0)
    flags = ctx.dq_device_flags()

    # the stages one by one (same entry points the step is made of), for the per-stage share of the matrix-core and
    # HBM peaks; outside the timed region
    def stage_times():
        shp = (cfg.b, cfg.n, cfg.n) if cfg.b > 1 else (cfg.n, cfg.n)
        Rb, Ub, Gb, dZb = (torch.empty(shp, device="cuda") for _ in range(4))
        Yb = torch.empty(Xd.shape, device="cuda")
        dYb = torch.empty(Xd.shape, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32)
        lossb = torch.zeros(cfg.b, device="cuda")
        Zs = Z_latent.clone()

        def tm(f, reps=5):
            f(); f()
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(reps):
                f()
            torch.cuda.synchronize()
            return (time.perf_counter() - t) / reps * 1e3

        n, T, b = cfg.n, cfg.T, cfg.b
        out = {}
        ms = tm(lambda: ctx.dq_qr_orth(Zs, Rb, Ub))
        fl = b * (8.0 / 3.0) * n ** 3
        out["qr_orth"] = {"ms": ms, "model_tflops": fl / ms / 1e9, "frac_fp32_mfma_peak": fl / ms / 1e9 / PEAK["fp32_mfma_tflops"]}
        ms = tm(lambda: ctx.dq_rotate_loss_grad(Xd, xdt, Rb, red, lossb, Gb))
        fl = b * 4.0 * T * n * n
        peak = PEAK["bf16_mfma_tflops"] if bf16 else PEAK["fp32_mfma_tflops"]
        out["rotate_loss_grad"] = {"ms": ms, "model_tflops": fl / ms / 1e9,
                                   ("frac_bf16_mfma_peak" if bf16 else "frac_fp32_mfma_peak"): fl / ms / 1e9 / peak}
        ms = tm(lambda: ctx.dq_qr_backward(Rb, Ub, Gb, dZb))
        fl = b * 4.0 * n ** 3
        out["qr_backward"] = {"ms": ms, "model_tflops": fl / ms / 1e9}
        if n % 4096 == 0:
            # 3 n^3 of the stage's model flops run on the bf16 matrix cores from three-plane splits (six times issued)
            out["qr_backward"]["issued_bf16_tflops_of_split_products"] = b * 18.0 * n ** 3 / ms / 1e9
            out["qr_backward"]["note"] = ("R^T G and R M run on the bf16 matrix cores from split operands; no single "
                                          "peak prices this stage")
        else:
            out["qr_backward"]["frac_fp32_mfma_peak"] = fl / ms / 1e9 / PEAK["fp32_mfma_tflops"]
        ctx.dq_rotate_loss_grad(Xd, xdt, Rb, red, lossb, Gb, Yb, dYb)
        ms = tm(lambda: ctx.dq_whip_loss_grad(Yb, red, lossb, dYb, xdt))
        by = b * T * n * (4.0 + (2.0 if bf16 else 4.0))
        out["whip_loss_grad"] = {"ms": ms, "bytes": by, "gbs": by / ms / 1e6, "frac_hbm_peak": by / ms / 1e6 / PEAK["hbm_gbs"]}
        # the row-wise objectives of the ablation: the same bytes per element as the Whip pass
        for name in ("variance", "kurtosis", "quant"):
            ms = tm(lambda: ctx.dq_objective_loss_grad(objectives[name], 4, Yb, red, lossb, dYb, xdt))
            out[name + "_loss_grad"] = {"ms": ms, "bytes": by, "gbs": by / ms / 1e6,
                                        "frac_hbm_peak": by / ms / 1e6 / PEAK["hbm_gbs"]}
        return out

    stages = None if args.no_stage_roofline else stage_times()

    host_loop = None
    if args.host_batches > 0 and cfg.b == 1 and args.optimizer == "sgd":
        host = [Xd.cpu().pin_memory() for _ in range(args.host_batches)]
        staging = torch.empty((2,) + tuple(Xd.shape), device="cuda", dtype=Xd.dtype)
        hl = torch.zeros(max(args.steps, 2), device="cuda")
        Zh = Z0.clone()
        ctx.dq_calib_run_host_batches(host, xdt, staging, Zh, cfg.lr, red, 2, hl)
        Zh.copy_(Z0)
        torch.cuda.synchronize()
        th = time.perf_counter()
        ctx.dq_calib_run_host_batches(host, xdt, staging, Zh, cfg.lr, red, args.steps, hl)
        torch.cuda.synchronize()
        th = time.perf_counter() - th
        host_loop = {"batches": args.host_batches, "bytes_per_batch": Xd.numel() * Xd.element_size(),
                     "ms_per_step": th * 1e3 / args.steps, "steps_per_s": args.steps / th,
                     "note": "one batch crosses PCIe per step, overlapped with the previous step"}
        del host, staging

    ms_per_step = dt * 1e3 / args.steps
    n, T, b = cfg.n, cfg.T, cfg.b
    F = flops_per_step(n, T, b, args.optimizer)
    launches = max(1, dom["launches"])
    raw_ms = dom["ms"] / launches
    avg_ms = max(raw_ms - bracket_ms, 1e-6)
    class_s = avg_ms * launches * 1e-3            # summed kernel time of the class over the K steps
    # algorithmic work of the class per step (the model's, not what the launches issue: the QR's products issue
    # 4.7 n^3 where the model counts 8/3 n^3, the rotation product issues its flops twice for the two planes of R)
    # The library's default (DQ_OPT_SPLIT_GEMM = 1) moves the full n^3 products of the derivative (R^T G and R M: 3 n^3 of
    # the model's 4 n^3, the triangular solve stays) and all six of the Cayley update from the fp32 to the bf16 matrix
    # cores where planes pay, 4096 and 8192 of the workloads here (six times the flops issued): the model's flops are booked to
    # the class that runs them.  The other large fp32 products (128 x 128 tiles) split their operands while they read them;
    # they stay in the fp32 class and are priced at the fp32 peak, which they may exceed.
    split = n % 4096 == 0
    side = 12.0 if args.optimizer == "cayley" else 20.0 / 3.0
    moved = (12.0 if args.optimizer == "cayley" else 3.0) if split else 0.0
    if dominant == B.DQ_K_GEMM_F32:
        work = b * ((side - moved) * n ** 3 + (0.0 if bf16 else 4.0 * T * n * n))
        roof = {"bound": "mfma", "achieved": work * args.steps / class_s / 1e12, "peak": PEAK["fp32_mfma_tflops"],
                "unit": "TFLOP/s"}
        # the tiles that split their operands run on the bf16 matrix cores, six products each
        roof["frac_split_peak"] = roof["achieved"] / (PEAK["bf16_mfma_tflops"] / 6.0)
    elif dominant == B.DQ_K_GEMM_BF16:
        work = b * ((4.0 * T * n * n if bf16 else 0.0) + moved * n ** 3)
        roof = {"bound": "mfma", "achieved": work * args.steps / class_s / 1e12, "peak": PEAK["bf16_mfma_tflops"],
                "unit": "TFLOP/s"}
    elif dominant == B.DQ_K_WHIP:
        work = dom["bytes"] / args.steps
        roof = {"bound": "hbm", "achieved": work * args.steps / class_s / 1e9, "peak": PEAK["hbm_gbs"], "unit": "GB/s"}
    else:
        work = dom["flops"] / args.steps
        roof = {"bound": "alu", "achieved": work * args.steps / class_s / 1e12, "peak": PEAK["fp32_valu_tflops"],
                "unit": "TFLOP/s"}
    roof["frac"] = roof["achieved"] / roof["peak"]
    traffic, traffic_src = measured_traffic(cfg.name, CLASS_KERNEL.get(names[dominant]))
    roof["traffic"] = traffic
    roof["traffic_unit"] = ("bytes per launch (fetch + write), from " + traffic_src +
                            " (counter collection serialises the streams: the QR's products are ordered by events there, see that file)"
                            ) if traffic_src else None
    roof["kernel"] = CLASS_KERNEL.get(names[dominant], names[dominant])
    roof["algorithmic_work_per_step"] = work
    roof["launches_per_step"] = dom["launches"] / args.steps
    roof["avg_launch_ms"] = avg_ms
    roof["avg_bracket_ms"] = raw_ms
    roof["bracket_overhead_ms"] = bracket_ms
    roof["class_ms_per_step"] = class_s * 1e3 / args.steps
    roof["ms_per_step_with_events"] = dt_bracketed * 1e3 / args.steps

    out = {
        "value": args.steps / dt,
        "unit": "steps/s",
        "ms_per_step": ms_per_step,
        "config": {"workload": f"{cfg.name}: n={cfg.n}, T={cfg.T}, b={cfg.b}, X {cfg.x_dtype}, Z fp32, "
                               f"{ {'adam': 'Adam', 'sgd': 'SGD', 'cayley': 'Cayley SGD (Alg. 3) on R, momentum 0.9,'}[args.optimizer]} lr={cfg.lr}"
                               + ("" if args.objective == "whip" else f", objective {args.objective}"),
                   "n": cfg.n, "T": cfg.T, "b": cfg.b},
        "dtype": "bf16 X/R/dY on MFMA with fp32 accumulate; fp32 QR and backward" if bf16 else "f32",
        "model_tflops": F / (ms_per_step * 1e-3) / 1e12,
        "flops_per_step": F,
        "loss_first": first_loss, "loss_last": last_loss,
        "device_flags": flags & ~B.DQ_FLAG_ILLCOND_PANEL,
        "panel_fallback_seen": bool(flags & B.DQ_FLAG_ILLCOND_PANEL),
        "roofline": roof,
        "stage_roofline": stages,
        "host_batch_loop": host_loop,
        "stage_ms_one_step": {k: round(v["ms"], 4) for k, v in breakdown.items()},
        "stage_launches_one_step": {k: v["launches"] for k, v in breakdown.items()},
    }
    ctx.close()
    del Xd, Zd, Z0
    torch.cuda.empty_cache()
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", default=None,
                    help="one workload; default: the 7b shape as the headline and the 70b shape beside it")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-stage-roofline", action="store_true",
                    help="skip the separate timing of the stage entry points (used when the run is profiled, so that "
                         "the trace holds calibration steps only)")
    ap.add_argument("--optimizer", choices=["sgd", "adam", "cayley"], default="sgd",
                    help="update rule: Alg. 1's SGD on the latent (the headline metric), Adam on the latent (Sec. 4.3, "
                         "Table 4), or Cayley SGD with momentum on the rotation itself (Alg. 3, the optimiser QR-Orth is "
                         "compared with in Table 4)")
    ap.add_argument("--objective", choices=["whip", "variance", "kurtosis", "quant"], default="whip",
                    help="what S4 evaluates: Eq. 4 (the headline metric) or one of the objectives the paper compares "
                         "it with (Sec. 5, objective ablation)")
    ap.add_argument("--host-batches", type=int, default=0,
                    help="also time the mini-batch loop with this many batches in pinned HOST memory "
                         "(dq_calib_run_host_batches: copies overlap the steps); reported beside the headline value, "
                         "which always has its inputs resident in HBM")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU only (no collectives, no sharding); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)

    head_name = args.config or "7b"
    head = run_config(head_name, args)
    out = {
        "metric": "QR-Orth calibration steps/sec",
        "value": head.pop("value"), "unit": head.pop("unit"),
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": head.pop("ms_per_step"),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": head.pop("dtype"), "data": "synthetic",
    }
    out.update(head)
    if args.config is None:
        # the other size the metric is quoted on, measured the same way (same step count, same warm-up)
        out["also"] = {"70b": run_config("70b", args)}
    if not args.no_cpu_baseline:
        from paper_2511_04063_amd import synth
        cfg = synth.CONFIGS[head_name]
        out["cpu_baseline"] = cpu_baseline(cfg.name, cfg.n, cfg.T)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
