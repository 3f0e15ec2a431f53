#!/usr/bin/env python3
"""Throughput of the Tucker-compressed VSIE coupling-matrix products on one
MI355X: compressed matvecs/s, counting both Z x and Z^* y.

One step = one Z x (Algorithm 1) and one Z^* y (Algorithm 2) on the default
workload: a 256^3 voxel grid (1 mm voxels), 3 field components, 2048 point
currents on 16 rings, columns compressed on the GPU at tolerance 1e-4 with
ranks capped at 32, complex64 vectors, FP32 products on MFMA.  Inputs are
resident in HBM before the timed region; compression is set-up, not timed.

Prints one JSON line on stdout (progress goes to stderr).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_FP32_MFMA = 157.3      # TFLOP/s, MI355X dense FP32 matrix
PEAK_BF16_MFMA = 2516.6     # TFLOP/s, dense BF16 matrix
PEAK_HBM = 8000.0           # GB/s

# HBM bytes per launch of the dominant kernel: rocprofv3 FETCH_SIZE and
# WRITE_SIZE (KiB per dispatch), each scaled by what the same counter reads for
# a plain copy of known size.  A figure holds only for the kernel source it was
# taken on (checked by hash); after a change it is reported as null until the
# counters are taken again.
MEASURED_TRAFFIC = {
    ("c2", "fp32", "adjoint"): {
        "bytes": 39121810,
        "source": "paper_2103_06393_amd/csrc/tv_fused_ws.hip",
        "sha256": "445803172685202790421745ad3263a637dd9c270cce35e2892f0a98b7a0314b",
        "profile": "profiles/ws_fused_c2_fp32_pmc.md",
        "launch": {"kernel": 1},
    },
    ("c5", "fp32", "adjoint"): {
        "bytes": 71082626731,
        "source": "paper_2103_06393_amd/csrc/tv_dtg_gemm.h",
        "sha256": "b5552eea3a7db2f95c1f26756217baefd772ff9ae18fa22ab5e86a6b13e63447",
        "profile": "profiles/dtg_c5_fp32_pmc.md",
        "launch": {"kernel": 2, "tile_t2": 128, "tile_t3": 4, "splits": 16},
    },
    ("c5", "fp32", "forward"): {
        "bytes": 60664371947,
        "source": "paper_2103_06393_amd/csrc/tv_dtg_gemm.h",
        "sha256": "b5552eea3a7db2f95c1f26756217baefd772ff9ae18fa22ab5e86a6b13e63447",
        "profile": "profiles/dtg_c5_fp32_pmc.md",
        "launch": {"kernel": 2, "tile_t2": 128, "tile_t3": 4, "splits": 1},
    },
    ("aca2-pwc", "fp32", "adjoint"): {
        "bytes": 3657544232,
        "source": "paper_2103_06393_amd/csrc/tv_fused_ws.hip",
        "sha256": "445803172685202790421745ad3263a637dd9c270cce35e2892f0a98b7a0314b",
        "profile": "profiles/aca_tucker_aca2_pwc_pmc.md",
        "launch": {"kernel": 1},
    },
}



KERNEL_FAMILY = {0: "phased", 1: "warp-specialised", 2: "decompress-then-GEMM"}


def kernel_label(family, d):
    """Kernels one product call runs, for the roofline line (d: 0 forward, 1 adjoint)."""
    if family == 0:
        return "tv::fused_f32"
    if family == 1:
        return "tv::ws_fused"
    if d == 0:
        return "tv_matvec call: dtg_decomp_kernel + dtg_split_gemm"
    return ("tv_rmatvec call: dtg_decomp_kernel + dtg_ypack_kernel + dtg_split_gemm + "
            "dtg_colgemm_reduce_kernel")


def mfma_peak(family, fp32):
    """Matrix peak of a product call in algorithmic TFLOP/s: BF16X3 executes
    three BF16 products per algorithmic one; the FP32 decompress-then-GEMM
    path six (an exact split into three planes), the other FP32 paths run on
    the FP32 matrix instructions."""
    if not fp32:
        return PEAK_BF16_MFMA / 3.0
    return PEAK_BF16_MFMA / 6.0 if family == 2 else PEAK_FP32_MFMA


def measured_traffic(workload: str, precision: str, direction: str, info=None):
    """HBM bytes per call from the committed counter profile, or None when
    the kernel source or the launch configuration differs from the profiled one."""
    e = MEASURED_TRAFFIC.get((workload, precision, direction))
    if not e:
        return None
    with open(os.path.join(ROOT, e["source"]), "rb") as f:
        if hashlib.sha256(f.read()).hexdigest() != e["sha256"]:
            return None
    if info is not None:
        d = 1 if direction == "adjoint" else 0
        have = {"kernel": info.kernel[d], "tile_t2": info.tile_t2[d],
                "tile_t3": info.tile_t3[d], "splits": info.splits[d]}
        if any(have[k] != v for k, v in e["launch"].items()):
            return None
    return e["bytes"]


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def time_products(plan, x, y, K, warmup):
    """Warm-up, then K steps of one Z x and one Z^* y on the current stream,
    bracketed by HIP events; returns (fwd_ms, adj_ms, total_ms, wall_s, xo)."""
    import torch
    from paper_2103_06393_amd import lib
    yo = torch.empty(plan.rows, dtype=torch.complex64, device="cuda")
    xo = torch.empty(plan.m, dtype=torch.complex64, device="cuda")
    wsf, wsa = plan.workspace(0, 1), plan.workspace(1, 1)
    st = torch.cuda.current_stream()
    sp = st.cuda_stream
    h = plan.handle

    def fwd():
        lib.tv_matvec(h, x.data_ptr(), plan.m, 1, yo.data_ptr(), plan.rows,
                      wsf.data_ptr(), wsf.numel(), sp)

    def adj():
        lib.tv_rmatvec(h, y.data_ptr(), plan.rows, 1, xo.data_ptr(), plan.m,
                       wsa.data_ptr(), wsa.numel(), sp)

    for _ in range(warmup):
        fwd()
        adj()
    torch.cuda.synchronize()
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(K)]
    start = torch.cuda.Event(enable_timing=True)
    end = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    w0 = time.perf_counter()
    start.record(st)
    for i in range(K):
        ev[i][0].record(st)
        fwd()
        ev[i][1].record(st)
        adj()
        ev[i][2].record(st)
    end.record(st)
    torch.cuda.synchronize()
    wall = time.perf_counter() - w0
    fwd_ms = sum(e[0].elapsed_time(e[1]) for e in ev) / K
    adj_ms = sum(e[1].elapsed_time(e[2]) for e in ev) / K
    return fwd_ms, adj_ms, start.elapsed_time(end), wall, xo


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(wl, plan, x_np, y_np, budget_s: float):
    """Time the FP64 oracle (Algorithms 1 and 2) on the plan's own factors,
    on a column subset sized to about ``budget_s`` seconds, scaled to one
    full product per direction."""
    import numpy as np
    from threadpoolctl import threadpool_info
    from oracle import matvec as om
    from tests.plans import abi_to_struct
    S = abi_to_struct(wl.grid.dims, wl.q, *plan.export_factors())
    m = S.m
    probe = list(range(0, m, max(1, m // 4)))[:4]
    Sp = om.TuckerStruct(S.dims, S.q, [S.t[j] for j in probe])
    t0 = time.perf_counter()
    om.alg1(Sp, x_np[probe])
    om.alg2(Sp, y_np)
    per_col = (time.perf_counter() - t0) / len(probe)
    ms = max(1, min(m, int(budget_s / max(per_col, 1e-6))))
    cols = sorted(set(int(round(v)) for v in np.linspace(0, m - 1, ms)))
    Ss = om.TuckerStruct(S.dims, S.q, [S.t[j] for j in cols])
    t0 = time.perf_counter()
    y_ref = om.alg1(Ss, x_np[cols])[:, 0]
    t1 = time.perf_counter()
    x_ref = om.alg2(Ss, y_np)[:, 0]
    t2 = time.perf_counter()
    scale = m / len(cols)
    per_pair = ((t1 - t0) + (t2 - t1)) * scale
    threads = sum(int(i.get("num_threads", 1)) for i in threadpool_info()
                  if i.get("user_api") == "blas") or 1
    return {
        "value": 2.0 / per_pair, "unit": "matvecs/s", "cores": threads,
        "kind": "oracle", "cpu_model": cpu_model(),
        "sample": f"{len(cols)} of {m} columns of the same plan (FP64 "
                  f"Algorithms 1 and 2 on the GPU plan's factors), scaled "
                  f"by {scale:.2f} to one Z x and one Z^* y",
    }, cols, y_ref, x_ref


def main(argv=None):
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="c5",
                    help="c1, c2, c3, c5 (default), c4 for the batched path, or "
                         "aca5 / aca2 / aca1 for the ACA+Tucker products on the "
                         "body-coil grids")
    ap.add_argument("--basis", default="pwc", choices=("pwc", "pwl"),
                    help="voxel basis of the aca* workloads")
    ap.add_argument("--gemm-reference", action="store_true",
                    help="time the stacked mode-1 GEMM alone with B materialised in HBM "
                         "(library complex GEMM at the workload's shapes)")
    ap.add_argument("--assemble", action="store_true",
                    help="aca* workloads: time Algorithm 3 (tv_aca_assemble) for r_c "
                         "steps instead of the products")
    ap.add_argument("--natural-ranks", action="store_true",
                    help="aca* workloads: keep the HOSVD ranks of the stand-in columns "
                         "instead of clamping them to the paper's reported 15..18")
    ap.add_argument("--precision", default="fp32", choices=("fp32", "bf16x3"))
    ap.add_argument("--cpu-budget", type=float, default=20.0,
                    help="seconds of oracle work for the CPU baseline")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--copy-bytes", type=int, default=0,
                    help="only run a plain device copy of this many bytes --steps "
                         "times (calibration of the HBM traffic counters)")
    ap.add_argument("--no-autotune", action="store_true")
    ap.add_argument("--no-bf16x3", action="store_true",
                    help="skip the BF16 hi/lo split measurement after the FP32 one")
    ap.add_argument("--tune-cache", default=os.path.join(
        os.environ.get("TMPDIR", "/tmp"), "tuckvsie_tune.json"),
        help="autotuner cache (JSON); a cached entry skips the timing runs")
    args = ap.parse_args(argv)
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (asked for --gpus {args.gpus}); "
              "the multi-GPU layout is a design, see the voxel-slab sharding "
              "notes", file=sys.stderr)
        return 2

    import numpy as np
    import torch
    import workloads
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import TuckerPlan

    if args.copy_bytes:
        src = torch.ones(args.copy_bytes // 4, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(args.warmup):
            dst.copy_(src)
        torch.cuda.synchronize()
        for _ in range(args.steps):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes": src.numel() * 4, "copies": args.steps}), flush=True)
        return 0
    if args.workload == "c4":
        return bench_batch(args)
    if args.gemm_reference:
        return bench_gemm_reference(args)
    if args.workload.startswith("aca"):
        return bench_assemble(args) if args.assemble else bench_aca(args)
    prec = lib.TV_PREC_BF16X3 if args.precision == "bf16x3" else lib.TV_PREC_FP32
    wl = workloads.make(args.workload)
    log(f"[bench] workload {wl.name}: grid {wl.grid.dims}, q={wl.q}, m={wl.m}")
    t0 = time.perf_counter()
    plan = TuckerPlan.compress_dipoles(
        wl.grid.dims, wl.grid.h, wl.k0, lib.field_code(wl.basis, wl.operator),
        wl.pos, wl.ori, wl.tol, wl.rank_min, wl.rank_cap or 0, precision=prec)
    torch.cuda.synchronize()
    log(f"[bench] compressed on GPU in {time.perf_counter() - t0:.2f} s")
    if not args.no_autotune:
        t0 = time.perf_counter()
        plan.autotune(2, args.tune_cache)
        torch.cuda.synchronize()
        log(f"[bench] autotuned in {time.perf_counter() - t0:.2f} s "
            f"(workspace fwd {lib.tv_workspace_bytes(plan.handle, 0, 1)} B, "
            f"adj {lib.tv_workspace_bytes(plan.handle, 1, 1)} B)")
    info = plan.info
    x_np = wl.x()[:, 0]
    y_np = wl.y()[:, 0]
    x = torch.from_numpy(x_np.astype(np.complex64)).cuda()
    y = torch.from_numpy(y_np.astype(np.complex64)).cuda()
    K = args.steps
    fwd_ms, adj_ms, total_ms, wall, xo = time_products(plan, x, y, K, args.warmup)
    ms_step = total_ms / K
    value = 2.0 * K / (total_ms / 1e3)
    tf_f = info.flops_matvec / (fwd_ms * 1e-3) / 1e12
    tf_a = info.flops_rmatvec / (adj_ms * 1e-3) / 1e12
    log(f"[bench] fwd {fwd_ms:.4f} ms ({tf_f:.1f} TFLOP/s), adj {adj_ms:.4f} ms "
        f"({tf_a:.1f} TFLOP/s), wall {wall:.3f} s for {K} steps")
    dom = "adjoint" if adj_ms >= fwd_ms else "forward"
    d = 1 if dom == "adjoint" else 0
    info = plan.info  # after autotuning: the launch configuration in use
    kname = kernel_label(info.kernel[d], d)
    pname = "fp32" if prec == lib.TV_PREC_FP32 else "bf16x3"
    ach = tf_a if dom == "adjoint" else tf_f
    peak = mfma_peak(info.kernel[d], prec == lib.TV_PREC_FP32)
    mode1 = 8.0 * wl.grid.n1 * wl.grid.n2 * wl.grid.n3 * info.sum_r1
    arith = ("BF16 hi/lo split" if prec != lib.TV_PREC_FP32 else
             "FP32 (three-plane BF16 split)" if info.kernel[d] == 2 else "FP32")
    out = {
        "metric": "compressed VSIE matvecs/s (Zx and Z^H y), TFLOP/s and % MFMA peak",
        "value": value, "unit": "matvecs/s", "n_gpus": 1, "steps": K,
        "warmup": args.warmup, "ms_per_step": ms_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32" if prec == lib.TV_PREC_FP32 else "bf16x3 (f32 accumulate)",
        "data": "synthetic",
        "config": {
            "workload": f"{wl.name}: {wl.grid.n1}x{wl.grid.n2}x{wl.grid.n3} grid, "
                        f"q={wl.q}, {wl.m} point currents, HOSVD tol {wl.tol:g}, "
                        f"rank cap {wl.rank_cap}, complex64 vectors, "
                        f"{arith} MFMA",
            "grid": list(wl.grid.dims), "q": wl.q, "m": wl.m,
            "mean_rank": [round(v, 3) for v in info.mean_rank],
            "max_rank": list(info.max_rank), "sum_r1": int(info.sum_r1),
            "plan_factor_bytes": int(info.factor_bytes),
        },
        "fwd_ms": fwd_ms, "adj_ms": adj_ms,
        "tflops_fwd": tf_f, "tflops_adj": tf_a,
        "flops_fwd": info.flops_matvec, "flops_adj": info.flops_rmatvec,
        "roofline": {"kernel": f"{kname} ({dom})", "bound": "mfma",
                     "achieved": ach, "peak": peak, "unit": "TFLOP/s",
                     "frac": ach / peak,
                     "traffic": measured_traffic(wl.name, pname, dom, info),
                     # the stacked mode-1 product alone (8 nv sum r1 flops, all
                     # on the matrix cores) over the same duration
                     "mode1_achieved": mode1 / ((adj_ms if dom == "adjoint" else fwd_ms)
                                                * 1e-3) / 1e12,
                     "mode1_frac": mode1 / ((adj_ms if dom == "adjoint" else fwd_ms)
                                            * 1e-3) / 1e12 / peak},
        "launch": {"tile_t2": list(info.tile_t2), "tile_t3": list(info.tile_t3),
                   "splits": list(info.splits),
                   "kernel": [KERNEL_FAMILY[v] for v in info.kernel]},
    }
    if not args.no_cpu:
        cb, cols, y_ref, x_ref = cpu_baseline(wl, plan, x_np, y_np, args.cpu_budget)
        out["cpu_baseline"] = cb
        # parity of the timed configuration on the sampled columns
        xs = np.zeros_like(x_np)
        xs[cols] = x_np[cols]
        ys = plan.matvec(torch.from_numpy(xs.astype(np.complex64)).cuda()).cpu().numpy()
        xa = xo.cpu().numpy()[cols]
        out["rel_err_fwd"] = float(np.linalg.norm(ys - y_ref) / np.linalg.norm(y_ref))
        out["rel_err_adj"] = float(np.linalg.norm(xa - x_ref) / np.linalg.norm(x_ref))
        log(f"[bench] oracle {cb['value']:.4f} matvecs/s on {cb['cores']} threads; "
            f"rel err fwd {out['rel_err_fwd']:.2e} adj {out['rel_err_adj']:.2e}")
    if prec == lib.TV_PREC_FP32 and not args.no_bf16x3:
        # the BF16 hi/lo split form on the same factors and inputs, its
        # speedup over FP32 and its error on the same sampled columns
        fac = plan.export_factors()
        plan.close()
        torch.cuda.empty_cache()
        bplan = TuckerPlan.from_factors(wl.grid.dims, wl.q, wl.m, *fac, lib.TV_PREC_BF16X3)
        del fac
        if not args.no_autotune:
            bplan.autotune(2, args.tune_cache)
        bi = bplan.info
        bf_f, bf_a, bf_total, _, bxo = time_products(bplan, x, y, K, args.warmup)
        bb = {"value": 2.0 * K / (bf_total / 1e3), "ms_per_step": bf_total / K,
              "fwd_ms": bf_f, "adj_ms": bf_a,
              "speedup_vs_fp32": ms_step / (bf_total / K),
              "tflops_fwd": bi.flops_matvec / (bf_f * 1e-3) / 1e12,
              "tflops_adj": bi.flops_rmatvec / (bf_a * 1e-3) / 1e12,
              "peak_three_products": PEAK_BF16_MFMA / 3.0,
              "launch": {"tile_t2": list(bi.tile_t2), "tile_t3": list(bi.tile_t3),
                         "splits": list(bi.splits)}}
        bb["frac"] = max(bb["tflops_fwd"] if bf_f > bf_a else bb["tflops_adj"], 0.0) / (
            PEAK_BF16_MFMA / 3.0)
        if not args.no_cpu:
            ys = bplan.matvec(torch.from_numpy(xs.astype(np.complex64)).cuda()).cpu().numpy()
            bb["rel_err_fwd"] = float(np.linalg.norm(ys - y_ref) / np.linalg.norm(y_ref))
            bb["rel_err_adj"] = float(np.linalg.norm(bxo.cpu().numpy()[cols] - x_ref) /
                                      np.linalg.norm(x_ref))
        log(f"[bench] bf16x3: fwd {bf_f:.4f} ms, adj {bf_a:.4f} ms, "
            f"{bb['speedup_vs_fp32']:.2f}x the FP32 step"
            + (f", rel err fwd {bb['rel_err_fwd']:.2e} adj {bb['rel_err_adj']:.2e}"
               if "rel_err_fwd" in bb else ""))
        out["bf16x3"] = bb
        bplan.close()
    else:
        plan.close()
    print(json.dumps(out), flush=True)
    return 0


def bench_gemm_reference(args):
    """The stacked mode-1 product Y^k_(1) = A_k B_k of one Z x with B
    materialised: per component, A_k (n1 x R_k, the stacked U1 factors) times
    B_k (R_k x n2 n3, every tensor's core applied in modes 2 and 3), R_k the
    plan's mean rows per component, complex64, as one batched library GEMM
    (rocBLAS through torch).  A reference point for the fused kernels, which
    never write B: its flops are the dominant term of theirs."""
    import numpy as np
    import torch
    import workloads
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import TuckerPlan

    wl = workloads.make(args.workload)
    plan = TuckerPlan.compress_dipoles(
        wl.grid.dims, wl.grid.h, wl.k0, lib.field_code(wl.basis, wl.operator),
        wl.pos, wl.ori, wl.tol, wl.rank_min, wl.rank_cap or 0)
    info = plan.info
    q, n1 = wl.q, wl.grid.n1
    ncols = wl.grid.n2 * wl.grid.n3
    R = int(round(info.sum_r1 / q))
    plan.close()
    g = torch.Generator(device="cuda").manual_seed(81)
    A = torch.randn((q, n1, R), dtype=torch.complex64, device="cuda", generator=g)
    B = torch.randn((q, R, ncols), dtype=torch.complex64, device="cuda", generator=g)
    C = torch.empty((q, n1, ncols), dtype=torch.complex64, device="cuda")
    for _ in range(args.warmup):
        torch.bmm(A, B, out=C)
    torch.cuda.synchronize()
    st = torch.cuda.current_stream()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(st)
    for _ in range(args.steps):
        torch.bmm(A, B, out=C)
    e1.record(st)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / args.steps
    flops = 8.0 * q * n1 * R * ncols
    tf = flops / (ms * 1e-3) / 1e12
    b_bytes = 8 * q * R * ncols
    log(f"[gemm] {q} x ({n1} x {R}) @ ({R} x {ncols}) complex64: {ms:.4f} ms, {tf:.1f} TFLOP/s "
        f"({100 * tf / PEAK_FP32_MFMA:.1f}% of FP32 peak), B {b_bytes / 1e6:.1f} MB")
    out = {
        "metric": "stacked mode-1 GEMM with B materialised (library complex GEMM)",
        "value": tf, "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "c64 (f32)", "data": "synthetic",
        "config": {"workload": f"{wl.name}: q={q} components of ({n1} x {R}) @ ({R} x {ncols})",
                   "b_bytes": b_bytes, "flops": flops},
        "frac_fp32_peak": tf / PEAK_FP32_MFMA,
    }
    print(json.dumps(out), flush=True)
    return 0


# Time of one y = Z_bc x with the ACA+HOSVD form on the paper's GPU (Table IX),
# seconds: context for the aca* workloads, not a target of the same metric.
PAPER_TABLE9_S = {("aca5", "pwc"): 1, ("aca5", "pwl"): 2, ("aca2", "pwc"): 2,
                  ("aca2", "pwl"): 6, ("aca1", "pwc"): 9, ("aca1", "pwl"): 33}


def bench_aca(args):
    """ACA+Tucker products (Sec. III.B substitution, Table III row
    ACA+Tucker) on the body-coil grids of Sec. IV.B.2: one step is one
    U (V^* x) and one V (U^* y).

    U has the paper's ACA rank r_c of columns; they stand in for Algorithm 3's
    columns with the point-current fields of r_c coil elements spread over
    the coil and shield, compressed on the GPU with Algorithm 3's HOSVD
    tolerance (3 x 1e-3) and ranks clamped to 15..18, the largest Tucker
    ranks of U reported in Sec. IV.B.2 (the point-current columns alone
    compress to ranks of 4..8).  V is m x r_c complex normal.  The products'
    cost depends on the grid, q, r_c, m and the ranks only.
    """
    import numpy as np
    import torch
    import workloads
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import AcaTuckerOperator, TuckerPlan

    prec = lib.TV_PREC_BF16X3 if args.precision == "bf16x3" else lib.TV_PREC_FP32
    wl = workloads.make_bodycoil(args.workload, args.basis)
    rc = workloads.aca_rank(args.workload)
    m = wl.m
    log(f"[aca] workload {wl.name} ({args.basis}): grid {wl.grid.dims}, q={wl.q}, "
        f"m={m}, r_c={rc}")
    pick = np.round(np.linspace(0, m - 1, rc)).astype(np.int64)
    rmin, rcap = (1, 0) if args.natural_ranks else (15, 18)
    t0 = time.perf_counter()
    plan = TuckerPlan.compress_dipoles(
        wl.grid.dims, wl.grid.h, wl.k0, lib.field_code(wl.basis, wl.operator),
        wl.pos[pick], wl.ori[pick], 3.0 * wl.tol, rmin, rcap, precision=prec)
    torch.cuda.synchronize()
    log(f"[aca] U compressed on GPU in {time.perf_counter() - t0:.2f} s")
    if not args.no_autotune:
        t0 = time.perf_counter()
        plan.autotune(2, args.tune_cache)
        torch.cuda.synchronize()
        log(f"[aca] autotuned in {time.perf_counter() - t0:.2f} s")
    info = plan.info
    V_np = workloads.complex_normal((m, rc), 63)
    op = AcaTuckerOperator(plan, torch.from_numpy(V_np.astype(np.complex64)).cuda())
    x_np = workloads.complex_normal(m, wl.seed_x)
    y_np = workloads.complex_normal(plan.rows, wl.seed_y)
    x = torch.from_numpy(x_np.astype(np.complex64)).cuda()
    y = torch.from_numpy(y_np.astype(np.complex64)).cuda()
    yo = torch.empty(plan.rows, dtype=torch.complex64, device="cuda")
    xo = torch.empty(m, dtype=torch.complex64, device="cuda")
    ws0, ws1 = op.workspace(0, 1), op.workspace(1, 1)
    st = torch.cuda.current_stream()
    sp = st.cuda_stream
    h, vp = plan.handle, op.Vc.data_ptr()

    def fwd():
        lib.tv_aca_matvec(h, vp, m, m, x.data_ptr(), m, 1, yo.data_ptr(),
                          plan.rows, ws0.data_ptr(), ws0.numel(), sp)

    def adj():
        lib.tv_aca_rmatvec(h, vp, m, m, y.data_ptr(), plan.rows, 1,
                           xo.data_ptr(), m, ws1.data_ptr(), ws1.numel(), sp)

    for _ in range(args.warmup):
        fwd()
        adj()
    torch.cuda.synchronize()
    K = args.steps
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(K)]
    start = torch.cuda.Event(enable_timing=True)
    end = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    start.record(st)
    for i in range(K):
        ev[i][0].record(st)
        fwd()
        ev[i][1].record(st)
        adj()
        ev[i][2].record(st)
    end.record(st)
    torch.cuda.synchronize()
    total_ms = start.elapsed_time(end)
    fwd_ms = sum(e[0].elapsed_time(e[1]) for e in ev) / K
    adj_ms = sum(e[1].elapsed_time(e[2]) for e in ev) / K
    fl_f = info.flops_matvec + 8.0 * m * rc
    fl_a = info.flops_rmatvec + 8.0 * m * rc
    tf_f = fl_f / (fwd_ms * 1e-3) / 1e12
    tf_a = fl_a / (adj_ms * 1e-3) / 1e12
    log(f"[aca] fwd {fwd_ms:.3f} ms ({tf_f:.1f} TFLOP/s), adj {adj_ms:.3f} ms "
        f"({tf_a:.1f} TFLOP/s)")
    dom = "adjoint" if adj_ms >= fwd_ms else "forward"
    d = 1 if dom == "adjoint" else 0
    info = plan.info
    kname = kernel_label(info.kernel[d], d)
    ach = tf_a if dom == "adjoint" else tf_f
    peak = mfma_peak(info.kernel[d], prec == lib.TV_PREC_FP32)
    mode1 = 8.0 * wl.grid.n1 * wl.grid.n2 * wl.grid.n3 * info.sum_r1
    out = {
        "metric": "ACA+Tucker coupling-matrix products/s (U (V^* x) and V (U^* y))",
        "value": 2.0 * K / (total_ms / 1e3), "unit": "matvecs/s", "n_gpus": 1,
        "steps": K, "warmup": args.warmup, "ms_per_step": total_ms / K,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32" if prec == lib.TV_PREC_FP32 else "bf16x3 (f32 accumulate)",
        "data": "synthetic",
        "config": {
            "workload": f"{wl.name} ({args.basis}): body-coil box "
                        f"{wl.grid.n1}x{wl.grid.n2}x{wl.grid.n3}, q={wl.q}, "
                        f"m={m} coil elements, r_c={rc} Tucker-compressed "
                        f"columns of U (HOSVD tol {3.0 * wl.tol:g}, ranks "
                        f"{'natural' if args.natural_ranks else 'clamped to 15..18'}), "
                        f"complex64",
            "grid": list(wl.grid.dims), "q": wl.q, "m": m, "r_c": rc,
            "mean_rank": [round(v, 3) for v in info.mean_rank],
            "max_rank": list(info.max_rank),
            "plan_factor_bytes": int(info.factor_bytes),
        },
        "fwd_ms": fwd_ms, "adj_ms": adj_ms, "tflops_fwd": tf_f, "tflops_adj": tf_a,
        "flops_fwd": fl_f, "flops_adj": fl_a,
        "paper_table9_s": PAPER_TABLE9_S.get((wl.name, args.basis)),
        "roofline": {"kernel": f"{kname} ({dom})", "bound": "mfma",
                     "achieved": ach, "peak": peak, "unit": "TFLOP/s",
                     "frac": ach / peak,
                     "traffic": None if args.natural_ranks else measured_traffic(
                         f"{wl.name}-{args.basis}", "fp32" if prec == lib.TV_PREC_FP32
                         else "bf16x3", dom, info)},
        "launch": {"tile_t2": list(info.tile_t2), "tile_t3": list(info.tile_t3),
                   "splits": list(info.splits)},
    }
    if not args.no_cpu:
        w_np = V_np.astype(np.complex64).astype(np.complex128).conj().T @ \
            x_np.astype(np.complex64).astype(np.complex128)
        t0 = time.perf_counter()
        V_np.conj().T @ x_np
        V_np @ w_np
        t_v = time.perf_counter() - t0
        cb, cols, y_ref, x_ref = cpu_baseline(wl, plan, w_np, y_np, args.cpu_budget)
        cb["value"] = 2.0 / (2.0 / cb["value"] + t_v)
        cb["sample"] += "; plus the two V products in full (numpy)"
        out["cpu_baseline"] = cb
        ws = np.zeros_like(w_np)
        ws[cols] = w_np[cols]
        ys = plan.matvec(torch.from_numpy(ws.astype(np.complex64)).cuda()).cpu().numpy()
        xa = plan.rmatvec(y).cpu().numpy()[cols]
        out["rel_err_fwd"] = float(np.linalg.norm(ys - y_ref) / np.linalg.norm(y_ref))
        out["rel_err_adj"] = float(np.linalg.norm(xa - x_ref) / np.linalg.norm(x_ref))
        log(f"[aca] oracle {cb['value']:.4f} products/s on {cb['cores']} threads; "
            f"rel err fwd {out['rel_err_fwd']:.2e} adj {out['rel_err_adj']:.2e}")
    plan.close()
    print(json.dumps(out), flush=True)
    return 0


# Assembly time of Algorithm 3 on the paper's GPU (Table VIII, "Algorithm 3-GPU"),
# seconds: context for --assemble.
PAPER_TABLE8_S = {("aca5", "pwc"): 206, ("aca5", "pwl"): 598, ("aca2", "pwc"): 1617,
                  ("aca2", "pwl"): 5333, ("aca1", "pwc"): 12936, ("aca1", "pwl"): 55241}


def bench_assemble(args):
    """Algorithm 3 (Tucker-based ACA assembly, Sec. III.C) on the body-coil
    stand-in: at most r_c steps (the paper's ACA rank), tolerance 1e-3,
    HOSVD 3e-3; the time is that of the steps run (the loop stops at the
    norm test or after r_c steps), each with a row and a column of Z, two
    products with the compressed U, the HOSVD of the new column and U's
    growth by that column."""
    import numpy as np
    import torch
    import workloads
    from paper_2103_06393_amd import lib

    wl = workloads.make_bodycoil(args.workload, args.basis)
    rc = workloads.aca_rank(args.workload)
    grid = lib.make_grid(*wl.grid.dims, wl.q, wl.m)
    st = torch.cuda.current_stream().cuda_stream
    torch.cuda.synchronize()
    log(f"[alg3] workload {wl.name} ({args.basis}): grid {wl.grid.dims}, q={wl.q}, "
        f"m={wl.m}, {rc} steps")
    t0 = time.perf_counter()
    ws = torch.empty(lib.tv_aca_assemble_workspace_bytes(grid, rc, wl.tol), dtype=torch.uint8,
                     device="cuda")
    h_plan, V, n, conv, piv, s = lib.tv_aca_assemble(
        grid, wl.grid.h, wl.k0, lib.field_code(wl.basis, wl.operator), wl.pos, wl.ori,
        wl.tol, 0.0, 1, 0, rc, lib.TV_PREC_FP32, st, ws.data_ptr(), ws.numel())
    torch.cuda.synchronize()
    sec = time.perf_counter() - t0
    info = lib.tv_plan_info(h_plan)
    log(f"[alg3] {n} terms in {sec:.2f} s ({1e3 * sec / max(n, 1):.1f} ms per step), "
        f"converged {conv}, mean ranks {[round(v, 2) for v in info.mean_rank]}, "
        f"U {info.factor_bytes / 2**20:.1f} MiB")
    lib.tv_plan_destroy(h_plan)
    out = {
        "metric": "Algorithm 3 (Tucker-based ACA assembly) time", "value": sec,
        "unit": "s", "n_gpus": 1, "steps": n, "warmup": 0,
        "ms_per_step": 1e3 * sec / max(n, 1), "higher_is_better": False,
        "scaling": "weak", "vs_baseline": None, "dtype": "f64 (f32 products with U)",
        "data": "synthetic",
        "config": {
            "workload": f"{wl.name} ({args.basis}): body-coil box "
                        f"{wl.grid.n1}x{wl.grid.n2}x{wl.grid.n3}, q={wl.q}, m={wl.m} coil "
                        f"elements, ACA tol {wl.tol:g}, HOSVD tol {3 * wl.tol:g}, {rc} steps",
            "grid": list(wl.grid.dims), "q": wl.q, "m": wl.m, "terms": n,
            "converged": conv, "mean_rank": [round(v, 3) for v in info.mean_rank],
            "max_rank": list(info.max_rank), "u_factor_bytes": int(info.factor_bytes),
        },
        "paper_table8_s": PAPER_TABLE8_S.get((wl.name, args.basis)),
    }
    print(json.dumps(out), flush=True)
    return 0


def batch_cpu_baseline(wls, plans, X, Y, Yo, Xo, p):
    """The FP64 oracle (Algorithms 1 and 2 with p right-hand sides) on the two
    coils with the fewest columns, on the GPU plans' own factors; also the
    GPU results' relative errors on those coils."""
    import numpy as np
    from threadpoolctl import threadpool_info
    from oracle import matvec as om
    from tests.plans import abi_to_struct
    order = np.argsort([w.m for w in wls])[:2]
    t = 0.0
    errs = {}
    for c in order:
        w, P = wls[c], plans[c]
        S = abi_to_struct(w.grid.dims, w.q, *P.export_factors())
        xc, yc = X[c].cpu().numpy(), Y[c].cpu().numpy()
        t0 = time.perf_counter()
        yr = om.alg1(S, xc, block_entries=1 << 28)
        xr = om.alg2(S, yc, block_entries=1 << 28)
        t += time.perf_counter() - t0
        ey = np.linalg.norm(Yo[c].cpu().numpy() - yr) / np.linalg.norm(yr)
        ex = np.linalg.norm(Xo[c].cpu().numpy() - xr) / np.linalg.norm(xr)
        errs[f"rel_err_coil{c}"] = [float(ey), float(ex)]
    threads = sum(int(i.get("num_threads", 1)) for i in threadpool_info()
                  if i.get("user_api") == "blas") or 1
    n = 2 * p * len(order)
    return {"value": n / t, "unit": "matvecs/s", "cores": threads, "kind": "oracle",
            "cpu_model": cpu_model(),
            "sample": f"the 2 coils with the fewest columns ({[wls[c].m for c in order]}), "
                      f"{p} right-hand sides, both directions, FP64 Algorithms 1 and 2 on the "
                      f"GPU plans' factors"}, errs


def bench_batch(args):
    """Batched path: 16 coils on a 96x128x112 grid, 32 right-hand sides
    each, one persistent launch per direction, captured into a graph."""
    import numpy as np
    import torch
    import workloads
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import TuckerPlan, batch_create
    wls = workloads.make_batch("c4")
    t0 = time.perf_counter()
    bf = args.precision == "bf16x3"
    prec = lib.TV_PREC_BF16X3 if bf else lib.TV_PREC_FP32
    plans = [TuckerPlan.compress_dipoles(w.grid.dims, w.grid.h, w.k0, 0, w.pos, w.ori,
                                         w.tol, w.rank_min, w.rank_cap, precision=prec)
             for w in wls]
    torch.cuda.synchronize()
    log(f"[bench] compressed {sum(w.m for w in wls)} columns in {time.perf_counter() - t0:.1f} s")
    p = 32
    X = [torch.from_numpy(w.x(p).astype(np.complex64)).cuda().t().contiguous().t() for w in wls]
    Y = [torch.from_numpy(w.y(p).astype(np.complex64)).cuda().t().contiguous().t() for w in wls]
    Yo = [torch.empty((p, P.rows), dtype=torch.complex64, device="cuda").t() for P in plans]
    Xo = [torch.empty((p, P.m), dtype=torch.complex64, device="cuda").t() for P in plans]
    hs = [P.handle for P in plans]
    t0 = time.perf_counter()
    cfg = [(0, 0), (0, 0)]
    if not args.no_autotune:
        st0 = torch.cuda.current_stream().cuda_stream
        cfg = [lib.tv_batch_autotune(hs, op, [p] * len(plans), args.tune_cache, st0)
               for op in (0, 1)]
        log(f"[bench] batch configurations (tsplit, workgroups per CU): forward {cfg[0]}, "
            f"adjoint {cfg[1]} (autotuned in {time.perf_counter() - t0:.1f} s)")
        t0 = time.perf_counter()
    bfwd, bfwd_arena = batch_create(hs, 0, [p] * len(plans), cfg[0])
    badj, badj_arena = batch_create(hs, 1, [p] * len(plans), cfg[1])
    log(f"[bench] batch objects (work queues, packed operands) built in "
        f"{time.perf_counter() - t0:.1f} s")
    wsf = torch.empty(lib.tv_batch_workspace_bytes(bfwd), dtype=torch.uint8, device="cuda")
    wsa = torch.empty(lib.tv_batch_workspace_bytes(badj), dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    fa = ([x.data_ptr() for x in X], [x.stride(1) for x in X], [y.data_ptr() for y in Yo],
          [y.stride(1) for y in Yo], wsf.data_ptr(), wsf.numel())
    aa = ([y.data_ptr() for y in Y], [y.stride(1) for y in Y], [x.data_ptr() for x in Xo],
          [x.stride(1) for x in Xo], wsa.data_ptr(), wsa.numel())
    g = torch.cuda.CUDAGraph()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    dir_ms = {}
    for name, bb, args_ in (("forward", bfwd, fa), ("adjoint", badj, aa)):
        with torch.cuda.stream(s):
            lib.tv_batch_run(bb, *args_, s.cuda_stream)       # first launch
            e0.record(s)
            for _ in range(2):
                lib.tv_batch_run(bb, *args_, s.cuda_stream)
            e1.record(s)
        torch.cuda.synchronize()
        dir_ms[name] = e0.elapsed_time(e1) / 2
        log(f"[bench] batched {name}: {dir_ms[name]:.1f} ms per launch")
    with torch.cuda.graph(g, stream=s):
        lib.tv_batch_run(bfwd, *fa, s.cuda_stream)
        lib.tv_batch_run(badj, *aa, s.cuda_stream)
    for _ in range(min(args.warmup, 2)):
        g.replay()
    torch.cuda.synchronize()
    log("[bench] graph captured and replayed")
    K = max(1, min(args.steps, 5))
    e0.record()
    for _ in range(K):
        g.replay()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / K
    # the same products one plan at a time through tv_matvec / tv_rmatvec
    # (fused single-vector kernels, p right-hand sides in sequence)
    Yp = [torch.empty_like(y) for y in Yo]
    Xp = [torch.empty_like(x) for x in Xo]
    def plain():
        for P, x, y, yo, xo in zip(plans, X, Y, Yp, Xp):
            P.matvec(x, out=yo)
            P.rmatvec(y, out=xo)
    plain()
    torch.cuda.synchronize()
    log("[bench] unbatched warm-up done")
    e0.record()
    plain()
    e1.record()
    torch.cuda.synchronize()
    ms_plain = e0.elapsed_time(e1)
    dev = max(float(torch.linalg.norm(a - b) / torch.linalg.norm(b))
              for a, b in zip(Yo + Xo, Yp + Xp))
    nmv = 2 * p * len(plans)
    fl = 0.0
    for P in plans:
        r = np.array(P.export_factors()[0], dtype=np.float64)
        n1, n2, n3 = P.dims
        nv = n1 * n2 * n3
        dec = r[:, 0] * r[:, 1] * r[:, 2] * n2 + r[:, 0] * r[:, 2] * n2 * n3 + r[:, 0] * nv
        fl += 2 * float(np.sum(8.0 * (dec + nv * p)))   # both directions
    # Table III's p-vector count per direction: decompression once per tensor
    # plus the application to the p right-hand sides
    fl_dir = fl / 2
    dom = max(dir_ms, key=dir_ms.get)
    peak = PEAK_BF16_MFMA / 3.0 if bf else PEAK_FP32_MFMA
    ach = fl_dir / (dir_ms[dom] * 1e-3) / 1e12
    log(f"[bench] batched {ms:.2f} ms per step ({nmv} products), one plan and vector at a time "
        f"{ms_plain:.2f} ms; max relative difference {dev:.2e}")
    out = {"metric": "compressed VSIE matvecs/s (Zx and Z^H y), batched",
           "value": nmv / (ms * 1e-3), "unit": "matvecs/s", "n_gpus": 1, "steps": K,
           "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None,
           "dtype": "bf16x3 apply (f32 decompression and accumulation)" if bf
           else "f32", "data": "synthetic",
           "config": {"workload": "c4: 16 coils (64..1024 point currents) on 96x128x112, "
                                  "32 right-hand sides each, graph replay of both directions"},
           "tflops": fl / (ms * 1e-3) / 1e12,
           "forward_ms": dir_ms["forward"], "adjoint_ms": dir_ms["adjoint"],
           "roofline": {"kernel": f"tv_batch_run ({dom}: mode-3 kernel + persistent batched "
                                  f"kernel{' + reduction' if dom == 'adjoint' else ''})",
                        "bound": "mfma", "achieved": ach, "peak": peak, "unit": "TFLOP/s",
                        "frac": ach / peak, "traffic": None},
           "launch": {"forward": list(cfg[0]), "adjoint": list(cfg[1]),
                      "fields": "tsplit, workgroups per CU"},
           "unbatched_ms_per_step": ms_plain, "batched_speedup": ms_plain / ms,
           "max_rel_diff_vs_unbatched": dev,
           "workspace_bytes": {"forward": int(wsf.numel()), "adjoint": int(wsa.numel())}}
    if not args.no_cpu:
        out["cpu_baseline"], errs = batch_cpu_baseline(wls, plans, X, Y, Yo, Xo, p)
        out.update(errs)
    lib.tv_batch_destroy(bfwd)
    lib.tv_batch_destroy(badj)
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
