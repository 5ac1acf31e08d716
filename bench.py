"""Benchmark: emulated FP64 DGEMM by FP8 Ozaki-II on one MI355X.

Default workload: m = n = k = 8192, column-major 'N','N', entries
(U[0,1) - 0.5) exp(0.5 N(0,1)) from a seeded PCG64, alpha = 1, beta = 0,
12 moduli (the paper's full-accuracy count), accurate mode (--mode fast for
the Cauchy-Schwarz scaling, with --moduli 13 as in the paper).  Inputs are
resident in HBM before the timed region.  One step = one ozaki2_dgemm call
(every stage of the path).  Prints one JSON line.

Beside the emulated rate it reports: the native FP64 DGEMM (torch.matmul on
float64, i.e. the vendor BLAS) on the same inputs, the normalised error of
both against a double-double reference on sampled rows, the residue-product
kernel against the MFMA roofline of the format its digits are in (timed with HIP
events on the library's stream), and the CPU oracle on a bounded sample of the
same workload.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "emulated FP64 TFLOP/s vs native FP64 DGEMM at ≤1e-15 err; FP8 MFMA util %"
# MI355X dense MFMA peaks, TFLOP/s (TOP/s), of the formats the residue products
# read: the digits (integers of magnitude <= 16, exact in either) of the FP8 lists
# are E2M3 in batches and with more than four 256 x 256 output tiles, E4M3 in
# smaller calls; the INT8 list's residues are INT8.
PEAK_TFLOPS = {"e2m3": 10000.0, "e4m3": 5000.0, "int8": 5000.0}
DTYPE = {"e2m3": "fp6e2m3-mfma (exact integer digits)->f64", "e4m3": "fp8e4m3-mfma->f64",
         "int8": "int8-mfma->f64"}
HBM_PEAK_GBS = 8000.0


def digit_format(moduli_list: str, m: int, n: int) -> str:
    """Format of the residue products' operands for an m x n output."""
    if moduli_list == "int8":
        return "int8"
    return "e2m3" if -(-m // 256) * -(-n // 256) > 4 else "e4m3"


def _parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=30)
    ap.add_argument("--size", type=int, default=8192, help="m = n = k")
    ap.add_argument("--m", type=int, default=None)
    ap.add_argument("--n", type=int, default=None)
    ap.add_argument("--k", type=int, default=None)
    ap.add_argument("--moduli", type=int, default=12)
    ap.add_argument("--phi", type=float, default=None,
                    help="spread of the entries (default 0.5; 1 for the batched workload)")
    ap.add_argument("--mode", choices=["accurate", "fast"], default="accurate",
                    help="scaling mode (fast: Cauchy-Schwarz bound, no bound product)")
    ap.add_argument("--moduli-list", choices=["hybrid", "karatsuba", "int8"], default="hybrid",
                    help="modulus list (karatsuba: the Karatsuba-only ablation, N = 13; "
                         "int8: the INT8 arm of Section II, N = 14-16)")
    ap.add_argument("--transA", choices=["N", "T"], default="N",
                    help="storage of op(A): N (m x k, lda = m) or T (k x m, lda = k)")
    ap.add_argument("--transB", choices=["N", "T"], default="N",
                    help="storage of op(B): N (k x n, ldb = k) or T (n x k, ldb = n)")
    ap.add_argument("--cancel", action="store_true",
                    help="rows 0..255 of op(A) orthogonal to columns 0..255 of op(B) up to "
                         "a 1e-8 perturbation (the large stress workload's block)")
    ap.add_argument("--config", type=int, default=2,
                    help="seed group of the inputs (the numbered workloads: 2 square, "
                         "3 rectangular, 5 large stress)")
    ap.add_argument("--workload", choices=["single", "batched"], default="single",
                    help="batched: 512 problems with m, n, k log-uniform in [64, 4096], "
                         "one batched call (graph replay, autotuned) against looped "
                         "single calls and looped native FP64 DGEMM")
    ap.add_argument("--count", type=int, default=512, help="problems of the batched workload")
    ap.add_argument("--vendor-fp8", action="store_true",
                    help="also time the vendor FP8 GEMM (torch._scaled_mm, E4M3 operands of "
                         "the same m x n x k, FP32 output) for context")
    ap.add_argument("--cpu-rows", type=int, default=48,
                    help="rows of op(A) in the CPU oracle sample")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-native", action="store_true")
    ap.add_argument("--traffic", type=str,
                    default=os.path.join(ROOT, "profiles", "residue_gemm_8192_n12_traffic.json"),
                    help="JSON file with measured HBM bytes per residue-product call (used "
                         "only for the workload it was measured on and while the GEMM "
                         "source is unchanged)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="before the timed steps, run a plain device copy of 1 GiB "
                         "(torch copy_) three times, as the reference kernel for "
                         "scaling hardware byte counters")
    args = ap.parse_args()
    if args.phi is None:
        args.phi = 1.0 if args.workload == "batched" else 0.5
    return args


def _cpu_baseline(A, B, N, rows, mode, moduli_list):
    """The oracle, as it stands, on op(A)[:rows] x op(B): a bounded slab of the
    same workload (its own emulated GEMM of shape rows x n x k)."""
    import numpy as np
    from oracle import ozaki2_ref as ref
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:  # noqa: BLE001
        threads = os.cpu_count() or 1
    Asub = np.ascontiguousarray(A[:rows])
    t0 = time.perf_counter()
    ref.emulate(Asub, B, N, mode=mode, moduli_set=moduli_list)
    dt = time.perf_counter() - t0
    m, k = Asub.shape
    n = B.shape[1]
    return {"value": 2.0 * m * n * k / dt / 1e12, "unit": "TFLOP/s", "cores": int(threads),
            "kind": "oracle",
            "sample": f"oracle emulate() on op(A)[:{rows}] x op(B) ({m}x{n}x{k}, "
                      f"N={N}, {mode} mode, {moduli_list} moduli), {dt:.1f} s wall"}


def _bench_batched(args):
    """The batched workload: `count` problems with m, n, k drawn log-uniformly
    from [64, 4096] (entries (U - 1/2) exp(phi N(0,1)) drawn on the GPU from a
    seeded generator, column-major NN), all emulated by ONE
    ozaki2_dgemm_batched call.  The first call autotunes the residue-product
    configuration; the timed steps replay the call's captured graph.  Beside
    it: the same problems as looped ozaki2_dgemm calls and as looped native
    FP64 DGEMMs (torch.matmul), and one eager timed pass for the kernel
    breakdown (the persistent residue-product launch against its MFMA peak)."""
    import numpy as np
    import torch

    import paper_2603_10634_amd as oz
    from workloads import batch_shapes, config_seed

    N = args.moduli
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    seed = config_seed(4, 0)
    shapes = batch_shapes(args.count, 64, 4096, seed)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    f64 = torch.float64
    tA, tB, tC = [], [], []
    for (m, n, k) in shapes:
        tA.append((torch.rand((k, m), generator=g, device=dev, dtype=f64) - 0.5) *
                  torch.exp(args.phi * torch.randn((k, m), generator=g, device=dev, dtype=f64)))
        tB.append((torch.rand((n, k), generator=g, device=dev, dtype=f64) - 0.5) *
                  torch.exp(args.phi * torch.randn((n, k), generator=g, device=dev, dtype=f64)))
        tC.append(torch.empty((n, m), dtype=f64, device=dev))
    cnt = len(shapes)
    ms = [s[0] for s in shapes]
    ns = [s[1] for s in shapes]
    ks = [s[2] for s in shapes]
    flops = float(sum(2.0 * m * n * k for m, n, k in shapes))

    stream = torch.cuda.current_stream(dev)
    oz.ozaki2_set_stream(stream)
    if oz.ozaki2_set_mode(args.mode) != 0 or oz.ozaki2_set_moduli_list(args.moduli_list) != 0:
        raise RuntimeError("invalid mode or moduli list")
    wbytes = oz.ozaki2_workspace_bytes_batched(ms, ns, ks, N)
    ws = torch.empty(wbytes + 256, dtype=torch.uint8, device=dev)
    oz.ozaki2_set_workspace((ws.data_ptr() + 255) // 256 * 256, wbytes)

    def batched():
        st = oz.ozaki2_dgemm_batched(["N"] * cnt, ["N"] * cnt, ms, ns, ks, [1.0] * cnt, tA, ms,
                                     tB, ks, [0.0] * cnt, tC, ms, N)
        if st != 0:
            raise oz.Ozaki2Error("ozaki2_dgemm_batched", st)

    def looped():
        for q in range(cnt):
            st = oz.ozaki2_dgemm("N", "N", ms[q], ns[q], ks[q], 1.0, tA[q], ms[q], tB[q], ks[q],
                                 0.0, tC[q], ms[q], N)
            if st != 0:
                raise oz.Ozaki2Error("ozaki2_dgemm", st)

    def timed(fn, steps):
        torch.cuda.synchronize(dev)
        t0 = time.perf_counter()
        for _ in range(steps):
            fn()
        torch.cuda.synchronize(dev)
        return (time.perf_counter() - t0) / steps * 1e3

    oz.ozaki2_set_autotune(True)
    batched()                                    # tunes the configuration, then runs
    torch.cuda.synchronize(dev)
    config = oz.ozaki2_get_schedule()
    oz.ozaki2_set_graph(True)
    for _ in range(args.warmup):
        batched()
    ms_batched = timed(batched, args.steps)      # graph replays
    oz.ozaki2_set_graph(False)
    # eager pass with the library's HIP events (one sub-batch: the caller
    # workspace holds the whole batch)
    oz.ozaki2_set_timing(True)
    kt = []
    for _ in range(max(3, args.steps // 3)):
        batched()
        kt.append(oz.ozaki2_get_kernel_times())
    oz.ozaki2_set_timing(False)
    k_mean = np.array(kt).mean(axis=0)
    for _ in range(max(2, args.warmup // 10)):
        looped()
    ms_looped = timed(looped, max(3, args.steps // 3))
    native = None
    if not args.no_native:
        nat = lambda: [torch.matmul(tA[q].T, tB[q].T) for q in range(cnt)]
        for _ in range(max(2, args.warmup // 10)):
            nat()
        ms_native = timed(nat, max(3, args.steps // 3))
        native = {"tflops": round(flops / (ms_native * 1e-3) / 1e12, 2),
                  "ms": round(ms_native, 3), "impl": "looped torch.matmul float64 (vendor BLAS)"}
    oz.ozaki2_set_autotune(False)
    oz.ozaki2_set_workspace(None, 0)
    value = flops / (ms_batched * 1e-3) / 1e12
    products = N if args.moduli_list == "int8" else 3 * N
    gemm_ms = float(k_mean[4])
    achieved = products * flops / (gemm_ms * 1e-3) / 1e12
    fmt = "int8" if args.moduli_list == "int8" else "e2m3"
    peak = PEAK_TFLOPS[fmt]
    out = {
        "metric": METRIC,
        "value": round(value, 3),
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_batched, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": DTYPE[fmt],
        "data": "synthetic",
        "config": {"workload": f"batched: {cnt} emulated dgemms, m, n, k log-uniform in "
                               f"[64, 4096], col-major NN, phi={args.phi}, {N} "
                               f"{args.moduli_list} moduli, {args.mode} mode; one "
                               "ozaki2_dgemm_batched call replayed from its graph",
                   "count": cnt, "sum_2mnk": flops, "num_moduli": N, "phi": args.phi,
                   "mode": args.mode, "moduli_list": args.moduli_list},
        "autotuned_config": config,
        "looped_single_calls": {"tflops": round(flops / (ms_looped * 1e-3) / 1e12, 3),
                                "ms": round(ms_looped, 3)},
        "native_fp64": native,
        "speedup_vs_looped_single": round(ms_looped / ms_batched, 3),
        "speedup_vs_native": (round(value / native["tflops"], 3) if native else None),
        "kernel_ms_mean_eager": [round(float(x), 4) for x in k_mean],
        "roofline": {"bound": "mfma", "achieved": round(achieved, 1), "peak": peak,
                     "unit": "TFLOP/s", "frac": round(achieved / peak, 4),
                     "traffic": None,
                     "kernel": f"k_residue6 (one launch: {products} {fmt} products per "
                               "problem, all problems; algorithmic flops on the unpadded "
                               "shapes)"},
        "cpu_baseline": None,
    }
    print(json.dumps(out), flush=True)


def main():
    args = _parse()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}): the library emulates "
              "each GEMM on one device and has no multi-GPU sharding.", file=sys.stderr)
        sys.exit(2)
    if args.workload == "batched":
        _bench_batched(args)
        return
    import numpy as np
    import torch

    import paper_2603_10634_amd as oz
    from workloads import cancellation_block, phi_matrix, phi_seed
    from workloads.reference import dd_dot_rows, normalised_error

    m = args.m or args.size
    n = args.n or args.size
    k = args.k or args.size
    N = args.moduli
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)

    seed = phi_seed(args.config, args.phi)
    A = phi_matrix(m, k, args.phi, seed)          # op(A), m x k
    B = phi_matrix(k, n, args.phi, seed + 1)      # op(B), k x n
    if args.cancel:
        A = cancellation_block(A, B, min(256, m), min(256, n), 1e-8, seed + 2)
    # column-major storage: 'N' stores op(A) (m x k, lda = m), which is A.T in
    # C order; 'T' stores A^T (k x m, lda = k), which is A in C order
    tA = torch.from_numpy(np.ascontiguousarray(A.T if args.transA == "N" else A)).to(dev)
    tB = torch.from_numpy(np.ascontiguousarray(B.T if args.transB == "N" else B)).to(dev)
    lda = m if args.transA == "N" else k
    ldb = k if args.transB == "N" else n
    tC = torch.empty((n, m), dtype=torch.float64, device=dev)

    stream = torch.cuda.current_stream(dev)
    oz.ozaki2_set_stream(stream)
    if oz.ozaki2_set_mode(args.mode) != 0:
        raise RuntimeError("ozaki2_set_mode failed")
    if oz.ozaki2_set_moduli_list(args.moduli_list) != 0:
        raise RuntimeError("ozaki2_set_moduli_list failed")
    # caller-owned workspace (so the fix-up count can be read back afterwards)
    wbytes = oz.ozaki2_workspace_bytes(m, n, k, N)
    ws = torch.empty(wbytes + 256, dtype=torch.uint8, device=dev)
    ws_base = (ws.data_ptr() + 255) // 256 * 256
    oz.ozaki2_set_workspace(ws_base, wbytes)
    offs, _ = oz.ozaki2_workspace_layout(m, n, k, N)

    def call():
        st = oz.ozaki2_dgemm(args.transA, args.transB, m, n, k, 1.0, tA, lda, tB, ldb, 0.0, tC,
                             m, N)
        if st != 0:
            raise oz.Ozaki2Error("ozaki2_dgemm", st)

    for _ in range(args.warmup):
        call()
    torch.cuda.synchronize(dev)
    if args.copy_calibration:
        src = torch.empty(1 << 27, dtype=torch.float64, device=dev).fill_(1.0)   # 1 GiB
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize(dev)
        del src, dst

    # timed region: K calls; the library records HIP events between its kernel
    # groups on `stream`, read back after each call
    oz.ozaki2_set_timing(True)
    ktimes = []
    torch.cuda.synchronize(dev)
    t0 = time.perf_counter()
    for _ in range(args.steps):
        call()
        ktimes.append(oz.ozaki2_get_kernel_times())
    torch.cuda.synchronize(dev)
    wall = time.perf_counter() - t0
    oz.ozaki2_set_timing(False)
    o = ws_base - ws.data_ptr() + offs[10]
    fixups = int(ws[o:o + 4].cpu().numpy().view(np.uint32)[0])
    ms_per_step = wall / args.steps * 1e3
    flops = 2.0 * m * n * k
    value = flops / (ms_per_step * 1e-3) / 1e12
    kt = np.array(ktimes)                        # steps x 6
    k_mean = kt.mean(axis=0)
    k_med = np.median(kt, axis=0)
    step_med_ms = float(np.median(kt.sum(axis=1)))

    # residue products (FP8 lists: three digit products per modulus; INT8 arm: one)
    # against the MFMA peak of their operands' format
    gemm_ms = float(k_mean[4])
    fmt = digit_format(args.moduli_list, m, n)
    peak = PEAK_TFLOPS[fmt]
    products = N if args.moduli_list == "int8" else 3 * N
    res_flops = products * flops
    achieved = res_flops / (gemm_ms * 1e-3) / 1e12
    traffic = None
    if (args.traffic and os.path.exists(args.traffic) and (m, n, k, N) == (8192, 8192, 8192, 12)
            and args.moduli_list == "hybrid"):
        from paper_2603_10634_amd.profile_summary import gemm_source_sha
        with open(args.traffic) as f:
            rec = json.load(f)
        if rec.get("gemm_source_sha256") == gemm_source_sha():
            traffic = rec.get("bytes_per_call")
    kernel = "k_residue6" if -(-m // 256) * -(-n // 256) > 4 else "k_residue_small / _gemm"
    roofline = {"bound": "mfma", "achieved": round(achieved, 1), "peak": peak,
                "unit": "TFLOP/s", "frac": round(achieved / peak, 4),
                "traffic": traffic,
                "kernel": f"{kernel}, {products} {fmt} products of {m}x{n}x{k} per call"}

    # accuracy against a double-double reference on sampled rows
    Cemu = tC.cpu().numpy().T                    # m x n
    rows = np.array([0, m // 3, m - 1])
    cols = np.arange(min(n, 2048))
    hi, lo = dd_dot_rows(A[rows], B[:, cols])
    absA = np.abs(A[rows])
    absB = np.abs(B[:, cols])
    err_emu = normalised_error(Cemu[np.ix_(rows, cols)], hi, lo, absA, absB)

    native = None
    if not args.no_native:
        tAr = torch.from_numpy(A).to(dev)
        tBr = torch.from_numpy(B).to(dev)
        for _ in range(max(3, args.warmup // 3)):
            Cn = torch.matmul(tAr, tBr)
        torch.cuda.synchronize(dev)
        t0 = time.perf_counter()
        for _ in range(args.steps):
            Cn = torch.matmul(tAr, tBr)
        torch.cuda.synchronize(dev)
        nat_ms = (time.perf_counter() - t0) / args.steps * 1e3
        Cn_h = Cn.cpu().numpy()
        err_nat = normalised_error(Cn_h[np.ix_(rows, cols)], hi, lo, absA, absB)
        native = {"tflops": round(flops / (nat_ms * 1e-3) / 1e12, 2), "ms": round(nat_ms, 3),
                  "error_normalised": err_nat, "impl": "torch.matmul float64 (vendor BLAS)"}
        del tAr, tBr, Cn

    vendor = None
    if args.vendor_fp8:
        # the vendor FP8 GEMM on operands of the same shape, for context: the
        # residue products run 3N such products (per the roofline above)
        fa = (torch.randn((m, k), device=dev) * 4).to(torch.float8_e4m3fn)
        fb = (torch.randn((n, k), device=dev) * 4).to(torch.float8_e4m3fn).T
        one = torch.ones((), device=dev, dtype=torch.float32)
        for _ in range(5):
            torch._scaled_mm(fa, fb, scale_a=one, scale_b=one, out_dtype=torch.float32)
        torch.cuda.synchronize(dev)
        t0 = time.perf_counter()
        reps = max(10, args.steps)
        for _ in range(reps):
            torch._scaled_mm(fa, fb, scale_a=one, scale_b=one, out_dtype=torch.float32)
        torch.cuda.synchronize(dev)
        v_ms = (time.perf_counter() - t0) / reps * 1e3
        vendor = {"tflops": round(flops / (v_ms * 1e-3) / 1e12, 1), "ms": round(v_ms, 4),
                  "impl": "torch._scaled_mm E4M3 x E4M3 -> FP32 (hipBLASLt)"}
        del fa, fb

    cpu = None
    if not args.no_cpu_baseline:
        cpu = _cpu_baseline(A, B, N, min(args.cpu_rows, m), args.mode, args.moduli_list)

    stage = dict(zip(["quant", "gemms", "requant", "dequant", "others"],
                     [float(k_med[0] + k_med[3]), float(k_med[1] + k_med[4]), 0.0,
                      float(k_med[5]), float(k_med[2])]))
    out = {
        "metric": METRIC,
        "value": round(value, 3),
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": DTYPE[fmt],
        "data": "synthetic",
        "config": {"workload": f"emulated dgemm {m}x{n}x{k} col-major "
                               f"{args.transA}{args.transB}, phi={args.phi}"
                               f"{' with cancellation block' if args.cancel else ''}, "
                               f"{N} {args.moduli_list} moduli, {args.mode} mode",
                   "m": m, "n": n, "k": k, "transA": args.transA, "transB": args.transB,
                   "num_moduli": N, "phi": args.phi, "cancel": args.cancel,
                   "mode": args.mode, "moduli_list": args.moduli_list,
                   "alpha": 1.0, "beta": 0.0},
        "error_normalised": err_emu,
        "native_fp64": native,
        "vendor_fp8_gemm": vendor,
        "speedup_vs_native": (round(value / native["tflops"], 3) if native else None),
        "mfma_util_pct": round(100 * achieved / peak, 2),
        "stage_ms_median": {kk: round(v, 4) for kk, v in stage.items()},
        "scale_fixup_lines": fixups,
        "workspace_bytes": wbytes,
        "kernel_ms_mean": [round(float(x), 4) for x in k_mean],
        "step_ms_median_events": round(step_med_ms, 4),
        "roofline": roofline,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
