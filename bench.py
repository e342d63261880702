#!/usr/bin/env python3
"""Benchmark of the CSR SPMM / SDDMM / FusedMM hot path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload large16k] [--no-cpu-baseline]

One step = spmm_csr + sddmm_csr + fusedmm_csr (whatever row analysis and combine passes
they contain) on one synthetic workload whose operands are already in HBM.  The default
workload is the 16384 x 16384, 20 %-dense configuration the benchmark spec's target is quoted on
(SPMM N=512; SDDMM D=64; FusedMM D=64, N=512).  Prints ONE JSON line:

  value        GFLOP/s of the whole step, flops = 2*nnz*N (SPMM) + 2*nnz*D (SDDMM)
               + 2*nnz*(D+N) (FusedMM)
  ops          per operation, from one HIP-event pair around all kernels of a call: GFLOP/s (mean, median, best), the
               fractions of the published FP32 peak and HBM bandwidth (algorithmic bytes, and the bytes counted by
               rocprofv3 in a recorded run of the same kernels: hbm_counter_*) and of the machine
               rates measured in this run (frac_*_measured), one cold run (caches flushed by writing a 1 GiB buffer) and
               the wall time of the very first call (workspace allocation included).  `kernels` says whether the matrix-core
               kernels or the vector kernels ran: of the first the rate of the 16-bit products that they work through
               (six bfloat16 ones for an FP32 one, or three half-precision ones by C where ranges of K are long, over every
               cell of S) and its share of the published peak, of the second the rate at
               which gathered dense rows reach the ALUs (nnz * width * 4 bytes / time)
  measured_peaks  the library's micro-benchmarks (csrk_microbench), run in this process before the timed region:
               device copy (GB/s), independent FP32 multiply-adds acc += x * y without packed FP32 (TFLOP/s), and
               conflict-free 128-bit LDS reads with 16 wavefronts per CU (TB/s)
  roofline     the dominant operation against what bounds its kernels: the matrix cores' published bfloat16 peak (2.5
               PFLOP/s dense), or for vector kernels the FP32 vector peak (157.3 TFLOP/s); `traffic` and
               `traffic_source`: HBM bytes per call from a recorded rocprofv3 --pmc run (profiles/), since
               counters cannot be read from inside the process; `frac_of_lds_ceiling` (vector kernels): against the rate
               the measured LDS read bandwidth allows (one 4-byte LDS operand per multiply-add)
  phases       where the wavefronts of the 512-column LDS-tiled kernels spend their cycles, for operations that these do
               (csrk_tile_phases: the measuring build of the same kernel, shares of the summed phase counters)
  sddmm_at_scale  SDDMM at the benchmark size with D = 64 and D = 128
  cpu_baseline the FP64 CPU oracle timed on a sample of the rows of the same workload
  planned      the same three calls through a plan (pattern analysed once, outside the timing), timed after
               the main region and not part of `value`

Only one GPU is used; --gpus N with N > 1 is refused.
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

BF16_MATRIX_PEAK_TFLOPS = 2500.0  # MI355X, published, dense
PRODUCTS = 6                      # bfloat16 products that the matrix-core kernels make of an FP32 one (by C: the library says)
FP32_VECTOR_PEAK_TFLOPS = 157.3   # MI355X, published: 256 CUs x 2.4 GHz x 256 flop/clk/CU
HBM_PEAK_GBS = 8000.0             # MI355X, published
# The rates this build's instruction mix can reach (plain multiply-adds, since packed FP32 is switched off; 128-bit LDS
# reads with 16 wavefronts per CU; a device copy) are MEASURED in the same run by the library's micro-benchmarks
# (binding.csrk_microbench) and reported as `measured_peaks`; the frac_*_measured fields divide by them.

KIND = {1: "spmm", 2: "sddmm", 3: "fusedmm"}


def hbm_traffic_from_profiles(workload: str, kernel_key: str):
    """HBM bytes per call of an operation as measured by rocprofv3 --pmc (FETCH_SIZE / WRITE_SIZE, scaled
    by a copy kernel) in a RECORDED run: counters cannot be read from inside this process, so the figure comes from
    the committed summary profiles/hbm_traffic_<workload>.json.  Returns (bytes or None, where it came from)."""
    path = os.path.join(ROOT, "profiles", f"hbm_traffic_{workload}.json")
    try:
        with open(path) as f:
            rec = json.load(f)
        return rec.get(kernel_key), f"recorded rocprofv3 --pmc run, profiles/hbm_traffic_{workload}.json (not measured in this run)"
    except (OSError, ValueError):
        return None, "none recorded for this workload"


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)     # the paper times 20 back-to-back runs
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="large16k")
    ap.add_argument("--scale", type=float, default=1.0, help="shrink M,K (debug only; invalid as a result)")
    ap.add_argument("--shape", default="", help="with --workload custom: M,K,density,N,D (e.g. 8192,8192,0.3,128,128)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-rows", type=int, default=0, help="rows in the oracle's timed sample (0 = auto)")
    ap.add_argument("--no-fusion-report", action="store_true")
    ap.add_argument("--no-plan", dest="plan", action="store_false",
                    help="skip the `planned` object (the same calls with the pattern analysed once by "
                         "csrk_plan_create, then *_csr_plan; timed after the main region, not part of `value`)")
    ap.add_argument("--plan", dest="plan", action="store_true", help="(default) include the `planned` object")
    ap.set_defaults(plan=True)
    ap.add_argument("--bf16", action="store_true",
                    help="also time the bfloat16-operand entry points on the same workload, beside the FP32 general "
                         "path (adds a `bf16_operands` object to the line)")
    ap.add_argument("--no-microbench", action="store_true",
                    help="skip the library's machine-rate micro-benchmarks (`measured_peaks` and the frac_*_measured fields)")
    ap.add_argument("--no-phases", action="store_true",
                    help="skip the `phases` object (one run of the measuring builds of the 512-column tiled kernels)")
    ap.add_argument("--no-sddmm-at-scale", action="store_true",
                    help="skip the `sddmm_at_scale` object (SDDMM alone on this pattern with D = 64 and D = 128)")
    ap.add_argument("--copy-probe-mib", type=int, default=0,
                    help="also run one plain device-to-device copy of this many MiB before the timed region: "
                         "the known-size kernel that rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE readings are scaled by")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on exactly one GPU; --gpus N with N > 1 is not supported "
              "(row-sharding across GPUs is a design note only, not built).", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from paper_2311_00368_amd import binding, inputs

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the HIP path has no CPU fallback.", file=sys.stderr)
        sys.exit(3)
    binding.load(build_if_missing=False)
    torch.cuda.set_device(0)

    t_gen = time.time()
    if args.workload == "custom":
        m_, k_, p_, n_, d_ = args.shape.split(",")
        w = inputs.custom_workload(int(m_), int(k_), float(p_), int(n_), int(d_))
    else:
        w = inputs.workload(args.workload, scale=args.scale)
    t_gen = time.time() - t_gen
    nnz = w.nnz
    dev = lambda a: torch.from_numpy(a).cuda()
    rp, ci, v = dev(w.rowptr), dev(w.colidx), dev(w.vals)
    ops = []
    flops = {}
    if "spmm" in w.ops:
        o = w.ops["spmm"]
        N = o["N"]
        B, O = dev(o["B"]), torch.empty((w.M, N), dtype=torch.float32, device="cuda")
        ops.append(("spmm", lambda: binding.spmm_csr(w.M, w.K, N, rp, ci, v, B, O)))
        flops["spmm"] = 2.0 * nnz * N
    if "sddmm" in w.ops:
        o = w.ops["sddmm"]
        Ds = o["D"]
        As, Bs, P = dev(o["A"]), dev(o["B"]), torch.empty((nnz,), dtype=torch.float32, device="cuda")
        ops.append(("sddmm", lambda: binding.sddmm_csr(w.M, w.K, Ds, rp, ci, v, As, Bs, P)))
        flops["sddmm"] = 2.0 * nnz * Ds
    if "fusedmm" in w.ops:
        o = w.ops["fusedmm"]
        Df, Nf = o["D"], o["N"]
        Af, Bf, Cf = dev(o["A"]), dev(o["B"]), dev(o["C"])
        Of = torch.empty((w.M, Nf), dtype=torch.float32, device="cuda")
        ops.append(("fusedmm", lambda: binding.fusedmm_csr(w.M, w.K, Df, Nf, rp, ci, v, Af, Bf, Cf, Of)))
        flops["fusedmm"] = 2.0 * nnz * (Df + Nf)
    step_flops = sum(flops.values())
    # algorithmic HBM bytes per call: S streamed once, every dense operand once, the output once
    csr_bytes = 8.0 * nnz + 4.0 * (w.M + 1)
    hbm_bytes, gather_bytes = {}, {}
    if "spmm" in w.ops:
        n_ = w.ops["spmm"]["N"]
        hbm_bytes["spmm"] = csr_bytes + 4.0 * n_ * (w.K + w.M)
        gather_bytes["spmm"] = 4.0 * nnz * n_
    if "sddmm" in w.ops:
        d_ = w.ops["sddmm"]["D"]
        hbm_bytes["sddmm"] = csr_bytes + 4.0 * nnz + 4.0 * d_ * (w.K + w.M)
        gather_bytes["sddmm"] = 4.0 * nnz * d_
    if "fusedmm" in w.ops:
        d_, n_ = w.ops["fusedmm"]["D"], w.ops["fusedmm"]["N"]
        hbm_bytes["fusedmm"] = csr_bytes + 4.0 * d_ * (w.K + w.M) + 4.0 * n_ * (w.K + w.M)
        gather_bytes["fusedmm"] = 4.0 * nnz * (d_ + n_)

    def step():
        for _, fn in ops:
            fn()

    if args.copy_probe_mib:
        src = torch.ones(args.copy_probe_mib << 18, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    peaks = None
    if not args.no_microbench:
        peaks = {"hbm_copy_GBps": round(binding.csrk_microbench(binding.CSRK_BENCH_HBM_COPY), 1),
                 "fma_f32_TFLOPs": round(binding.csrk_microbench(binding.CSRK_BENCH_FMA_F32), 2),
                 "lds_read_b128_TBps": round(binding.csrk_microbench(binding.CSRK_BENCH_LDS_READ), 2),
                 "note": "measured in this run by the library's own kernels: 1 GiB device copy (read + written "
                         "bytes), independent plain v_fma_f32 (packed FP32 is off), conflict-free 128-bit LDS reads "
                         "with 16 wavefronts per CU"}
    first_call_ms = {}
    for name, fn in ops:                       # very first call of each operation: allocates the workspace
        torch.cuda.synchronize()
        t_first = time.perf_counter()
        fn()
        torch.cuda.synchronize()
        first_call_ms[name] = (time.perf_counter() - t_first) * 1e3
    for _ in range(max(0, args.warmup - 1)):
        step()
    torch.cuda.synchronize()
    binding.csrk_profile_enable(args.steps * len(ops))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    records = binding.csrk_profile_collect(args.steps * len(ops) + 8)
    binding.csrk_profile_enable(0)

    ms_per_step = (t1 - t0) * 1e3 / args.steps
    # which kernels did the calls: the last bits differ if it was not the vector kernels
    outputs = {"spmm": lambda: O, "sddmm": lambda: P, "fusedmm": lambda: Of}
    on_matrix_cores = {}
    mfma_switch = os.environ.get("CSRK_MFMA")
    for name, fn in ops:
        fn()
        first = outputs[name]().clone()
        os.environ["CSRK_MFMA"] = "3"
        fn()
        on_matrix_cores[name] = not torch.equal(first, outputs[name]())
        if mfma_switch is None:
            del os.environ["CSRK_MFMA"]
        else:
            os.environ["CSRK_MFMA"] = mfma_switch
    widths = {name: sum(v_ for k_, v_ in w.ops[name].items() if k_ in ("N", "D")) for name, _ in ops}
    op_codes = {"spmm": binding.CSRK_OP_SPMM, "sddmm": binding.CSRK_OP_SDDMM, "fusedmm": binding.CSRK_OP_FUSEDMM}
    matrix_products = {name: binding.csrk_matrix_core_form(op_codes[name], w.M, w.K, w.ops[name].get("N", 0), w.ops[name].get("D", 0))[0]
                       for name, _ in ops}
    matrix_flops = {name: 2.0 * w.M * w.K * (matrix_products[name] * w.ops[name].get("N", 0) + PRODUCTS * w.ops[name].get("D", 0))
                    for name, _ in ops}
    # one cold run per operation: a 1 GiB fill pushes the operands out of L2 and the 256 MB memory-side cache
    cold_ms = {}
    flush = torch.empty(1 << 28, dtype=torch.float32, device="cuda")
    for name, fn in ops:
        flush.fill_(1.0)
        torch.cuda.synchronize()
        binding.csrk_profile_enable(1)
        fn()
        torch.cuda.synchronize()
        rec = binding.csrk_profile_collect(4)
        binding.csrk_profile_enable(0)
        if rec:
            cold_ms[name] = rec[0][1]
    del flush
    per_op = {}
    for kind, ms in records:
        per_op.setdefault(KIND[kind], []).append(ms)
    op_report = {}
    for name, times in per_op.items():
        avg, mn, med = float(np.mean(times)), float(np.min(times)), float(np.median(times))
        tf = flops[name] / avg / 1e9
        op_report[name] = {
            "kernel_ms_avg": round(avg, 4), "kernel_ms_median": round(med, 4), "kernel_ms_min": round(mn, 4),
            "kernel_ms_cold": round(cold_ms[name], 4) if name in cold_ms else None,
            "first_call_wall_ms": round(first_call_ms[name], 3),
            "gflops_avg": round(flops[name] / avg / 1e6, 1), "gflops_best": round(flops[name] / mn / 1e6, 1),
            "frac_fp32_peak": round(tf / FP32_VECTOR_PEAK_TFLOPS, 4),
            "hbm_algorithmic_bytes": int(hbm_bytes[name]),
            "hbm_GBps": round(hbm_bytes[name] / avg / 1e6, 1),
            "frac_hbm_peak": round(hbm_bytes[name] / avg / 1e6 / HBM_PEAK_GBS, 4),
            "kernels": "matrix cores" if on_matrix_cores[name] else "vector",
        }
        if on_matrix_cores[name]:
            op_report[name]["matrix_core_TFLOPs"] = round(matrix_flops[name] / avg / 1e9, 1)
            op_report[name]["frac_bf16_peak"] = round(matrix_flops[name] / avg / 1e9 / BF16_MATRIX_PEAK_TFLOPS, 4)
        else:
            op_report[name]["gathered_TBps"] = round(gather_bytes[name] / avg / 1e9, 2)
        counted, _ = hbm_traffic_from_profiles(args.workload, name)
        if counted:         # FETCH_SIZE + WRITE_SIZE of a recorded rocprofv3 --pmc run of the same kernels
            op_report[name]["hbm_counter_bytes"] = int(counted)
            op_report[name]["hbm_counter_GBps"] = round(counted / avg / 1e6, 1)
            op_report[name]["frac_hbm_peak_counter"] = round(counted / avg / 1e6 / HBM_PEAK_GBS, 4)
        if peaks:
            op_report[name]["frac_hbm_copy_measured"] = round(hbm_bytes[name] / avg / 1e6 / peaks["hbm_copy_GBps"], 4)
            if not on_matrix_cores[name]:
                op_report[name]["frac_fma_measured"] = round(tf / peaks["fma_f32_TFLOPs"], 4)
                op_report[name]["frac_lds_read_measured"] = round(gather_bytes[name] / avg / 1e9 / peaks["lds_read_b128_TBps"], 4)
    # dominant kernel = the one the step spends most time in
    dom = max(per_op, key=lambda k: float(np.mean(per_op[k])))
    dom_ms = float(np.mean(per_op[dom]))
    achieved = flops[dom] / dom_ms / 1e9      # TFLOP/s
    traffic, traffic_source = hbm_traffic_from_profiles(args.workload, dom)
    if on_matrix_cores[dom]:
        rate = matrix_flops[dom] / dom_ms / 1e9
        roofline = {
            "kernel": dom, "bound": "mfma", "achieved": round(rate, 1), "peak": BF16_MATRIX_PEAK_TFLOPS,
            "unit": "TFLOP/s", "frac": round(rate / BF16_MATRIX_PEAK_TFLOPS, 4),
            "useful_TFLOPs": round(achieved, 3),
            "ceiling_note": "rate of the 16-bit products that the matrix cores work through: "
                            f"{matrix_products[dom] if w.ops[dom].get('N') else PRODUCTS} for an FP32 product (scores: {PRODUCTS}), over every "
                            "cell of S (stored or not); useful_TFLOPs counts 2 flops per stored entry and column; the peak "
                            "is the published dense one at 2.4 GHz, the clock under this load is 2.0 GHz (power)",
        }
    else:
        roofline = {
            "kernel": dom, "bound": "alu", "achieved": round(achieved, 3), "peak": FP32_VECTOR_PEAK_TFLOPS,
            "unit": "TFLOP/s", "frac": round(achieved / FP32_VECTOR_PEAK_TFLOPS, 4),
            "ceiling_note": "peak is the published FP32 vector rate; every multiply-add of the vector kernels needs its own 4 "
                            "bytes of a gathered dense row from LDS, so their own ceiling is the LDS read rate "
                            "(measured_peaks.lds_read_b128_TBps / 4 bytes x 2 flops), well below the ALU peak",
        }
    roofline.update({"traffic": traffic, "traffic_source": traffic_source, "flops_per_launch": flops[dom],
                     "avg_launch_ms": round(dom_ms, 4)})

    result = {
        "metric": "GFLOP/s (2*nnz*N) for SPMM + SDDMM + FusedMM, one pass each",
        "value": round(step_flops / ms_per_step / 1e6, 1),
        "unit": "GFLOP/s",
        "n_gpus": 1, "steps": args.steps, "warmup": max(1, args.warmup),
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"{w.name}: {w.M}x{w.K} CSR, nnz={nnz}, {w.recipe}",
                   "ops": {k: {kk: vv for kk, vv in o.items() if kk in ("N", "D")} for k, o in w.ops.items()},
                   "scale": args.scale, "seed": 0},
        "ops": op_report,
        "roofline": roofline,
        "device": torch.cuda.get_device_name(0),
        "input_gen_s": round(t_gen, 2),
    }
    if peaks:
        result["measured_peaks"] = peaks
        if not on_matrix_cores[dom]:
            result["roofline"]["frac_of_lds_ceiling"] = round(achieved / (peaks["lds_read_b128_TBps"] / 4.0 * 2.0), 4)

    if not args.no_phases and "fusedmm" in w.ops and w.ops["fusedmm"]["N"] == 512 and w.ops["fusedmm"]["D"] == 64 \
            and w.M % 64 == 0:
        # where a wavefront's cycles go in the two 512-column tiled kernels (measuring builds, one run each), where these
        # do the call
        ph = {}
        for opname, opcode in (("spmm", binding.CSRK_OP_SPMM), ("fusedmm", binding.CSRK_OP_FUSEDMM)):
            if on_matrix_cores.get(opname, True):
                continue
            cyc, tiles, _ = binding.csrk_tile_phases(opcode, w.M, w.K, 64, 512, rp, ci, v, Af, Bf, Cf, Of)
            total = sum(cyc)
            ph[opname] = {"tiles_per_wavefront": tiles, "cycles_per_wavefront": round(total),
                          "share": {n: round(c / total, 4) for n, c in zip(binding.PHASE_NAMES, cyc) if c > 0}}
        if ph:
            result["phases"] = ph

    if not args.no_sddmm_at_scale:
        # SDDMM alone at this size with both dot lengths of the workloads (the paper times SDDMM on its own too)
        sd = {}
        Psd = torch.empty((nnz,), dtype=torch.float32, device="cuda")
        for Dsd in (64, 128):
            Asd = dev(inputs.normal(0, inputs.STREAM_A, (w.M, Dsd)))
            Bsd = dev(inputs.normal(0, inputs.STREAM_B, (w.K, Dsd)))
            call = lambda: binding.sddmm_csr(w.M, w.K, Dsd, rp, ci, v, Asd, Bsd, Psd)
            call()
            call()
            torch.cuda.synchronize()
            binding.csrk_profile_enable(10)
            for _ in range(10):
                call()
            torch.cuda.synchronize()
            ms = [t for _, t in binding.csrk_profile_collect(16)]
            binding.csrk_profile_enable(0)
            sd[f"D{Dsd}"] = {"ms_min": round(min(ms), 4), "ms_avg": round(sum(ms) / len(ms), 4),
                             "gflops_avg": round(2.0 * nnz * Dsd / (sum(ms) / len(ms)) / 1e6, 1)}
            del Asd, Bsd
        result["sddmm_at_scale"] = sd

    if "fusedmm" in w.ops and not args.no_fusion_report:
        # the paper's central claim is the gain from fusing: time SDDMM -> SPMM through a materialised
        # score array against the fused call, same operands (outside the timed region above)
        o = w.ops["fusedmm"]
        Pu = torch.empty((nnz,), dtype=torch.float32, device="cuda")
        Ou = torch.empty((w.M, o["N"]), dtype=torch.float32, device="cuda")

        def unfused():
            binding.sddmm_csr(w.M, w.K, o["D"], rp, ci, v, Af, Bf, Pu)
            binding.spmm_csr(w.M, w.K, o["N"], rp, ci, Pu, Cf, Ou)

        def fused():
            binding.fusedmm_csr(w.M, w.K, o["D"], o["N"], rp, ci, v, Af, Bf, Cf, Of)

        def time_ms(fn, reps=10):
            fn()
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(reps):
                fn()
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / reps

        tu, tf = time_ms(unfused), time_ms(fused)
        result["fusion"] = {"unfused_sddmm_then_spmm_ms": round(tu, 4), "fused_ms": round(tf, 4),
                            "fused_speedup": round(tu / tf, 3),
                            "max_abs_diff": float((Ou - Of).abs().max().item())}

    if args.plan:
        # a caller that reuses the pattern: analysis once, then calls that launch only the kernel that does the work
        t0 = time.perf_counter()
        plan = binding.csrk_plan_create(w.M, w.K, rp, ci)
        torch.cuda.synchronize()
        create_ms = (time.perf_counter() - t0) * 1e3
        pcalls = []
        if "spmm" in w.ops:
            pcalls.append(("spmm", lambda: binding.spmm_csr_plan(plan, N, v, B, O)))
        if "sddmm" in w.ops:
            pcalls.append(("sddmm", lambda: binding.sddmm_csr_plan(plan, Ds, v, As, Bs, P)))
        if "fusedmm" in w.ops:
            pcalls.append(("fusedmm", lambda: binding.fusedmm_csr_plan(plan, Df, Nf, v, Af, Bf, Cf, Of)))
        planned = {}
        for name, fn in pcalls:
            fn()
            fn()
            torch.cuda.synchronize()
            binding.csrk_profile_enable(args.steps)
            for _ in range(args.steps):
                fn()
            torch.cuda.synchronize()
            ms = [t for _, t in binding.csrk_profile_collect(args.steps + 4)]
            binding.csrk_profile_enable(0)
            planned[name] = {"ms_min": round(min(ms), 4), "ms_avg": round(sum(ms) / len(ms), 4),
                             "gflops_avg": round(flops[name] / (sum(ms) / len(ms) * 1e-3) / 1e9, 1),
                             "unplanned_ms_avg": result["ops"][name]["kernel_ms_avg"]}
        nnz_p, sorted_p, even_p = binding.csrk_plan_info(plan)
        binding.csrk_plan_destroy(plan)
        result["planned"] = {"ops": planned, "plan_create_wall_ms": round(create_ms, 3),
                             "columns_ascending": sorted_p, "rows_even": even_p,
                             "note": "whole calls, same event pair as `ops`; the plan replaces the per-call row "
                                     "analysis and the stand-by launches behind a tiled kernel"}

    if args.bf16:
        # the paper's stated future work: dense operands in bfloat16, FP32 arithmetic.  Same workload; beside them the
        # FP32 general path (CSRK_KTILE=3, which also keeps the matrix-core kernels out), whose kernels they share where
        # they do not run on the matrix cores.
        def to_dev_bf16(a):
            bits, _ = inputs.to_bf16(a)
            return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)

        calls16, calls32 = [], []
        if "spmm" in w.ops:
            B16 = to_dev_bf16(w.ops["spmm"]["B"])
            calls16.append(("spmm", lambda: binding.spmm_csr_bf16(w.M, w.K, N, rp, ci, v, B16, O)))
            calls32.append(("spmm", lambda: binding.spmm_csr(w.M, w.K, N, rp, ci, v, B, O)))
        if "sddmm" in w.ops:
            As16, Bs16 = to_dev_bf16(w.ops["sddmm"]["A"]), to_dev_bf16(w.ops["sddmm"]["B"])
            calls16.append(("sddmm", lambda: binding.sddmm_csr_bf16(w.M, w.K, Ds, rp, ci, v, As16, Bs16, P)))
            calls32.append(("sddmm", lambda: binding.sddmm_csr(w.M, w.K, Ds, rp, ci, v, As, Bs, P)))
        if "fusedmm" in w.ops:
            o = w.ops["fusedmm"]
            Af16, Bf16, Cf16 = to_dev_bf16(o["A"]), to_dev_bf16(o["B"]), to_dev_bf16(o["C"])
            calls16.append(("fusedmm", lambda: binding.fusedmm_csr_bf16(w.M, w.K, Df, Nf, rp, ci, v, Af16, Bf16, Cf16, Of)))
            calls32.append(("fusedmm", lambda: binding.fusedmm_csr(w.M, w.K, Df, Nf, rp, ci, v, Af, Bf, Cf, Of)))

        def time_calls(calls, reps=10):
            out = {}
            for name, fn in calls:
                fn()
                fn()
                torch.cuda.synchronize()
                binding.csrk_profile_enable(reps)
                for _ in range(reps):
                    fn()
                torch.cuda.synchronize()
                ms = [t for _, t in binding.csrk_profile_collect(reps + 4)]
                binding.csrk_profile_enable(0)
                out[name] = {"ms_min": round(min(ms), 4), "ms_avg": round(sum(ms) / len(ms), 4),
                             "gflops_best": round(flops[name] / (min(ms) * 1e-3) / 1e9, 1)}
            return out

        r16 = time_calls(calls16)
        saved = os.environ.get("CSRK_KTILE")
        os.environ["CSRK_KTILE"] = "3"
        r32 = time_calls(calls32)
        if saved is None:
            os.environ.pop("CSRK_KTILE", None)
        else:
            os.environ["CSRK_KTILE"] = saved
        result["bf16_operands"] = {"bf16": r16, "fp32_general_path": r32,
                                   "note": "whole calls; the bf16 ones on the matrix cores where the library chooses these"}

    if not args.no_cpu_baseline:
        import oracle
        # bounded sample: every `stride`-th row, sized for roughly 10-30 s of CPU work
        target_flops = 150e9
        stride = max(1, int(round(step_flops / target_flops)))
        rows = np.arange(0, w.M, stride, dtype=np.int32)
        if args.cpu_rows:
            rows = rows[: args.cpu_rows]
        row_nnz = int(np.sum(w.rowptr[rows + 1] - w.rowptr[rows]))

        def oracle_pass():
            fl = 0.0
            if "spmm" in w.ops:
                o = w.ops["spmm"]
                oracle.spmm(w.M, w.K, o["N"], w.rowptr, w.colidx, w.vals, o["B"], rows=rows)
                fl += 2.0 * row_nnz * o["N"]
            if "sddmm" in w.ops:
                o = w.ops["sddmm"]
                oracle.sddmm(w.M, w.K, o["D"], w.rowptr, w.colidx, w.vals, o["A"], o["B"], rows=rows)
                fl += 2.0 * row_nnz * o["D"]
            if "fusedmm" in w.ops:
                o = w.ops["fusedmm"]
                oracle.fusedmm(w.M, w.K, o["D"], o["N"], w.rowptr, w.colidx, w.vals, o["A"], o["B"], o["C"],
                               rows=rows)
                fl += 2.0 * row_nnz * (o["D"] + o["N"])
            return fl

        # repeat the sample until about 10 s of CPU work have been timed (at most 12 passes)
        t_begin = time.perf_counter()
        cpu_flops, passes = 0.0, 0
        while passes < 12 and (passes == 0 or time.perf_counter() - t_begin < 10.0):
            cpu_flops += oracle_pass()
            passes += 1
        t_cpu = time.perf_counter() - t_begin
        result["cpu_baseline"] = {
            "value": round(cpu_flops / t_cpu / 1e9, 2), "unit": "GFLOP/s", "cores": oracle.num_threads(),
            "kind": "oracle",
            "sample": f"every {stride}th row ({len(rows)} rows, {row_nnz} stored entries) of the same workload, "
                      f"all three operations, {passes} passes, {t_cpu:.1f} s",
        }
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
