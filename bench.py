#!/usr/bin/env python3
"""Benchmark of the LiquidQuant W4A8 GEMM on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME] [--details FILE]
                    [--no-curve] [--no-configs] [--no-calib] [--no-cpu]

A step is one pass of the whole hot path (load packed W4 + group parameters, unpack,
LiquidQuant dequantisation, INT8 MFMA, per-token x per-channel scaling, FP16 store) over
one batch of synthetic activations, with every input already resident in HBM.  Weights
rotate through enough distinct copies (> 512 MB in total) that the 256 MB Infinity Cache
cannot serve them.  The headline workload is the compute-bound end of the metric's M
range (prefill, M=4096, N=K=8192, group 64).  The same JSON line, short enough to survive in the
tail of a log, carries
  * roofline / roofline_hbm: the dominant kernel of the headline and of the HBM-bound
    point (70B up-projection at M=16) against the nominal peaks;
  * calibration: what this GPU reaches on a pure streaming read and on a register-only
    INT8 MFMA loop (constant and random operands);
  * curve_N8192_K8192: [M, TOPS, fraction of the roofline] for M = 1..4096;
  * cpu_baseline: the CPU oracle timed on a bounded sample.
With --details FILE everything else is measured too and written there, with the above in full:
  * curve_N4096_K4096: the same for decode-sized weights;
  * configs: every workload row (decode, 7B MLP, 70B layers, prefill sweep), median of five
    batches, with rotating weights and with one weight buffer (cache-warm) side by side;
  * activation_quant: the per-token FP16 -> INT8 quantisation kernel upstream of the GEMM;
  * ablation_pipeline, ablation_dequant, mfma_shape: the headline shape on the explicit
    producer / consumer form, with the widened dequantisation, and on the other MFMA shape;
  * reference_w8a8_own, reference_w8a8_vendor: INT8 weights without dequantisation;
  * grouped_moe: mixture-of-experts layers in one grouped call vs one call per expert.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

PEAK_HBM_GBS = 8000.0     # MI355X HBM3E, published
PEAK_INT8_TOPS = 5033.0   # dense INT8 MFMA: 256 CU x 4 SIMD x 2048 ops/clk x 2.4 GHz
ROTATE_BYTES = 512 << 20
# HBM-side bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE runs of this file, scaled by what
# the same counters read for a plain 1 GiB copy, --copy-ref) cannot be read from inside a timed
# run: they are carried per (workload, kernel) in profiles/traffic.json, the data file the
# summaries under profiles/ are written from, and are null for anything not profiled.
HBM_WORKLOAD = "l70b_up_M16_N28672_K8192"   # the HBM-bound point of the result line


def measured_traffic(workload, kernel):
    try:
        with open(os.path.join(ROOT, "profiles", "traffic.json")) as f:
            table = json.load(f)
        return table.get(f"{workload}|{kernel}", {}).get("bytes_per_launch")
    except (OSError, ValueError):
        return None


def algorithmic_bytes(M, N, K, g):
    """Bytes the method must move once: packed codes + group parameters + X + Y + scales."""
    return N * K // 2 + 2 * N * K // g + M * K + 2 * M * N + 4 * N + 4 * M


def algorithmic_ops(M, N, K):
    return 2 * M * N * K


class DeviceProblem:
    """Packed weights of one shape in `copies` distinct device buffers + activations."""

    def __init__(self, shape, Ms, torch, api, WL):
        self.shape = shape
        N, K, g = shape.N, shape.K, shape.group
        rng = np.random.Generator(np.random.PCG64(shape.seed))
        W = WL.make_weights(N, K, shape.sigma_w, rng=rng)
        self.packed, self.gparams, self.w_scales = api.liquidquant_pack_weights(W, g)
        del W
        per_copy = self.packed.nbytes + self.gparams.nbytes
        self.copies = max(1, math.ceil(ROTATE_BYTES / per_copy))
        dev = "cuda:0"
        hp, hg = torch.from_numpy(self.packed), torch.from_numpy(self.gparams)
        self.d_packed = [hp.to(dev) for _ in range(self.copies)]
        self.d_gparams = [hg.to(dev) for _ in range(self.copies)]
        self.d_w_scales = torch.from_numpy(self.w_scales).to(dev)
        # FP16 activations from the seeded generator; their INT8 form and per-token scales come
        # from the library's own quantisation kernel (outside every timed region)
        self.X16, self.dX, self.dsx, self.dY = {}, {}, {}, {}
        for M in Ms:
            self.X16[M] = WL.make_activations_f16(M, K, shape.outlier_frac, seed=shape.seed + 1000 + M)
            self.dX[M], self.dsx[M] = api.w4a8_quantize_activations(torch.from_numpy(self.X16[M]).to(dev))
            self.dY[M] = torch.empty((M, N), dtype=torch.float16, device=dev)
        torch.cuda.synchronize()

    def launch(self, M, i, api, stream, variant=-1, rotate=True):
        c = i % self.copies if rotate else 0
        s = self.shape
        if variant < 0:
            api.w4a8_gemm(self.dX[M], self.dsx[M], self.d_packed[c], self.d_gparams[c], self.d_w_scales,
                          s.N, s.K, s.group, out=self.dY[M], stream=stream.cuda_stream)
        else:
            api.w4a8_gemm_variant(variant, self.dX[M], self.dsx[M], self.d_packed[c], self.d_gparams[c],
                                  self.d_w_scales, s.N, s.K, s.group, want_acc=False, out_y=self.dY[M],
                                  stream=stream.cuda_stream)


def time_launches(launch, steps, warmup, torch, stream, graph=False):
    """Average milliseconds per launch over `steps` back-to-back calls of launch(i) (HIP
    events on the launch stream), after `warmup` untimed ones.  With graph=True the `steps`
    launches are captured once into a HIP graph and replayed, which takes the Python/ctypes
    launch cost (about 9 us per call) out of the measurement of kernels shorter than that."""
    with torch.cuda.stream(stream):
        for i in range(warmup):
            launch(i)
        stream.synchronize()
        g = None
        if graph:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                for i in range(steps):
                    launch(warmup + i)
            g.replay()  # untimed first replay
            stream.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(stream)
        if g is not None:
            g.replay()
        else:
            for i in range(steps):
                launch(warmup + i)
        e1.record(stream)
        stream.synchronize()
        torch.cuda.synchronize()
    return e0.elapsed_time(e1) / steps


def time_steps(prob, M, steps, warmup, torch, api, stream, variant=-1, graph=False, rotate=True):
    return time_launches(lambda i: prob.launch(M, i, api, stream, variant, rotate), steps, warmup, torch,
                         stream, graph)


def is_tiny(shape, M):
    """Kernels expected to run shorter than a Python launch: timed inside a HIP graph."""
    return shape.N * shape.K <= (1 << 26) and M <= 32


def time_median(prob, M, torch, api, stream, rotate=True, batches=5, est_ms=None):
    """Median over `batches` of the per-launch average of a batch of back-to-back launches."""
    graph = is_tiny(prob.shape, M)
    # about 50 ms of untimed launches first: the first batches after a change of kernel run at
    # unsettled clocks (measured: up to 15 % slower)
    t_end = time.perf_counter() + 0.05
    while time.perf_counter() < t_end:
        time_steps(prob, M, 20, 0, torch, api, stream, graph=False, rotate=rotate)
    if est_ms is None:
        est_ms = time_steps(prob, M, 10, 3, torch, api, stream, graph=False, rotate=rotate)
    steps = max(20, min(200, int(8.0 / max(est_ms, 1e-3))))
    ts = [time_steps(prob, M, steps, 3 if b == 0 else 0, torch, api, stream, graph=graph, rotate=rotate)
          for b in range(batches)]
    return statistics.median(ts)


def point(shape, M, ms, api, calib=None, ms_same=None):
    t = ms * 1e-3
    ops, byt = algorithmic_ops(M, shape.N, shape.K), algorithmic_bytes(M, shape.N, shape.K, shape.group)
    t_mem, t_mma = byt / (PEAK_HBM_GBS * 1e9), ops / (PEAK_INT8_TOPS * 1e12)
    p = {
        "M": M, "N": shape.N, "K": shape.K, "group": shape.group, "us": round(ms * 1e3, 3),
        "tops": round(ops / t / 1e12, 3), "gbs": round(byt / t / 1e9, 1),
        "bound": "hbm" if t_mem >= t_mma else "mfma",
        "frac_of_roofline": round(max(t_mem, t_mma) / t, 4),
        "variant": api.w4a8_describe_launch(M, shape.N, shape.K, shape.group)[0],
    }
    if ms_same is not None:
        p["us_same_buffer"] = round(ms_same * 1e3, 3)
    if calib:
        # the same roofline with this GPU's measured streaming rate and random-operand MFMA rate
        t_meas = max(byt / (calib["stream_read_gbs"] * 1e9), ops / (calib["mfma_i8_random_tops"] * 1e12))
        p["frac_of_measured"] = round(t_meas / t, 4)
        # the paper's cost model (Sec. 3.2, Eq. 6) fed with the measured rates and the row tile
        # of the kernel that runs: as printed (dequantisation and MMA in series) and with the
        # two overlapped
        from paper_2509_01229_amd import cost_model as CM

        rates = CM.Rates(calib["stream_read_gbs"] * 1e9, calib["mfma_i8_random_tops"] * 1e12,
                         CM.NOMINAL_VALU_LANE_OPS_PER_S)
        first = p["variant"].split("+")[0]
        m_tile = next((t for t in (32, 64, 128, 256) if f"_m{t}" in first), 16)   # (the 16-row kernels name no tile)
        pr = CM.predict(M, shape.N, shape.K, shape.group, rates, m_tile)
        p["model_us"] = {"eq6_serial": round(pr["serial"] * 1e6, 2), "overlapped": round(pr["overlapped"] * 1e6, 2)}
    return p


def calibrate(torch, api, stream):
    """Pure streaming read (512 MiB per launch, and 120 MB slices of it in turn) and the
    register-only MFMA loop, each as the median of five batches."""
    buf = torch.randint(0, 256, (ROTATE_BYTES + (96 << 20),), dtype=torch.uint8, device="cuda:0")
    big = buf[:ROTATE_BYTES]
    out = {}

    def med(launch, steps):
        return statistics.median(time_launches(launch, steps, 2, torch, stream) for _ in range(5))

    ms = med(lambda i: api.w4a8_calib_stream_read(big, stream.cuda_stream), 10)
    out["stream_read_gbs"] = round(ROTATE_BYTES / (ms * 1e-3) / 1e9, 1)
    slice_bytes = 120 << 20
    slices = [buf[j * slice_bytes:(j + 1) * slice_bytes] for j in range(buf.numel() // slice_bytes)]
    ms = med(lambda i: api.w4a8_calib_stream_read(slices[i % len(slices)], stream.cuda_stream), 50)
    out["stream_read_gbs_120MiB_launches"] = round(slice_bytes / (ms * 1e-3) / 1e9, 1)
    del slices, big, buf
    torch.cuda.empty_cache()
    for key, rnd in (("mfma_i8_constant_tops", False), ("mfma_i8_random_tops", True)):
        ops = []
        ms = med(lambda i: ops.append(api.w4a8_calib_mfma_i8(500, rnd, stream.cuda_stream)), 10)
        out[key] = round(ops[0] / (ms * 1e-3) / 1e12, 1)
    out["note"] = ("read: 16-byte non-temporal loads over 512 MiB per launch; mfma: 64 x 500 "
                   "v_mfma_i32_32x32x32_i8 per wave, two waves per SIMD, register operands")
    return out


def activation_quant_points(torch, api, WL, stream, calib):
    """The per-token FP16 -> INT8 quantisation upstream of the GEMM (with smooth divide):
    algorithmic bytes 2*M*K in + M*K out + scales; HBM-bound."""
    rows = []
    for M, K in ((16, 8192), (4096, 8192), (2048, 28672)):
        X = torch.from_numpy(WL.make_activations_f16(M, K, 0.001, seed=M + K)).to("cuda:0")
        copies = max(1, min(8, math.ceil(ROTATE_BYTES / (3 * M * K))))
        Xs = [X] + [X.clone() for _ in range(copies - 1)]
        smooth = torch.from_numpy(WL.make_smooth(K, seed=K)).to("cuda:0")
        q = torch.empty((M, K), dtype=torch.int8, device="cuda:0")
        sc = torch.empty((M,), dtype=torch.float32, device="cuda:0")

        def launch(i):
            api.w4a8_quantize_activations(Xs[i % copies], smooth, out_q=q, out_scales=sc, stream=stream.cuda_stream)

        tiny = M * K < (1 << 22)
        ms = statistics.median(time_launches(launch, 50, 5, torch, stream, graph=tiny) for _ in range(5))
        byt = 3 * M * K + 4 * M + 4 * K
        r = {"M": M, "K": K, "us": round(ms * 1e3, 3), "gbs": round(byt / (ms * 1e-3) / 1e9, 1),
             "frac_of_roofline": round(byt / (ms * 1e-3) / 1e9 / PEAK_HBM_GBS, 4), "bound": "hbm"}
        if calib:
            r["frac_of_measured"] = round(r["gbs"] / calib["stream_read_gbs"], 4)
        rows.append(r)
        del Xs, X, q
        torch.cuda.empty_cache()
    return rows


def vendor_w8a8_reference(torch, stream):
    """Context only: the vendor INT8 GEMM (torch._int_mm, W8A8, no dequantisation, INT32 out)
    on N = K = 8192 with Gaussian-like INT8 operands and rotating weights -- the role the
    W8A8 baseline plays in the paper's kernel comparison (Sec. 7.3)."""
    rows = []
    try:
        N = K = 8192
        gen = torch.Generator(device="cuda:0").manual_seed(0)
        Bs = [torch.clamp(torch.randn((K, N), device="cuda:0", generator=gen) * 40, -127, 127).to(torch.int8)
              for _ in range(8)]
        for M in (32, 256, 1024, 4096):
            A = torch.clamp(torch.randn((M, K), device="cuda:0", generator=gen) * 40, -127, 127).to(torch.int8)
            out = torch.empty((M, N), dtype=torch.int32, device="cuda:0")

            def launch(i):
                torch._int_mm(A, Bs[i % 8], out=out)

            ms = statistics.median(time_launches(launch, 30, 5, torch, stream) for _ in range(3))
            rows.append({"M": M, "N": N, "K": K, "us": round(ms * 1e3, 2),
                         "tops": round(algorithmic_ops(M, N, K) / (ms * 1e-3) / 1e12, 1)})
    except Exception as e:  # the reference is optional; the product does not depend on it
        rows.append({"error": f"{type(e).__name__}: {e}"[:200]})
    return rows


def own_w8a8_reference(prob, torch, api, stream):
    """The W8A8 reference kernel of this library (same tiles and pipeline as the W4A8 kernel,
    INT8 weights fed to the MFMA as loaded) on the dequantised weights of the headline
    problem, so that both kernels compute the same integers; W4A8 timed beside it."""
    s = prob.shape
    N, K, g = s.N, s.K, s.group
    rows = []
    Wd = api.w4a8_dequant_dump(prob.d_packed[0], prob.d_gparams[0], N, K, g)
    torch.cuda.synchronize()
    packed = torch.from_numpy(api.w8a8_pack_weights(Wd.cpu().numpy()))
    del Wd
    copies = max(1, math.ceil(ROTATE_BYTES / (N * K)))
    dW = [packed.to("cuda:0") for _ in range(copies)]
    for M in (256, 1024, 4096):
        if M not in prob.dX:
            continue

        def launch(i):
            api.w8a8_gemm(prob.dX[M], prob.dsx[M], dW[i % copies], prob.d_w_scales, N, K, out_y=prob.dY[M],
                          stream=stream.cuda_stream)

        ms8 = statistics.median(time_launches(launch, 30, 5, torch, stream) for _ in range(3))
        ms4 = statistics.median(time_steps(prob, M, 30, 5, torch, api, stream) for _ in range(3))
        rows.append({"M": M, "N": N, "K": K, "w8a8_us": round(ms8 * 1e3, 2),
                     "w8a8_tops": round(algorithmic_ops(M, N, K) / (ms8 * 1e-3) / 1e12, 1),
                     "w4a8_us": round(ms4 * 1e3, 2),
                     "w4a8_tops": round(algorithmic_ops(M, N, K) / (ms4 * 1e-3) / 1e12, 1)})
    del dW
    torch.cuda.empty_cache()
    return rows


def grouped_moe_points(torch, api, WL, stream):
    """Mixture-of-experts layers shaped like Mixtral-8x7B (8 experts, top-2 routing, hidden
    4096, intermediate 14336; Sec. 7.3 of the paper): one grouped call against one
    w4a8_gemm call per expert, same kernels, rotating weight copies."""
    rows_out = []
    E = 8
    for lname, N, K in (("moe_up", 14336, 4096), ("moe_down", 4096, 14336)):
        g = 64
        # two distinct experts' weights, repeated: timing does not depend on the values
        packs = [api.liquidquant_pack_weights(WL.make_weights(N, K, 0.02, seed=70 + e), g) for e in range(2)]
        codes = np.concatenate([packs[e % 2][0] for e in range(E)])
        gps = np.concatenate([packs[e % 2][1] for e in range(E)])
        sws = np.stack([packs[e % 2][2] for e in range(E)])
        copies = max(1, math.ceil(ROTATE_BYTES / (codes.nbytes + gps.nbytes)))
        d_codes = [torch.from_numpy(codes).to("cuda:0") for _ in range(copies)]
        d_gps = [torch.from_numpy(gps).to("cuda:0") for _ in range(copies)]
        d_sw = torch.from_numpy(sws).to("cuda:0")
        cb, gb = api.liquidquant_packed_size(N, K, g)
        for B in (16, 256, 4096):
            rng = np.random.Generator(np.random.PCG64(B))
            rows = rng.multinomial(2 * B, [1.0 / E] * E)
            offs = np.concatenate([[0], np.cumsum(rows)]).astype(int)
            M = int(offs[-1])
            dX, dsx = api.w4a8_quantize_activations(torch.from_numpy(WL.make_activations_f16(M, K, 0.0, seed=B)).to("cuda:0"))
            Y = torch.empty((M, N), dtype=torch.float16, device="cuda:0")
            Xe = [dX[offs[e]:offs[e + 1]] for e in range(E)]
            sxe = [dsx[offs[e]:offs[e + 1]].clone() for e in range(E)]  # own allocations: 16-byte aligned
            Ye = [Y[offs[e]:offs[e + 1]] for e in range(E)]

            def grouped(i):
                api.w4a8_grouped_gemm(offs, dX, dsx, d_codes[i % copies], d_gps[i % copies], d_sw, N, K, g,
                                      out_y=Y, stream=stream.cuda_stream)

            def sequential(i):
                c = i % copies
                for e in range(E):
                    if rows[e]:
                        api.w4a8_gemm(Xe[e], sxe[e], d_codes[c][e * cb:(e + 1) * cb], d_gps[c][e * gb:(e + 1) * gb],
                                      d_sw[e], N, K, g, out=Ye[e], stream=stream.cuda_stream)

            # both inside a HIP graph: eight short launches from Python would otherwise be
            # timed by the interpreter, not by the GPU
            t_g = statistics.median(time_launches(grouped, 10, 2, torch, stream, graph=True) for _ in range(3))
            t_s = statistics.median(time_launches(sequential, 10, 2, torch, stream, graph=True) for _ in range(3))
            ops = algorithmic_ops(M, N, K)
            byt = E * (cb + gb) + M * K + 2 * M * N
            rows_out.append({"layer": lname, "experts": E, "N": N, "K": K, "tokens": B, "rows": rows.tolist(),
                             "us_grouped": round(t_g * 1e3, 2), "us_per_expert_calls": round(t_s * 1e3, 2),
                             "speedup": round(t_s / t_g, 2), "tops": round(ops / (t_g * 1e-3) / 1e12, 1),
                             "gbs": round(byt / (t_g * 1e-3) / 1e9, 1)})
        del d_codes, d_gps
        torch.cuda.empty_cache()
    return rows_out


def cpu_baseline(prob, M, budget_s=12.0):
    """The C oracle (as it stands) on a bounded row sample of the same workload."""
    from oracle import c_oracle
    from oracle import lqq_oracle as O
    from paper_2509_01229_amd import api

    s = prob.shape
    codes, s_u8, a = api.liquidquant_unpack_weights(prob.packed, prob.gparams, s.N, s.K, s.group)
    canon = O.pack_canonical(codes)
    del codes
    X, sx = O.quantize_activations(prob.X16[M][:min(M, 4096)])  # the oracle's own per-token quantisation
    t0 = time.perf_counter()
    c_oracle.w4a8_gemm(X[:1], sx[:1], canon, s_u8, a, prob.w_scales, s.group)
    t_one = time.perf_counter() - t0                       # dominated by the dequantisation
    n3 = min(3, len(X))
    t0 = time.perf_counter()
    c_oracle.w4a8_gemm(X[:n3], sx[:n3], canon, s_u8, a, prob.w_scales, s.group)
    t_three = time.perf_counter() - t0
    per_row = max((t_three - t_one) / 2, 1e-6)
    rows = int(max(1, min(len(X), (budget_s - t_one) / per_row)))
    t0 = time.perf_counter()
    c_oracle.w4a8_gemm(X[:rows], sx[:rows], canon, s_u8, a, prob.w_scales, s.group)
    dt = time.perf_counter() - t0
    return {
        "value": round(algorithmic_ops(rows, s.N, s.K) / dt / 1e12, 6), "unit": "TOPS",
        "cores": c_oracle.threads(), "kind": "oracle",
        "sample": f"rows 0..{rows} of X (of M={M}), all N={s.N} K={s.K} group={s.group}; one full "
                  f"dequantisation included; {dt:.1f} s",
    }


def short_line(out):
    """The result line: the contract's keys and one figure or two of each section."""
    line = {k: v for k, v in out.items() if k not in ("configs", "activation_quant", "grouped_moe")
            and not k.startswith(("curve_", "reference_", "ablation_", "mfma_shape"))}
    if "curve_N8192_K8192" in out:
        line["curve_N8192_K8192"] = [[p["M"], p["tops"], p["frac_of_roofline"]] for p in out["curve_N8192_K8192"]]
    if "calibration" in out:
        line["calibration"] = {k: v for k, v in out["calibration"].items() if k != "note"}
    if "cpu_baseline" in out:
        line["cpu_baseline"] = {k: out["cpu_baseline"][k] for k in ("value", "unit", "cores", "kind")}
    return line


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="prefill_M4096_N8192_K8192")
    ap.add_argument("--variant", type=int, default=-1, help="force a kernel variant (tuning)")
    ap.add_argument("--no-curve", action="store_true")
    ap.add_argument("--no-configs", action="store_true")
    ap.add_argument("--no-calib", action="store_true")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--details", metavar="FILE", help="measure every section and write it to FILE as JSON")
    ap.add_argument("--copy-ref", action="store_true",
                    help="only run a plain device-to-device copy of 1 GiB five times (reference "
                         "for scaling the profiler's FETCH_SIZE / WRITE_SIZE counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build runs on one GPU only (the path has no collective); use --gpus 1")

    import torch

    from paper_2509_01229_amd import api
    from paper_2509_01229_amd import workloads as WL

    if not torch.cuda.is_available():
        sys.exit("bench.py needs a GPU")
    if args.copy_ref:
        src = torch.ones(1 << 30, dtype=torch.uint8, device="cuda:0")
        dst = torch.empty_like(src)
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_ref_bytes_read": 1 << 30, "copy_ref_bytes_written": 1 << 30, "copies": 5}))
        return
    api.lib()
    torch.cuda.set_device(0)
    stream = torch.cuda.Stream()

    head = WL.by_name(args.workload)
    curve_Ms = [] if args.no_curve else [1, 2, 4, 8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096]
    family = [s for s in WL.ALL_SHAPES if (s.N, s.K, s.group, s.seed) == (head.N, head.K, head.group, head.seed)]
    Ms = sorted(set(curve_Ms + [head.M] + ([] if args.no_configs else [s.M for s in family])))
    prob = DeviceProblem(head, Ms, torch, api, WL)

    # Untimed pre-warm of about 0.2 s so that the timed steps run at settled clocks, then the
    # W warm-up steps and the K timed steps of the contract.
    t_end = time.perf_counter() + 0.2
    while time.perf_counter() < t_end:
        time_steps(prob, head.M, 10, 0, torch, api, stream, args.variant)
    ms = time_steps(prob, head.M, args.steps, args.warmup, torch, api, stream, args.variant)
    hp = point(head, head.M, ms, api)
    ops = algorithmic_ops(head.M, head.N, head.K)
    byt = algorithmic_bytes(head.M, head.N, head.K, head.group)
    if hp["bound"] == "mfma":
        roof = {"bound": "mfma", "achieved": round(ops / (ms * 1e-3) / 1e12, 2), "peak": PEAK_INT8_TOPS,
                "unit": "TOP/s"}
    else:
        roof = {"bound": "hbm", "achieved": round(byt / (ms * 1e-3) / 1e9, 1), "peak": PEAK_HBM_GBS,
                "unit": "GB/s"}
    roof["frac"] = round(roof["achieved"] / roof["peak"], 4)
    roof["kernel"] = hp["variant"]
    roof["traffic"] = measured_traffic(head.name, hp["variant"])
    roof["algorithmic_bytes"] = byt
    roof["algorithmic_ops"] = ops

    out = {
        "metric": "W4A8 GEMM TOPS and % of HBM / int8-MFMA roofline vs M (1..4096)",
        "value": hp["tops"], "unit": "TOPS", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms, 5), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "int8 x uint4->int8, int32 accumulate, fp16 out", "data": "synthetic",
        "config": {"workload": head.name, "M": head.M, "N": head.N, "K": head.K, "group": head.group,
                   "weight_copies_rotated": prob.copies},
        "roofline": roof,
    }

    calib = None
    if not args.no_calib:
        calib = calibrate(torch, api, stream)
        out["calibration"] = calib
        if roof["bound"] == "mfma":
            roof["frac_of_measured_random_operand_mfma"] = round(roof["achieved"] / calib["mfma_i8_random_tops"], 4)
        else:
            roof["frac_of_measured_stream_read"] = round(roof["achieved"] / calib["stream_read_gbs"], 4)

    if not args.no_curve:
        out["curve_N8192_K8192" if (head.N, head.K) == (8192, 8192) else f"curve_N{head.N}_K{head.K}"] = [
            point(head, M, time_median(prob, M, torch, api, stream, batches=3), api, calib) for M in curve_Ms]

    if not args.no_configs:
        # every workload row: rotating weights (HBM-cold) and one weight buffer side by side
        rows = []
        groups = []
        for s in WL.DECODE + WL.MLP_7B + WL.LAYERS_70B + WL.PREFILL:
            if not args.details and s.name != HBM_WORKLOAD:
                continue
            key = (s.N, s.K, s.group, s.seed)
            if not groups or groups[-1][0] != key:
                groups.append((key, []))
            groups[-1][1].append(s)
        for key, shapes in groups:
            if key == (head.N, head.K, head.group, head.seed):
                p2 = prob
            else:
                extra_Ms = curve_Ms if (shapes[0].N, shapes[0].K) == (4096, 4096) else []
                p2 = DeviceProblem(shapes[0], sorted(set([s.M for s in shapes] + extra_Ms)), torch, api, WL)
                if extra_Ms:  # the second curve of the metric: decode-sized weights
                    out["curve_N4096_K4096"] = [
                        point(shapes[0], M, time_median(p2, M, torch, api, stream, batches=3), api, calib)
                        for M in extra_Ms]
            # the oracle beside every family of configs: a bounded row sample of its largest batch
            fam_cpu = None
            if args.details and not args.no_cpu and p2 is not prob:
                fam_cpu = cpu_baseline(p2, max(s.M for s in shapes if s.M in p2.dX), budget_s=2.5)
            for s in shapes:
                if s.M not in p2.dX:
                    continue
                cold = time_median(p2, s.M, torch, api, stream, rotate=True)
                warm = time_median(p2, s.M, torch, api, stream, rotate=False, est_ms=cold)
                r = point(s, s.M, cold, api, calib, ms_same=warm)
                r["workload"] = s.name
                if fam_cpu:
                    r["cpu_oracle"] = fam_cpu
                rows.append(r)
            if p2 is not prob:
                del p2
                torch.cuda.empty_cache()
        out["configs"] = rows
        hb = next((r for r in rows if r["workload"] == HBM_WORKLOAD), None)
        if hb:
            out["roofline_hbm"] = {
                "bound": "hbm", "achieved": hb["gbs"], "peak": PEAK_HBM_GBS, "unit": "GB/s",
                "frac": round(hb["gbs"] / PEAK_HBM_GBS, 4),
                "traffic": measured_traffic(hb["workload"], hb["variant"]),
                "algorithmic_bytes": algorithmic_bytes(hb["M"], hb["N"], hb["K"], hb["group"]),
                "kernel": hb["variant"], "workload": hb["workload"]}
            if calib:
                out["roofline_hbm"]["frac_of_measured_stream_read"] = round(hb["gbs"] / calib["stream_read_gbs"], 4)

    if args.details and not args.no_configs:
        out["activation_quant"] = activation_quant_points(torch, api, WL, stream, calib)
        out["reference_w8a8_own"] = own_w8a8_reference(prob, torch, api, stream)
        # Fig. 13's pipeline comparison on this chip: the dispatcher's implicit form against the
        # explicit producer / consumer form (dequantised weights handed over through LDS)
        names = api.w4a8_variant_names()
        if "excp_m128" in names:
            t_im = statistics.median(time_steps(prob, head.M, 30, 5, torch, api, stream) for _ in range(3))
            t_ex = statistics.median(time_steps(prob, head.M, 30, 5, torch, api, stream, names.index("excp_m128"))
                                     for _ in range(3))
            out["ablation_pipeline"] = {"workload": head.name, "implicit_us": round(t_im * 1e3, 2),
                                        "explicit_lds_round_trip_us": round(t_ex * 1e3, 2),
                                        "explicit_over_implicit": round(t_ex / t_im, 3)}
        # Fig. 13's other half: the same tiled kernel (two waves per SIMD, X through LDS by
        # registers) with LiquidQuant's 7-instruction dequantisation and with the widened
        # overflow-safe form it replaces
        if "widened_dq_m128" in names and "duo_m128_s1" in names:
            t_lq = statistics.median(time_steps(prob, head.M, 30, 5, torch, api, stream, names.index("duo_m128_s1"))
                                     for _ in range(3))
            t_wd = statistics.median(time_steps(prob, head.M, 30, 5, torch, api, stream, names.index("widened_dq_m128"))
                                     for _ in range(3))
            out["ablation_dequant"] = {"workload": head.name, "kernel": "duo_m128_s1",
                                       "liquidquant_us": round(t_lq * 1e3, 2), "widened_us": round(t_wd * 1e3, 2),
                                       "widened_over_liquidquant": round(t_wd / t_lq, 3)}
        # the MFMA shape under a power-bound load: the same 256 x 256 tile kernel (one wave per
        # SIMD, persistent) on v_mfma_i32_32x32x32_i8 and on v_mfma_i32_16x16x64_i8
        if "solo_pt_m256" in names and "solo16_pt_m256" in names:
            t_32 = statistics.median(time_steps(prob, head.M, 30, 5, torch, api, stream, names.index("solo_pt_m256"))
                                     for _ in range(3))
            t_16 = statistics.median(time_steps(prob, head.M, 30, 5, torch, api, stream, names.index("solo16_pt_m256"))
                                     for _ in range(3))
            out["mfma_shape"] = {"workload": head.name, "mfma_32x32x32_us": round(t_32 * 1e3, 2),
                                 "mfma_16x16x64_us": round(t_16 * 1e3, 2), "ratio": round(t_32 / t_16, 3)}
        del prob.d_packed[1:], prob.d_gparams[1:]
        torch.cuda.empty_cache()
        out["reference_w8a8_vendor"] = vendor_w8a8_reference(torch, stream)
        out["grouped_moe"] = grouped_moe_points(torch, api, WL, stream)

    if not args.no_cpu:
        out["cpu_baseline"] = cpu_baseline(prob, head.M)
        for r in out.get("configs", []):
            r.setdefault("cpu_oracle", out["cpu_baseline"])  # rows of the headline's own family

    if args.details:
        with open(args.details, "w") as f:
            json.dump(out, f, indent=1)
    print(json.dumps(short_line(out)), flush=True)


if __name__ == "__main__":
    main()
