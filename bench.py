#!/usr/bin/env python3
"""BaKron solve benchmark on one MI355X.

One step = one bakron_solve (the whole hot path: workspace init, every leaf
wavefront and every divide-and-conquer push) on one synthetic LLM-shaped
layer whose inputs are already resident in HBM.  Default workload: the
28672 x 8192 Llama-70B-MLP-shaped layer (INT4, per-row scales, 1% damping),
the largest of the five layer shapes; --config 1..4 select the others.

Prints ONE JSON line on stdout; progress goes to stderr.
"""
from __future__ import annotations

import argparse
import json
import os
import platform
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "BaKron solve ms/layer and TFLOP/s (fraction of fp32 MFMA peak), 1 MI355X"
PEAK_FP32_MFMA = 157.3      # TFLOP/s, 256 CU x 4 SIMD x 64 flop/clk x 2.4 GHz
PEAK_HBM = 8000.0           # GB/s
PEAK_FP64_MFMA = 78.6       # TFLOP/s, dense fp64 matrix peak
PEAK_SPLIT = 2500.0 / 6     # TFLOP/s, fp32 products as six bf16 products at the dense bf16 peak
# Paper, Table 3: 4096 x 4096 solved in 0.288 s on one RTX PRO 6000 (fp32).
PAPER_4096_S = 0.288
# Paper, Table 3 (seconds on one RTX PRO 6000, fp32): (m, n): (GPTQ, BaKron, BaKron-antidiagonal)
PAPER_T3 = {(1024, 1024): (0.005, 0.025, 0.092), (2048, 2048): (0.012, 0.074, 0.599),
            (4096, 4096): (0.025, 0.288, 7.648), (8192, 8192): (0.059, 1.839, 110.379),
            (8192, 2048): (0.013, 0.335, 6.445), (2048, 8192): (0.046, 0.322, 6.037),
            (14336, 4096): (0.030, 1.600, 72.886), (4096, 14336): (0.088, 1.717, 73.437)}


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def device_peak() -> dict:
    """CU count and peak clock of device 0 as the HIP runtime reports them,
    and the fp32 MFMA peak they imply (256 flop per clock per CU); the
    published 157.3 TFLOP/s is what `frac` uses."""
    import ctypes
    out = {}
    try:
        hip = ctypes.CDLL("libamdhip64.so")
        v = ctypes.c_int()
        # hipDeviceAttributeMultiprocessorCount = 63, hipDeviceAttributeClockRate = 5 (kHz)
        for name, attr in (("cus", 63), ("peak_clock_khz", 5)):
            if hip.hipDeviceGetAttribute(ctypes.byref(v), attr, 0) == 0:
                out[name] = v.value
    except OSError:
        return out
    if "cus" in out and "peak_clock_khz" in out:
        out["fp32_mfma_peak_tflops"] = out["cus"] * 256 * out["peak_clock_khz"] * 1e3 / 1e12
    return out


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or "unknown"


def cpu_baseline(cfg_inputs, rows: int) -> dict:
    """The fp64 oracle's Alg. 5 (BaKron-recursive: divide and conquer with
    BLAS-3 feedback, on every BLAS thread of the host) timed free-running on
    a bounded sample of the same workload: the layer made of the first `rows`
    output rows (those rows of W, the leading rows x rows block of the
    output-side Gram B, all of A), solved in full including its own
    factorisation (timed separately).  The rate is counted TFLOP/s
    (rows * n * (rows + n) / seconds); ms_per_layer scales it to the whole
    layer by counted work."""
    import numpy as np
    import oracle
    W = cfg_inputs["W"]
    m, n = W.shape
    k = min(int(rows), m)
    Ws = np.ascontiguousarray(W[:k])
    Bs = np.ascontiguousarray(cfg_inputs["B"][:k, :k])
    ss = np.ascontiguousarray(cfg_inputs["scale"][:k])
    t0 = time.perf_counter()
    LA = oracle.normalized_factor_rev(cfg_inputs["A"], cfg_inputs["damp"])
    LB = oracle.normalized_factor_rev(Bs, cfg_inputs["damp"])
    t_fac = time.perf_counter() - t0
    t0 = time.perf_counter()
    oracle.babai_recursive(Ws, LA, LB, ss, cfg_inputs["bits"])
    t_solve = time.perf_counter() - t0
    F_sample = float(k) * n * (k + n)
    F = float(m) * n * (m + n)
    rate = F_sample / t_solve
    threads = oracle.blas_threads()
    return dict(value=rate / 1e12, unit="TFLOP/s", cores=threads, kind="oracle",
                sample=(f"the {k}x{n} layer formed by the first {k} output rows of the same "
                        f"{m}x{n} workload (W rows, leading {k}x{k} block of B, all of A), solved "
                        f"in full by the fp64 oracle's Alg. 5 (BLAS-3 feedback on {threads} BLAS "
                        f"threads, leaf rounding single-threaded) in {t_solve:.1f} s; "
                        f"ms_per_layer scales the counted rate to the whole layer"),
                ms_per_layer=F / rate * 1e3, sample_seconds=t_solve, factor_seconds=t_fac,
                sample_counted_flops=F_sample, host_cpu=cpu_model(), host_nproc=os.cpu_count())


def cpu_full(cfg_inputs) -> dict:
    """The oracle's Alg. 5 on the whole layer, free-running, no extrapolation
    (factorisation by the RevCholesky route timed separately)."""
    import oracle
    W = cfg_inputs["W"]
    m, n = W.shape
    t0 = time.perf_counter()
    LA = oracle.normalized_factor_rev(cfg_inputs["A"], cfg_inputs["damp"])
    LB = oracle.normalized_factor_rev(cfg_inputs["B"], cfg_inputs["damp"])
    t_fac = time.perf_counter() - t0
    log(f"[bench] cpu full: factors {t_fac:.1f} s")
    t0 = time.perf_counter()
    oracle.babai_recursive(W, LA, LB, cfg_inputs["scale"], cfg_inputs["bits"])
    t_solve = time.perf_counter() - t0
    F = float(m) * n * (m + n)
    return dict(kind="oracle-full-layer", solve_seconds=t_solve, factor_seconds=t_fac,
                counted_tflops=F / t_solve / 1e12, blas_threads=oracle.blas_threads(),
                host_cpu=cpu_model(), host_nproc=os.cpu_count(), m=m, n=n)


def validate_outputs(pk, f, W, s, bits, codes, V) -> dict:
    """Checks of the timed solves' outputs, outside the timed region: a debug
    solve (which also validates the scales and exports the pre-rounding
    values x) must reproduce the last timed solve's codes and V bit for bit,
    V must be the single fp32 product s_i * c_ij, and every code must be the
    quantisation of the solve's own x (clamp(rint(x)); code 0 where s_i = 0).
    Raises on any mismatch.  Parity with the fp64 oracle is the tests' job."""
    import torch
    cd, vd, x = pk.solve(W, f, bits, s, debug=True)
    torch.cuda.synchronize()
    if not f.check():
        raise RuntimeError("validation solve: a tile-ordering wait gave up")
    l = (1 << (bits - 1)) - 1
    same = bool(torch.equal(cd, codes)) and bool(torch.equal(vd.view(torch.int32), V.view(torch.int32)))
    sv = (s[:, None] * codes.to(torch.float32))
    v_ok = bool(torch.equal(sv, V))     # value equality: V may hold -0.0 where x < 0 rounds to 0
    zero = (s == 0)[:, None].expand_as(x)
    q = torch.where(zero, torch.zeros_like(x), torch.clamp(torch.round(x), -l, l))
    own = bool(torch.equal(q.to(torch.int8), codes))
    del cd, vd, x, sv, q
    out = dict(repeat_bitwise=same, v_is_s_times_code=v_ok, codes_round_own_x=own)
    if not all(out.values()):
        raise RuntimeError(f"output validation failed: {out}")
    return out


def measured_traffic(kernel: str, workload: str, sources=("solve.hip", "split.h", "common.h")):
    """HBM bytes per launch from the committed rocprofv3 FETCH_SIZE/WRITE_SIZE
    summary, or None if there is none for this kernel and workload or the
    kernel sources changed since it was measured."""
    import hashlib
    path = os.path.join(ROOT, "profiles", f"{kernel}_{workload}_hbm-traffic.json")
    if not os.path.exists(path):
        return None
    rec = json.load(open(path))
    src = b"".join(open(os.path.join(ROOT, "paper_2608_06291_amd", "csrc", f), "rb").read()
                   for f in sources)
    if hashlib.sha256(src).hexdigest() != rec.get("source_sha256"):
        return None
    return rec["bytes_per_launch"]


def table3(max_antidiag_elems: int):
    """Runtime comparison on the paper's Table 3 shapes: GPTQ (B = I: the
    one-sided kernel, Alg. 1 on every row), BaKron and BaKron-antidiagonal
    (Alg. 3), solve only
    (factorisation excluded, as in the paper).  Synthetic inputs: A, B the
    AR(1) Toeplitz matrices rho^|i-j| (rho 0.5 / 0.2), W ~ N(0, 0.02^2), per-row
    INT4 scales max|W_i|/7, damping 0.01.  Prints one JSON line per shape."""
    import torch
    import paper_2608_06291_amd as pk
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(dev)   # not the legacy default stream (see main)
    torch.cuda.set_stream(stream)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def timed(fn, reps):
        for _ in range(3):   # first call allocates; the rest settle clocks after the previous shape
            fn()
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(reps):
            fn()
        e1.record(stream)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps / 1e3

    def toeplitz(d, rho):
        i = torch.arange(d, device=dev, dtype=torch.float32)
        return rho ** (i[:, None] - i[None, :]).abs()

    rows = []
    for (m, n), paper in PAPER_T3.items():
        g = torch.Generator(device=dev).manual_seed(m * 100003 + n)
        W = torch.randn((m, n), generator=g, device=dev) * 0.02
        s = (W.abs().amax(dim=1) / 7.0).contiguous()
        A, B = toeplitz(n, 0.5), toeplitz(m, 0.2)
        f2 = pk.factor(A, B, 0.01)
        f1 = pk.factor(A, None, 0.01)
        codes = torch.empty((m, n), dtype=torch.int8, device=dev)
        V = torch.empty((m, n), dtype=torch.float32, device=dev)
        t_gptq = timed(lambda: pk.solve(W, f1, 4, s, codes=codes, V=V), 20)
        t_bk = timed(lambda: pk.solve(W, f2, 4, s, codes=codes, V=V), 20)
        t_ad = None
        if m * n <= max_antidiag_elems:
            t0 = time.perf_counter()
            pk.solve_antidiag(W, f2, 4, s, codes=codes, V=V)
            torch.cuda.synchronize()
            t_ad = time.perf_counter() - t0
        f1.close()
        f2.close()
        r = dict(m=m, n=n, gptq_s=t_gptq, bakron_s=t_bk, antidiag_s=t_ad,
                 speedup=(t_ad / t_bk) if t_ad else None,
                 paper_s=dict(gptq=paper[0], bakron=paper[1], antidiag=paper[2],
                              speedup=paper[2] / paper[1]))
        rows.append(r)
        print(json.dumps(r), flush=True)
        del W, A, B, codes, V
        torch.cuda.empty_cache()
    log("| m x n | GPTQ (s) | BaKron (s) | BaKron-antidiag (s) | speedup | paper speedup |")
    for r in rows:
        ad = f"{r['antidiag_s']:.3f}" if r["antidiag_s"] else "-"
        sp = f"{r['speedup']:.1f}x" if r["speedup"] else "-"
        log(f"| {r['m']} x {r['n']} | {r['gptq_s']:.4f} | {r['bakron_s']:.4f} | {ad} | {sp} | "
            f"{r['paper_s']['speedup']:.1f}x |")


# Kronecker-factor construction (App. A) at the paper's calibration size:
# 256 sequences x 2048 tokens (App. D), on Llama-3-8B's MLP and on a 4096 x 4096
# projection with a backpropagated (global) Hessian.
FACTOR_N = 256 * 2048
FACTOR_WORKLOADS = (("mlp-local-up-4096x14336", "kfac"), ("mlp-local-up-4096x14336", "shampoo"),
                    ("global-4096x4096", "kfac"), ("global-4096x4096", "shampoo"),
                    ("global-4096x4096", "shampoo3"))


def _gram_flops(N: int, d: int) -> float:
    """Algorithmic flops of one Gram over N samples of dimension d: a multiply
    and an add per sample for each of the d (d + 1) / 2 distinct entries."""
    return float(N) * d * (d + 1)


def factors_bench(steps: int, warmup: int, n_samples: int, cpu_seconds: float, do_cpu: bool,
                  only: str | None = None):
    """One JSON line per Kronecker-factor workload: the whole factor
    construction per step (every Gram, weight and mask of the pair), the
    dominant Gram launch timed alone for the roofline, 48 entries of each
    factor checked against the fp64 oracle, and the oracle's own CPU rate."""
    import numpy as np
    import torch
    import paper_2608_06291_amd as pk
    import workloads
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(dev)
    torch.cuda.set_stream(stream)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    N = n_samples
    cache = {}
    todo = [w for w in FACTOR_WORKLOADS if only is None or ":".join(w) == only]
    if not todo:
        raise SystemExit(f"unknown --factor-only {only}; one of "
                         + ", ".join(":".join(w) for w in FACTOR_WORKLOADS))
    for name, style in todo:
        if name not in cache:
            cache.clear()
            torch.cuda.empty_cache()
            log(f"[factors] generating {name}, N = {N}")
            if name.startswith("mlp"):
                p = workloads.mlp_samples_torch(N, 4096, 14336, 0, dev, "g")
                cache[name] = (p["x"], p["feat"], p["Wd"])
                del p
            else:
                p = workloads.kron_samples_torch(N, 4096, 4096, 0, dev)
                cache[name] = (p["a"], p["b"], None)
            torch.cuda.synchronize()
        a, b, D = cache[name]
        n, m = a.shape[1], b.shape[1]
        iters = int(style[len("shampoo"):] or 1) if style.startswith("shampoo") else 1
        base_style = "shampoo" if iters > 1 else style
        if D is not None:
            run = lambda: pk.mlp_local_factors(a, b, D, base_style, iters=iters)  # noqa: E731
            # D^T D over the dm rows of D, then the two N-sample Grams
            F = _gram_flops(D.shape[0], m) + _gram_flops(N, n) + _gram_flops(N, m)
        else:
            run = lambda: pk.kron_factors(a, b, base_style, iters=iters)  # noqa: E731
            F = _gram_flops(N, n) + _gram_flops(N, m)
        # each later power step adds the two Grams and the two quadratic forms
        # (2 N d^2 flops for the product X M, N d for the fused row sums)
        F = F * iters + (iters - 1) * (2.0 * N * (n * n + m * m) + N * (n + m))
        for _ in range(warmup):
            A, B = run()
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(steps):
            A, B = run()
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / steps
        # the dominant launch pair: the Gram of the wider operand b over N samples
        # (k_gram and its slice reduction; the mask and weights as in the step)
        w = pk.sample_weights(a) if base_style == "shampoo" else None
        M = None
        if D is not None:
            M = pk.gram(D, None, 1.0)
        C = torch.empty((m, m), dtype=torch.float32, device=dev)
        work = torch.empty(pk.gram_workspace_bytes(N, m), dtype=torch.uint8, device=dev)
        pk.gram(b, w, 1.0 / N, M, C, work)
        torch.cuda.synchronize()
        reps = max(2, steps)
        e0.record(stream)
        for _ in range(reps):
            pk.gram(b, w, 1.0 / N, M, C, work)
        e1.record(stream)
        torch.cuda.synchronize()
        g_ms = e0.elapsed_time(e1) / reps
        g_tf = _gram_flops(N, m) / (g_ms * 1e-3) / 1e12
        q_ms = q_tf = None
        if iters > 1:
            # the power steps' quadratic form of the wider operand, timed alone
            wq = torch.empty((N,), dtype=torch.float32, device=dev)
            pk.quadform_weights(b, B, wq)
            torch.cuda.synchronize()
            e0.record(stream)
            for _ in range(reps):
                pk.quadform_weights(b, B, wq)
            e1.record(stream)
            torch.cuda.synchronize()
            q_ms = e0.elapsed_time(e1) / reps
            q_tf = (2.0 * N * m * m + N * m) / (q_ms * 1e-3) / 1e12
            del wq
        # sampled parity: 48 entries of A and B against the fp64 oracle (one
        # power step: the later steps' weights need the whole previous pair,
        # which the oracle cannot form at this size; their parity is tested
        # at smaller sizes)
        import oracle
        h = oracle.hessian
        rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([5000, n, m])))

        def pairs(d):
            pr = [(int(i), int(j)) for i, j in rng.integers(0, d, (40, 2))]
            return pr + [(i, i) for i in rng.integers(0, d, 8).tolist()]

        def cols(X, pr):
            idx = sorted({i for q in pr for i in q})
            sub = X[:, idx].double().cpu().numpy()
            pos = {c: t for t, c in enumerate(idx)}
            return sub, [(pos[i], pos[j]) for i, j in pr]

        def wts(X, c=None):   # Shampoo weights tr(.) of every sample, fp64 on the CPU
            out = np.empty(X.shape[0])
            for k0 in range(0, X.shape[0], 16384):
                blk = X[k0:k0 + 16384].double().cpu().numpy()
                out[k0:k0 + 16384] = h.trace_quad(blk[:, :, None] * (1.0 if c is None else
                                                                      np.sqrt(c)[None, :, None]))
            return out

        pa, pb = pairs(n), pairs(m)
        wA = wB = None
        rel = None
        if base_style == "shampoo" and iters == 1:
            if D is not None:
                Dn = D.double().cpu().numpy()
                wA = wts(b, np.sum(Dn * Dn, axis=0))   # g^T diag(D^T D) g
            else:
                wA = wts(b)
            wB = wts(a)
        if iters == 1:
            sa, qa = cols(a, pa)
            sb, qb = cols(b, pb)
            eA = h.expect_outer_entries(sa, qa, wA)
            eB = h.expect_outer_entries(sb, qb, wB)
            if D is not None:
                sd, qd = cols(D, pb)
                eB = eB * D.shape[0] * h.expect_outer_entries(sd, qd)
            gA = np.array([A[i, j].item() for i, j in pa])
            gB = np.array([B[i, j].item() for i, j in pb])
            rel = float(max(np.max(np.abs(gA - eA) / np.abs(eA).max()),
                            np.max(np.abs(gB - eB) / np.abs(eB).max())))
        cpu = None
        if do_cpu:
            cpu = factors_cpu_baseline(a, b, D, base_style, iters, F, cpu_seconds)
        out = {
            "metric": "Kronecker-factor construction TFLOP/s (App. A), 1 MI355X",
            "value": F / (ms * 1e-3) / 1e12, "unit": "TFLOP/s", "n_gpus": 1, "steps": steps,
            "warmup": warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": "f32", "data": "synthetic",
            "config": {"workload": f"{name}-{style}", "samples": N, "n": n, "m": m,
                       "algorithmic_flops": F, "sampled_max_rel_err": rel},
            "roofline": {"kernel": "k_gram + k_gram_reduce (Gram of the N x %d operand)" % m,
                         "bound": "mfma", "achieved": g_tf, "peak": PEAK_SPLIT,
                         "unit": "TFLOP/s", "frac": g_tf / PEAK_SPLIT,
                         "traffic": measured_traffic("k_gram", f"{name}-{style}",
                                                     ("hessian.hip", "split.h", "common.h")),
                         "launch_ms": g_ms},
            "cpu_baseline": cpu,
        }
        if q_ms is not None:
            out["quadform"] = {"kernel": "k_quadform + k_quadform_reduce (N x %d operand)" % m,
                               "bound": "mfma", "achieved": q_tf, "peak": PEAK_SPLIT,
                               "unit": "TFLOP/s", "frac": q_tf / PEAK_SPLIT, "launch_ms": q_ms}
        print(json.dumps(out), flush=True)
        log(f"[factors] {name} {style}: {ms:.1f} ms/step, {out['value']:.1f} TFLOP/s; "
            f"Gram {g_ms:.1f} ms = {g_tf:.1f} TFLOP/s ({100 * g_tf / PEAK_SPLIT:.0f}% of a "
            f"sixth of the bf16 peak)" + (f"; quadratic form {q_ms:.1f} ms = {q_tf:.1f} TFLOP/s" if q_ms else "")
            + (f"; sampled rel err {rel:.2e}" if rel is not None else ""))
        del A, B, C, work, M, w
    cache.clear()


def factors_cpu_baseline(a, b, D, style, iters, F, seconds):
    """Time the fp64 oracle on the first samples of the same workload
    (K-FAC / Shampoo factors from its per-sample definitions, the MLP-local b
    formed explicitly) and extrapolate linearly in the number of samples."""
    import oracle
    h = oracle.hessian
    N = a.shape[0]
    k = 1
    while True:
        sa = a[:k].double().cpu().numpy()
        sb = b[:k].double().cpu().numpy()
        t0 = time.perf_counter()
        if D is not None:
            h.mlp_local_factors(sa, sb, D.double().cpu().numpy(), style, iters=iters)
        elif style == "kfac":
            h.kfac_factors(sa, sb)
        else:
            h.shampoo_factors(sa, sb, iters=iters)
        t = time.perf_counter() - t0
        if t >= seconds / 4 or k >= N:
            break
        k = min(N, max(k * 2, int(k * seconds / 4 / max(t, 1e-3))))
    t_full = t * N / k
    try:
        from threadpoolctl import threadpool_info
        cores = max([i.get("num_threads", 1) for i in threadpool_info()] + [1])
    except Exception:
        cores = 1
    return dict(value=F / t_full / 1e12, unit="TFLOP/s", cores=cores, kind="oracle",
                sample=f"first {k} of {N} samples of the same workload, {t:.1f} s measured; "
                       f"extrapolated linearly in the sample count",
                s_per_step=t_full, host_cpu=cpu_model())


def quant_bench(steps: int):
    """Quantiser variants on the 4096 x 4096 layer (INT4): the solve with
    per-row symmetric scales against the general path (asymmetric alphabet,
    128-column group scales, per-column factors), and the MSE scale search
    (App. D) per row and per 128-column group.  One JSON line each."""
    import numpy as np
    import torch
    import paper_2608_06291_amd as pk
    import workloads
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(dev)
    torch.cuda.set_stream(stream)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def timed(fn, reps):
        for _ in range(3):   # first call allocates; the rest settle clocks after the previous shape
            fn()
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(reps):
            fn()
        e1.record(stream)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    c = workloads.make(2, seed=0, device="cuda")
    m, n = c["cfg"].m, c["cfg"].n
    W = torch.from_numpy(c["W"]).to(dev)
    f = pk.factor(torch.from_numpy(c["A"]).to(dev), torch.from_numpy(c["B"]).to(dev), c["damp"])
    codes = torch.empty((m, n), dtype=torch.int8, device=dev)
    V = torch.empty((m, n), dtype=torch.float32, device=dev)
    s_row = torch.from_numpy(c["scale"]).to(dev)
    s_grp = pk.mse_scales(W, 4, "asym", group_size=128)
    col = torch.from_numpy(np.random.Generator(np.random.PCG64(5)).uniform(0.75, 1.25, n)
                           .astype(np.float32)).to(dev)
    F = float(m) * n * (m + n)
    rows = []
    for label, kw, sc in (("per-row symmetric", {}, s_row),
                          ("asymmetric, 128-column groups, column factors",
                           dict(alphabet="asym", group_size=128, col_scale=col), s_grp)):
        ms = timed(lambda: pk.solve(W, f, 4, sc, codes=codes, V=V, **kw), steps)
        rows.append(dict(kind="solve", quantiser=label, ms=ms, tflops=F / ms / 1e9))
    for g in (0, 128):
        ms = timed(lambda: pk.mse_scales(W, 4, "sym", group_size=g), steps)
        # candidates x entries evaluated (one division, rint, product, fp64 square-add each)
        rows.append(dict(kind="mse_scales", group_size=g, ms=ms,
                         evaluations_per_s=101.0 * m * n / (ms * 1e-3)))
    f.close()
    for r in rows:
        r.update(workload="attn-proj-4096x4096", bits=4)
        print(json.dumps(r), flush=True)
        log(f"[quant] {r}")


def factorise_bench(dims, steps: int):
    """bakron_factor alone on factor pairs (damping, reverse Cholesky,
    triangular inverse and packing; A and B concurrently), inputs the AR(1)
    Toeplitz matrices rho^|i-j| (rho 0.5 for A, 0.2 for B) resident in HBM.
    Each entry of `dims` is d (A and B both d x d) or n:m (A n x n, B m x m,
    as in a layer's factor pair).  Counted fp64 work 2 d^3 / 3 per factor
    (d^3 / 3 for its Cholesky and d^3 / 3 for its inverse).  One JSON line per
    entry, with the median of `steps` calls after one warm-up call."""
    import torch
    import paper_2608_06291_amd as pk
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(dev)
    torch.cuda.set_stream(stream)

    def ar1(d, rho):
        i = torch.arange(d, device=dev, dtype=torch.float32)
        return rho ** (i[:, None] - i[None, :]).abs()

    for spec in dims:
        n, m = (int(x) for x in spec.split(":")) if ":" in spec else (int(spec), int(spec))
        A, B = ar1(n, 0.5), ar1(m, 0.2)
        pk.factor(A, B, 0.01).close()            # warm-up: scratch allocation, clocks
        torch.cuda.synchronize()
        ts = []
        for _ in range(steps):
            t0 = time.perf_counter()
            f = pk.factor(A, B, 0.01)
            torch.cuda.synchronize()
            ts.append((time.perf_counter() - t0) * 1e3)
            f.close()
        ms = sorted(ts)[len(ts) // 2]
        flops = 2.0 * (n ** 3 + m ** 3) / 3.0
        tf = flops / (ms * 1e-3) / 1e12
        print(json.dumps({"metric": "bakron_factor ms (A n x n and B m x m, concurrently)",
                          "value": ms, "unit": "ms", "higher_is_better": False, "n": n, "m": m,
                          "steps": steps, "counted_fp64_tflop": flops / 1e12,
                          "fp64_tflops": tf, "frac_fp64_mfma_peak": tf / PEAK_FP64_MFMA,
                          "data": "synthetic"}), flush=True)
        del A, B
        torch.cuda.empty_cache()


def flow_bench(L: int, d: int, N: int, style: str):
    """Sec. 5's recursive flow over a stack of L square layers (width d, N
    calibration samples, SiLU): per phase, the summed device time of the
    model's forward/backward, the Kronecker factors, the factorisation, the
    scale search and the BaKron solve, plus the layer-evaluation counts.  One
    JSON line."""
    import time as _t
    import torch
    import paper_2608_06291_amd as pk
    from paper_2608_06291_amd import flow
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(dev)
    torch.cuda.set_stream(stream)
    gen = torch.Generator(device=dev).manual_seed(11)
    W = [(torch.randn((d, d), generator=gen, device=dev) * (2.0 / d) ** 0.5) for _ in range(L)]
    import workloads
    x0 = workloads.ar1_samples_torch(N, d, 0.5, gen, dev, spike_rank=4, norm_sigma=0.5)
    g_out = torch.randn((N, d), generator=gen, device=dev)
    torch.cuda.synchronize()
    phase = {k: 0.0 for k in ("model", "factors", "factorise", "scales", "solve")}

    class Timed(flow.LayerStack):
        def forward_layer(self, l, x, stats):
            t0 = _tick()
            out = super().forward_layer(l, x, stats)
            phase["model"] += _tock(t0)
            return out

        def backward_layer(self, l, y, g, stats):
            t0 = _tick()
            out = super().backward_layer(l, y, g, stats)
            phase["model"] += _tock(t0)
            return out

    def _tick():
        e = torch.cuda.Event(enable_timing=True)
        e.record(stream)
        return e

    def _tock(e):
        e2 = torch.cuda.Event(enable_timing=True)
        e2.record(stream)
        e2.synchronize()
        return e.elapsed_time(e2)

    stack = Timed(W)
    iters = int(style[len("shampoo"):] or 1) if style.startswith("shampoo") else 1
    base = "shampoo" if style.startswith("shampoo") else "kfac"

    def step(l, a, b):
        t0 = _tick()
        A, B = pk.kron_factors(a, b, base, iters=iters)
        phase["factors"] += _tock(t0)
        t0 = _tick()
        f = pk.factor(A, B, 0.5)
        phase["factorise"] += _tock(t0)
        t0 = _tick()
        sc = pk.mse_scales(stack.W[l], 3)
        phase["scales"] += _tock(t0)
        t0 = _tick()
        pk.solve(stack.W[l], f, 3, sc)
        phase["solve"] += _tock(t0)
        f.close()

    t0 = _t.perf_counter()
    st = flow.recursive_flow(stack, x0, g_out, step)
    torch.cuda.synchronize()
    wall = _t.perf_counter() - t0
    total = sum(phase.values())
    out = dict(kind="flow", layers=L, width=d, samples=N, factors=style, wall_s=wall,
               phase_ms=phase, core_share=phase["solve"] / total,
               layer_forwards=st.layer_forwards, layer_backwards=st.layer_backwards,
               peak_live_pairs=st.peak_live_pairs)
    print(json.dumps(out), flush=True)
    log(f"[flow] {out}")


def main():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", type=int, default=5)
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--profile-steps", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=15.0,
                    help="with --factors: seconds of oracle work for its CPU baseline")
    ap.add_argument("--cpu-rows", type=int, default=12288,
                    help="rows of the layer sample the CPU baseline solves (oracle, Alg. 5)")
    ap.add_argument("--cpu-full", action="store_true",
                    help="only time the fp64 oracle (Alg. 5) on the whole configured layer on the "
                         "host cores (no GPU work) and exit")
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="only run a plain device-to-device copy of this many MiB (10 times) and "
                         "exit: the reference for scaling rocprofv3 FETCH_SIZE/WRITE_SIZE counters")
    ap.add_argument("--table3", action="store_true",
                    help="only run the runtime comparison on the paper's Table 3 shapes (GPTQ, BaKron, "
                         "BaKron-antidiagonal) and exit; one JSON line per shape")
    ap.add_argument("--table3-max-antidiag-elems", type=int, default=1 << 27,
                    help="skip BaKron-antidiagonal (quartic work) above this many matrix entries")
    ap.add_argument("--factors", action="store_true",
                    help="only run the Kronecker-factor construction workloads (App. A: K-FAC and "
                         "single-step Shampoo, global and MLP-local) and exit; one JSON line each")
    ap.add_argument("--quant", action="store_true",
                    help="only time the quantiser variants and the MSE scale search on the "
                         "4096 x 4096 layer and exit")
    ap.add_argument("--factorise", default=None, metavar="d|n:m[,...]",
                    help="time bakron_factor alone on factor pairs, d x d both or A n x n and "
                         "B m x m (damping, reverse Cholesky, triangular inverse)")
    ap.add_argument("--flow", default=None, metavar="L,d,N[,style]",
                    help="only run the recursive backprop flow (Sec. 5) over L layers of width d "
                         "with N samples (style kfac or shampooK) and exit")
    ap.add_argument("--factor-only", default=None,
                    help="with --factors: run only this workload:style (e.g. global-4096x4096:kfac)")
    ap.add_argument("--factor-samples", type=int, default=FACTOR_N,
                    help="calibration samples for --factors (default 256 x 2048)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: --gpus {args.gpus} is not supported: the BaKron solve runs on one "
              "GPU (multi-GPU sharding is a design note only); run with --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    if args.table3:
        table3(args.table3_max_antidiag_elems)
        return

    if args.quant:
        quant_bench(args.steps)
        return

    if args.factorise:
        factorise_bench(args.factorise.split(","), max(args.steps, 1))
        return
    if args.flow:
        parts = args.flow.split(",")
        flow_bench(int(parts[0]), int(parts[1]), int(parts[2]), parts[3] if len(parts) > 3 else "kfac")
        return

    if args.factors:
        factors_bench(args.steps, args.warmup, args.factor_samples, args.cpu_seconds,
                      not args.no_cpu_baseline, args.factor_only)
        return

    if args.copy_calibration_mib > 0:
        nbytes = args.copy_calibration_mib << 20
        src = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda:0")
        dst = torch.empty_like(src)
        for _ in range(10):
            dst.copy_(src)
        torch.cuda.synchronize()
        log(f"[bench] copied {nbytes} bytes 10 times")
        return

    import paper_2608_06291_amd as pk
    import workloads

    if args.cpu_full:
        log(f"[bench] generating config {args.config} (seed {args.seed})")
        c = workloads.make(args.config, seed=args.seed, device="cuda")
        out = cpu_full(c)
        out["workload"] = c["cfg"].name
        print(json.dumps(out), flush=True)
        return

    dev = torch.device("cuda:0")
    log(f"[bench] generating config {args.config} (seed {args.seed})")
    c = workloads.make(args.config, seed=args.seed, device="cuda")
    cfg = c["cfg"]
    m, n = cfg.m, cfg.n
    A = torch.from_numpy(c["A"]).to(dev)
    B = torch.from_numpy(c["B"]).to(dev)
    W = torch.from_numpy(c["W"]).to(dev)
    s = torch.from_numpy(c["scale"]).to(dev)
    codes = torch.empty((m, n), dtype=torch.int8, device=dev)
    V = torch.empty((m, n), dtype=torch.float32, device=dev)
    torch.cuda.synchronize()

    # a stream of its own: on the legacy default stream the solver keeps every
    # launch on that stream (the default stream synchronises implicitly with
    # the CU-restricted streams that overlap node pushes with segment launches)
    stream = torch.cuda.Stream(dev)
    torch.cuda.set_stream(stream)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    f = pk.factor(A, B, c["damp"])
    e1.record(stream)
    torch.cuda.synchronize()
    factor_ms = e0.elapsed_time(e1)
    log(f"[bench] factor {factor_ms:.1f} ms")

    for _ in range(args.warmup):
        pk.solve(W, f, c["bits"], s, codes=codes, V=V)
    torch.cuda.synchronize()
    log(f"[bench] warmup {args.warmup} done")

    t0 = time.perf_counter()
    e0.record(stream)
    for _ in range(args.steps):
        pk.solve(W, f, c["bits"], s, codes=codes, V=V)
    e1.record(stream)
    torch.cuda.synchronize()
    wall_ms = (time.perf_counter() - t0) * 1e3
    total_ms = e0.elapsed_time(e1)
    ms = total_ms / args.steps
    F = float(m) * n * (m + n)
    tflops = F / (ms * 1e-3) / 1e12
    log(f"[bench] {args.steps} steps: {ms:.3f} ms/layer, {tflops:.2f} counted TFLOP/s "
        f"(wall {wall_ms / args.steps:.3f} ms/step)")
    # the timed solves are valid only if no tile-ordering wait gave up (the
    # record is sticky over all solves since the last check)
    if not f.check():
        log("[bench] FAILED: a tile-ordering wait of a timed solve gave up; no result line")
        sys.exit(3)
    validation = validate_outputs(pk, f, W, s, c["bits"], codes, V)
    log(f"[bench] outputs validated: {validation}")

    # per-kernel durations: the same solve with HIP event pairs around each launch
    f.profile(True)
    agg = {k: dict(ms=0.0, launches=0, flops=0.0, mfma_flops=0.0) for k in (*f.PROFILE_CLASSES, "node_fp32")}
    prof_ms = 0.0
    for _ in range(args.profile_steps):
        e0.record(stream)
        pk.solve(W, f, c["bits"], s, codes=codes, V=V)
        e1.record(stream)
        torch.cuda.synchronize()
        prof_ms += e0.elapsed_time(e1)
        st = dict(f.profile_read(), node_fp32=f.profile_read_node_fp32())
        for k in agg:
            for q in agg[k]:
                agg[k][q] += st[k][q]
    f.profile(False)
    P = max(args.profile_steps, 1)
    kern = {}
    for k, a in agg.items():
        L = max(a["launches"], 1)
        kern[k] = dict(launches_per_step=a["launches"] / P, ms_per_step=a["ms"] / P,
                       avg_launch_us=a["ms"] / L * 1e3, flops_per_step=a["flops"] / P,
                       mfma_flops_per_step=a["mfma_flops"] / P)
    node, seg = kern["node"], kern["segment"]
    tf = {k: agg[k]["flops"] / max(agg[k]["ms"], 1e-12) / 1e9 for k in agg}
    mf = {k: agg[k]["mfma_flops"] / max(agg[k]["ms"], 1e-12) / 1e9 for k in agg}
    for k in ("segment", "node", "node_fp32"):
        kern[k]["achieved_tflops"] = tf[k]
        kern[k]["mfma_executed_tflops"] = mf[k]
    # the pushes of short nodes run on fp32 MFMA, the others as split products:
    # each priced against its own peak (time at the peaks over time taken)
    split = {q: agg["node"][q] - agg["node_fp32"][q] for q in agg["node"]}
    split_tf = split["flops"] / max(split["ms"], 1e-12) / 1e9
    node["mfma_utilisation"] = (split["mfma_flops"] / PEAK_SPLIT + agg["node_fp32"]["mfma_flops"] / PEAK_FP32_MFMA) \
        / max(agg["node"]["ms"], 1e-12) / 1e9
    node["split"] = dict(launches_per_step=split["launches"] / P, ms_per_step=split["ms"] / P,
                         achieved_tflops=split_tf if split["launches"] else None)
    # the segment launches carry the sequential chain: per tile anti-diagonal
    n_diag = (m + 31) // 32 + (n + 31) // 32 - 1
    seg["us_per_tile_diagonal"] = seg["ms_per_step"] * 1e3 / n_diag
    # and per sequential step of the method (one element anti-diagonal, m + n - 1)
    seg["us_per_element_diagonal"] = seg["ms_per_step"] * 1e3 / (m + n - 1)
    # wavefront bandwidth: HBM bytes per launch (rocprofv3 counters, while the
    # kernel source is unchanged) over the live average launch duration
    seg_traffic = measured_traffic("k_seg", cfg.name)
    if seg_traffic is not None and seg["avg_launch_us"] > 0:
        seg["hbm_gbps"] = seg_traffic / (seg["avg_launch_us"] * 1e-6) / 1e9
        seg["hbm_frac"] = seg["hbm_gbps"] / PEAK_HBM
    node_traffic = measured_traffic("k_node", cfg.name)   # of the split pushes
    if node_traffic is not None and split["launches"]:
        node["split"]["hbm_gbps"] = node_traffic * split["launches"] / (split["ms"] * 1e-3) / 1e9
    # dominant kernel class: the one with the larger share of the step.  The
    # segment launches are fp32 MFMA work (94% of their counted flops are the
    # near-field pulls on the matrix cores); the node pushes, short ones aside,
    # multiply fp32 operands as six bf16 products, priced against a sixth of the
    # bf16 peak; where the short ones (fp32 MFMA) take more of the step, they are
    # the kernel that is priced.
    dominant = "segment" if seg["ms_per_step"] >= node["ms_per_step"] else "node"
    if dominant == "segment":
        roof = dict(kernel="k_seg (persistent tile-wavefront rounding with near-field pulls)",
                    bound="mfma", achieved=tf["segment"], peak=PEAK_FP32_MFMA, unit="TFLOP/s",
                    frac=tf["segment"] / PEAK_FP32_MFMA, traffic=seg_traffic)
    elif split["ms"] >= agg["node_fp32"]["ms"]:
        roof = dict(kernel="k_node (divide-and-conquer band push), split bf16 MFMA", bound="mfma",
                    achieved=split_tf, peak=PEAK_SPLIT, unit="TFLOP/s",
                    frac=split_tf / PEAK_SPLIT, traffic=node_traffic)
    else:
        roof = dict(kernel="k_node32 (band push of short nodes), fp32 MFMA", bound="mfma",
                    achieved=tf["node_fp32"], peak=PEAK_FP32_MFMA, unit="TFLOP/s",
                    frac=tf["node_fp32"] / PEAK_FP32_MFMA, traffic=None)
    log(f"[bench] kernels: {json.dumps(kern)}")

    cpu = None
    if not args.no_cpu_baseline:
        log(f"[bench] cpu baseline: oracle Alg. 5 on a {args.cpu_rows}-row sample")
        cpu = cpu_baseline(c, args.cpu_rows)
        log(f"[bench] cpu baseline {cpu['value'] * 1e3:.2f} counted GFLOP/s in "
            f"{cpu['sample_seconds']:.1f} s ({cpu['cores']} BLAS threads); "
            f"{cpu['ms_per_layer']:.0f} ms/layer by counted work")

    vs = None
    if (m, n) == (4096, 4096):
        vs = tflops / (F / PAPER_4096_S / 1e12)
    out = {
        "metric": METRIC, "value": tflops, "unit": "TFLOP/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": vs,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": cfg.name, "m": m, "n": n, "bits": cfg.bits, "damp": cfg.damp,
                   "seed": args.seed, "counted_flops": F, "ms_per_layer": ms,
                   "frac_fp32_mfma_peak": tflops / PEAK_FP32_MFMA, "factor_ms": factor_ms,
                   "end_to_end_ms": factor_ms + ms, "profiled_ms_per_step": prof_ms / P,
                   "validation": validation, "device": device_peak(),
                   "vs_baseline_note": ("paper Table 3, 4096x4096 in 0.288 s on one RTX PRO 6000 "
                                        "fp32 (other hardware, unspecified matrix contents)")
                   if vs is not None else None},
        "roofline": roof,
        "kernels": kern,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)
    f.close()


if __name__ == "__main__":
    main()
