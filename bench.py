#!/usr/bin/env python3
"""GRAPE forward + gradient throughput on one MI355X.

One step = one pass of the whole hot path (plan, slice propagators, forward
and backward scans, fidelity, adjoint gradient) over a batch of B independent
6-qubit Ising problems (d = 64, m = 12 controls, N = 2000 slices,
dt = 0.002, u ~ N(0, 0.5), Haar-random targets; seeded copies 1..B), with
all inputs resident in HBM.  value = slice-steps per second of the headline
precision; the plain FP64 path is timed beside it.  Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "GRAPE slice-steps/s (fwd+grad, d=64) vs plain FP64; p50/p99 request latency"
# dense matrix-core peaks of the adjoint kernel's products: FP64, and FP16 in FP32 and
# split BF16 (Hermitian Hamiltonians)
PEAK_TFLOPS = {"fp64": 78.6, "fp32": 2500.0, "bf16x3": 2500.0}
CFG = 3  # 6-qubit Ising chain, d = 64
WORKLOADS = {2: "4-qubit Heisenberg chain", 3: "6-qubit Ising chain", 4: "7-qubit Heisenberg chain"}


def permutation_runs(Hc: np.ndarray, group: int = 4):
    """For controls with one nonzero per row whose columns form a permutation
    (Pauli strings), the number of dot-product sets the FP32 adjoint's sampled
    last step forms per column: controls in one group of `group` with the
    previous control's columns share one.  None when some control is not such
    a permutation (the adjoint then takes its last two products)."""
    d = Hc.shape[1]
    cols = []
    for H in Hc:
        nz = H != 0
        if (nz.sum(axis=1) > 1).any():
            return None
        col = np.where(nz.any(axis=1), nz.argmax(axis=1), np.arange(d))
        if len(set(col.tolist())) != d:
            return None
        cols.append(col)
    runs = 0
    for j in range(len(cols)):
        if j % group == 0 or not np.array_equal(cols[j], cols[j - 1]):
            runs += 1
    return runs


def slice_flops(plan: np.ndarray, d: int, m: int, prec: str, runs=None) -> dict:
    """MFMA flops per stage of the block form as it was counted for Hermitian
    problems (hermitian_flops takes its FP64 adjoint at d > 64) for slices with plan
    rows (s, q, qb), and the adjoint's count in the conventional 8 d^3 per
    complex product ("adjoint_8d3").

    Complex d x d products per slice: expm q - 1 + s (Horner; at d > 64 in
    FP32 Paterson-Stockmeyer, 2 + floor((q - 3) / 2) + s for q >= 3); scans
    one per direction; adjoint 6 + 3 floor((qb - 3) / 2) + 3 s (one for W,
    three for the square of the block, three per Paterson-Stockmeyer step
    with a matrix digit, two for the last step's top-right block, three per
    squaring), one fewer where the FP32 expm keeps X^2 for the FP32 adjoint
    (d > 16, q >= 2), and two fewer where the FP32 adjoint samples its last step
    (d > 16, at d = 128 with m <= 16, s = 0, `runs` not None: permutation
    controls), which costs
    16 d^2 runs real flops on the vector ALU instead ("adjoint_valu").
    A product costs 8 d^3 real flops in the four-product form and 6 d^3 in
    the three-product (Gauss) form.  FP32 and FP64 use the latter in every
    stage at 32 <= d <= 64, and FP32 also in the expm and adjoint at d = 128.
    The split-BF16 path runs its adjoint on three BF16 products per real one,
    24 d^3 BF16 flops per complex product, and its expm and scans in FP32
    (three-product form).  Assembly and the gradient inner products run on
    the vector ALU and are not counted."""
    s, q, qb = plan[:, 0].astype(np.float64), plan[:, 1].astype(np.float64), plan[:, 2].astype(np.float64)
    G4, G3 = 8.0 * d ** 3, 6.0 * d ** 3
    mid = prec in ("fp32", "fp64", "bf16x3") and 32 <= d <= 64
    big32 = prec == "fp32" and d > 64
    g_adj = 24.0 * d ** 3 if prec == "bf16x3" else (G3 if (mid or big32) else G4)
    g_expm = G3 if (mid or big32) else G4
    g_scan = G3 if mid else G4
    if prec == "fp32" and d > 64:
        n_exp = np.where(q < 2, 0, np.where(q == 2, 1, 2 + (q - 3) // 2)) + s
    else:
        n_exp = q - 1 + s
    keep_x2 = prec == "fp32" and d > 16
    n_adj = 6 + 3 * np.maximum(0, (qb - 3) // 2) + 3 * s - (keep_x2 * (q >= 2))
    on = prec == "fp32" and d > 16 and (d <= 64 or m <= 16) and runs is not None
    sampled = (s == 0) if on else np.zeros_like(s, dtype=bool)
    n_adj = n_adj - 2 * sampled
    valu = float((16.0 * d * d * (runs or 0) * sampled).sum())
    return {"expm": float((g_expm * n_exp).sum()), "scan": float(2 * g_scan * len(s)),
            "adjoint": float((g_adj * n_adj).sum()), "adjoint_8d3": float((8.0 * d ** 3 * n_adj).sum()),
            "adjoint_valu": valu}


def series_orders(problems, plan: np.ndarray, prec: str, d: int = 64) -> np.ndarray:
    """Orders of the commutator series per slice: the least n with
    x^(n+1)/(n+1)! <= ur (1 - x/(n+2)), x = 2 theta / 2^s, as the plan picks them.
    At d > 64 Horner's rule also needs the n at which the remainder of the sum of
    x^n/(n+1)! is met, and takes two products at least."""
    ur = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    n1 = lambda H: np.abs(H).sum(axis=0).max()
    theta = np.concatenate([p.dt * (n1(p.H0) + np.abs(p.u).T @ np.array([n1(H) for H in p.Hc])) for p in problems])
    x = 2 * theta / 2.0 ** plan[:, 0]

    def least(t):  # n from 1 while the term that starts at t stays above the bound
        n = np.ones(len(x))
        for k in range(1, 30):
            on = (t > ur * (1 - x / (k + 2))) & (n == k)
            n[on] = k + 1
            t = t * x / (k + 2)
        return n

    n = least(x * x / 2)
    return n if d <= 64 else np.maximum(np.maximum(n, least(x / 2)), 2)


def series_flops(problems, plan: np.ndarray, d: int, prec: str) -> dict:
    """Matrix-core flops of the segmented Hermitian path (d <= 64, and FP32 at d = 128)
    over all slices: the exponential's products (its form by q at d <= 64,
    Paterson-Stockmeyer in X^2 and 128), its s squarings, one chain product and the
    series' one product per order; with s > 0 also the gradient's doublings, two
    products for Z and one squaring each, and two for Y (at d <= 64 the last squaring is
    the forward pass's; at d = 128 the exponential is formed again).  FP32 (and split BF16,
    which runs the same kernels) takes three FP16 products per real one, 24 d^3 flops
    per complex product, and its chain in FP32 by the three-product form, 6 d^3 (at
    d = 16 by the four-product form, 8 d^3); FP64 takes three products per complex one,
    at d = 16 four in its chain."""
    s, q, m = plan[:, 0], plan[:, 1], series_orders(problems, plan, prec, d)
    if d > 64:
        n_exp = np.where(q < 2, 0, np.where(q == 2, 1, 2 + (q - 3) // 2))
        n_adj = m - (s > 0) + np.where(s > 0, n_exp + 3 * s + 2, 0)
    else:
        n_exp = np.where(q <= 3, q - 1, np.where(q == 4, 2, np.where(q <= 8, 3, 2 + (q - 1) // 3)))
        n_adj = m + np.where(s > 0, 3 * s - (d > 16) + 2, 0)
    g = 6.0 * d ** 3 if prec == "fp64" else 24.0 * d ** 3
    chain = 8.0 if d <= 16 else 6.0
    return {"expm": float(g * (n_exp + s).sum()), "chain": chain * d ** 3 * len(q), "adjoint": float(g * n_adj.sum()),
            "adjoint_8d3": float(8.0 * d ** 3 * n_adj.sum())}


def hermitian_flops(problems, plan: np.ndarray, d: int, m: int, prec: str) -> dict:
    """Matrix-core flops of a gradient of Hermitian problems, and the kernel of its
    adjoint stage: segments, but the block form in FP64 at d > 64, whose exponential
    runs Paterson-Stockmeyer."""
    if d <= 64 or prec != "fp64":
        return dict(series_flops(problems, plan, d, prec), kernel="k_seg_grad" if d <= 64 else "k_seg_grad128")
    s, q = plan[:, 0], plan[:, 1]
    n_exp = np.where(q < 2, 0, np.where(q == 2, 1, 2 + (q - 3) // 2)) + s
    return dict(slice_flops(plan, d, m, prec), expm=float(8.0 * d ** 3 * n_exp.sum()), kernel="k_adjoint128")


def worst_rel_grad_err(grad, ref):
    """max over the batch of max|grad_b - ref_b| / max|ref_b|: each problem
    against its own gradient scale, as the parity tests gate it."""
    num = (grad - ref).abs().flatten(1).max(dim=1).values
    den = ref.abs().flatten(1).max(dim=1).values
    return float((num / den).max().item())


def time_runner(qoc, torch, runner, batch, steps, warmup):
    """Times `steps` steps (events between steps only), then runs as many
    again with libqoc's per-stage events for the stage breakdown, so that
    those events do not add to the timed steps."""
    F = torch.empty(batch.B, dtype=torch.float64, device="cuda")
    grad = torch.empty((batch.B, batch.m, batch.N), dtype=torch.float64, device="cuda")
    for _ in range(warmup):
        runner.gradient(batch, F, grad)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ev[0].record(stream)
    for i in range(steps):
        runner.gradient(batch, F, grad)
        ev[i + 1].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    qoc.stage_times()
    qoc.stage_timing(True)
    for _ in range(steps):
        runner.gradient(batch, F, grad)
    torch.cuda.synchronize()
    qoc.stage_timing(False)
    stages = qoc.stage_times()
    ms = ev[0].elapsed_time(ev[-1]) / steps
    per = np.array([ev[i].elapsed_time(ev[i + 1]) for i in range(steps)])
    lat = {"p50_ms": round(float(np.percentile(per, 50)), 4), "p99_ms": round(float(np.percentile(per, 99)), 4),
           "mean_ms": round(float(per.mean()), 4)}
    return {"ms_per_step": ms, "wall_s": wall, "stages": stages, "F": F.cpu().numpy(), "grad": grad,
            "step_time": lat}


def measured_traffic(kernel_avg_ms):
    """HBM bytes per launch of the gradient kernel from the committed rocprofv3
    counter summary (FETCH_SIZE and WRITE_SIZE, each scaled by its reading for a
    plain 1 GiB copy), or None when the kernel sources changed since then."""
    import hashlib

    path = os.path.join(ROOT, "profiles", "k_seg_grad_counters.json")
    csrc = os.path.join(ROOT, "paper_2208_12187_amd", "csrc")
    try:
        with open(path) as f:
            z = json.load(f)
        src = b"".join(open(os.path.join(csrc, n), "rb").read() for n in sorted(os.listdir(csrc)))
    except OSError:
        return None
    if hashlib.sha256(src).hexdigest() != z.get("csrc_sha256"):
        return None
    return (z["fetch_kib"] * z["fetch_scale"] + z["write_kib"] * z["write_scale"]) * 1024.0


def serving_leg(n_requests):
    """Request latency through the continuous-batching engine: the serving
    workload (d from {2, ..., 128} with its weights, N ~ U{100..2000},
    2 log2(d) controls, FP32, seeded trace 5) offered all at once to measure
    capacity, then replayed with Poisson arrivals at 70% of that capacity,
    batched and again one request at a time on the same arrival times.

    It runs in a child process that does not load torch, as a serving
    process would (started before this process loads the GPU runtime): the
    engine keeps one stream per padded dimension (four),
    and HIP backs a process's streams with four hardware queues by default.
    In this process torch's stream takes one of them, two of the engine's
    streams then share a queue, and the small-d ticks wait behind the d = 128
    ones (measured: small-d p50 about 5 ms instead of 0.5 ms)."""
    import subprocess

    cmd = [sys.executable, "-m", "paper_2208_12187_amd.serve", "--requests", str(n_requests)]
    r = subprocess.run(cmd, cwd=ROOT, stdout=subprocess.PIPE, stderr=None, text=True, timeout=600)
    if r.returncode != 0:
        raise RuntimeError(f"serving benchmark failed with status {r.returncode}")
    out = json.loads(r.stdout.strip().splitlines()[-1])
    out["process"] = "child process without torch"
    return out


def state_flops(plan, d, m):
    """VALU flops per slice of the state gradient kernel (row-table controls):
    2 Qp matrix-vector products of H0 (8 d^2 each) with the control terms
    (8 m d each), Qp = max(q, qb - 1), and the bilinear forms a_i^dag Hc[j] b_l
    (per control and row about 2 qb (qb + 1) + 16 qb)."""
    q, qb = plan[:, 1].astype(np.float64), plan[:, 2].astype(np.float64)
    Qp = np.maximum(q, qb - 1)
    return float((2 * Qp * (8.0 * d * d + 8.0 * m * d) + m * d * (2 * qb * (qb + 1) + 16 * qb)).sum())


def state_leg(qoc, torch, steps, warmup, B=32):
    """State-to-state transfer on the configuration-3 system (d = 64, m = 12,
    N = 2000): |0...0> to a Haar state, a batch of B, FP32 and FP64."""
    from workloads import make_state_batch

    probs = make_state_batch(3, B)
    p0 = probs[0]
    batch = qoc.StateBatch.from_problems(probs)
    out = {"workload": f"6-qubit Ising chain state transfer, d={p0.d}, m={p0.m}, N={p0.N}, batch of {B}"}
    F = torch.empty(B, dtype=torch.float64, device="cuda")
    grad = torch.empty((B, p0.m, p0.N), dtype=torch.float64, device="cuda")
    res = {}
    for prec in ("fp32", "fp64"):
        r = qoc.StateRunner(B, p0.d, p0.m, p0.N, prec)
        for _ in range(warmup):
            r.gradient(batch, F, grad)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(steps):
            r.gradient(batch, F, grad)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / steps
        qoc.stage_times()
        qoc.stage_timing(True)
        for _ in range(steps):
            r.gradient(batch, F, grad)
        torch.cuda.synchronize()
        qoc.stage_timing(False)
        st = qoc.stage_times()
        plan = np.concatenate([qoc.slice_plan(p.H0, p.Hc, p.u, p.dt, prec, True) for p in probs])
        g_ms = st["state_grad"][0] / max(st["state_grad"][1], 1)
        fl = state_flops(plan, p0.d, p0.m)
        res[prec] = (F.cpu().numpy().copy(), grad.cpu().numpy().copy())
        out[prec] = {"value": round(B * p0.N / (ms / 1e3), 1), "unit": "slice-steps/s", "ms_per_step": round(ms, 4),
                     "stages_ms": {k: round(v[0] / max(v[1], 1), 4) for k, v in st.items() if v[1]},
                     "state_grad_roofline": {"bound": "alu", "achieved": round(fl / (g_ms / 1e3) / 1e12, 2),
                                             "peak": 78.6, "unit": "TFLOP/s",
                                             "frac": round(fl / (g_ms / 1e3) / 1e12 / 78.6, 4)}}
        del r
    (F32, g32), (F64, g64) = res["fp32"], res["fp64"]
    out["max_abs_dF_fp32_vs_fp64"] = float(np.max(np.abs(F32 - F64)))
    out["grad_err_fp32_vs_fp64"] = float(np.max(np.abs(g32 - g64).reshape(B, -1).max(1)
                                                / np.abs(g64).reshape(B, -1).max(1)))
    return out


def lindblad_leg(qoc, torch, steps, warmup, B=16, nq=3, N=1000):
    """Open-system GRAPE (general generators in Liouville space): B open
    Heisenberg chains of nq qubits with amplitude damping and dephasing on every
    qubit, Liouville dimension 4^nq, N slices, FP32 and FP64."""
    from paper_2208_12187_amd import lindblad
    from workloads import make_lindblad

    probs = [make_lindblad(nq, N, dt=0.02, seed=b) for b in range(B)]
    Gs = [lindblad.liouvillian(p.H0, p.Hc, p.Ls) for p in probs]
    c128 = lambda xs: torch.from_numpy(np.stack(xs)).to("cuda")
    batch = qoc.Batch(c128([g[0] for g in Gs]), c128([g[1] for g in Gs]),
                      torch.from_numpy(np.stack([p.u for p in probs])).to("cuda"), probs[0].dt,
                      c128([lindblad.target_superoperator(p.V) for p in probs]))
    D, m = batch.d, batch.m
    out = {"workload": f"{nq}-qubit open Heisenberg chain (damping + dephasing), Liouville d={D}, m={m}, N={N}, "
                       f"batch of {B}"}
    F = torch.empty(B, dtype=torch.float64, device="cuda")
    grad = torch.empty((B, m, N), dtype=torch.float64, device="cuda")
    res = {}
    for prec in ("fp32", "fp64"):
        r = qoc.Runner(B, D, m, N, prec, generators=True)
        for _ in range(warmup):
            r.gradient(batch, F, grad)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(steps):
            r.gradient(batch, F, grad)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / steps
        res[prec] = (F.cpu().numpy().copy(), grad.cpu().numpy().copy())
        out[prec] = {"value": round(B * N / (ms / 1e3), 1), "unit": "slice-steps/s", "ms_per_step": round(ms, 4)}
        del r
    (F32, g32), (F64, g64) = res["fp32"], res["fp64"]
    out["max_abs_dF_fp32_vs_fp64"] = float(np.max(np.abs(F32 - F64)))
    out["grad_err_fp32_vs_fp64"] = float(np.max(np.abs(g32 - g64).reshape(B, -1).max(1)
                                                / np.abs(g64).reshape(B, -1).max(1)))
    return out


def trm_leg(max_iter=60):
    """The paper's trust-region method on the GRAPE residual of configuration
    2 (d = 16, m = 8, N = 1000: 512 residuals, 8001 parameters), FP64."""
    from paper_2208_12187_amd import trm
    from workloads import make_config

    p = make_config(2)
    _, _, info = trm.trm_grape(p, "fp64", max_iter=max_iter)
    it = len(info["steps"])
    return {"workload": "4-qubit Heisenberg chain, d=16, m=8, N=1000, FP64; residual 2 d^2 = 512, parameters m N + 1",
            "iterations": it, "accepted": sum(1 for s in info["steps"] if s[3]), "reason": info["reason"],
            "F_start": info["F"][0], "F_end": info["F"][-1], "seconds": round(info["seconds"], 3),
            "jacobian_s": round(info["jac_s"], 3), "svd_s": round(info["svd_s"], 3),
            "ms_per_iteration": round(1e3 * info["seconds"] / max(it, 1), 2)}


def cpu_baseline():
    """The CPU oracle on one full configuration-3 problem (N = 2000 slices,
    the first problem of the benchmark batch), with the BLAS thread pools at
    their default size and again at one thread.  Returns (baseline, one-thread
    baseline, oracle result)."""
    import oracle
    from threadpoolctl import threadpool_info, threadpool_limits
    from workloads import make_config

    threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    p = make_config(CFG, copy=1)

    def median3():
        ts = []
        for _ in range(3):
            t0 = time.perf_counter()
            r = oracle.grape_ref(p)
            ts.append(time.perf_counter() - t0)
        return float(np.median(ts)), r

    dt, ref = median3()
    with threadpool_limits(1):
        dt1, _ = median3()
    model = ""
    try:
        with open("/proc/cpuinfo") as f:
            model = next((l.split(":", 1)[1].strip() for l in f if l.startswith("model name")), "")
    except OSError:
        pass
    sample = f"one configuration-3 problem (d=64, m=12, N={p.N}) fwd+grad, median of 3"
    return ({"value": p.N / dt, "unit": "slice-steps/s", "cores": int(threads), "kind": "oracle",
             "sample": f"{sample}: {dt:.2f} s", "cpu": model},
            {"value": round(p.N / dt1, 2), "unit": "slice-steps/s", "cores": 1, "kind": "oracle",
             "sample": f"{sample}: {dt1:.2f} s", "cpu": model}, ref)


def main():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--batch", type=int, default=32)
    ap.add_argument("--config", type=int, default=CFG, choices=[2, 3, 4],
                    help="workload: 3 = 6-qubit Ising d=64 (the headline), 2 = d=16, 4 = d=128")
    ap.add_argument("--precision", default="fp32", choices=["fp32", "fp64", "bf16x3"])
    ap.add_argument("--no-bf16", action="store_true", help="skip the split-BF16 leg")
    ap.add_argument("--no-fp64", action="store_true", help="skip the plain FP64 comparison leg")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-b1", action="store_true", help="skip the single-problem leg")
    ap.add_argument("--no-dense", action="store_true", help="skip the leg with the dense control kernels forced")
    ap.add_argument("--no-serving", action="store_true", help="skip the serving-engine trace replay")
    ap.add_argument("--no-state", action="store_true", help="skip the state-to-state leg")
    ap.add_argument("--no-lindblad", action="store_true", help="skip the open-system (Lindblad) leg")
    ap.add_argument("--no-trm", action="store_true", help="skip the trust-region fit leg")
    ap.add_argument("--serving-requests", type=int, default=4096,
                    help="requests in the serving trace (Poisson arrivals at 70%% of measured capacity)")
    ap.add_argument("--copy-gib", type=float, default=0.0,
                    help="before timing, run one plain device-to-device copy of this many GiB "
                         "(a reference of known size for hardware byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}); the multi-GPU design is "
              "described but not built", file=sys.stderr)
        sys.exit(2)

    # the serving replay runs first, in a child process started before this
    # process loads the GPU runtime
    serving = None if args.no_serving else serving_leg(args.serving_requests)
    if serving is not None:
        print("[bench] serving leg done", file=sys.stderr, flush=True)

    import torch
    from paper_2208_12187_amd import qoc
    from workloads import make_batch

    torch.cuda.init()
    if args.copy_gib > 0:
        n = int(args.copy_gib * (1 << 30)) // 4
        src = torch.ones(n, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
        torch.cuda.empty_cache()
    B = args.batch
    problems = make_batch(args.config, B)
    d, m, N = problems[0].d, problems[0].m, problems[0].N
    batch = qoc.Batch.from_problems(problems)
    plans = {pr: np.concatenate([qoc.slice_plan(p.H0, p.Hc, p.u, p.dt, pr, True) for p in problems])
             for pr in ("fp32", "fp64", "bf16x3")}
    flops = {pr: hermitian_flops(problems, plans[pr], d, m, pr) for pr in plans if pr != "bf16x3" or 16 < d <= 64}
    flops_dense = flops[args.precision]

    def leg(prec, steps, bsz=B, bat=batch, dense_controls=False):
        r = qoc.Runner(bsz, d, m, N, prec, dense_controls=dense_controls)
        out = time_runner(qoc, torch, r, bat, steps, args.warmup)
        del r
        torch.cuda.empty_cache()
        return out

    head = leg(args.precision, args.steps)
    ms = head["ms_per_step"]
    value = B * N / (ms / 1e3)

    # roofline of the dominant kernel (adjoint), from its own event timings
    adj_ms, adj_n = head["stages"]["adjoint"]
    adj_avg_s = adj_ms / max(adj_n, 1) / 1e3
    adj_flops = flops[args.precision]["adjoint"]
    achieved = adj_flops / adj_avg_s / 1e12
    peak = PEAK_TFLOPS[args.precision]
    traffic = measured_traffic(adj_ms / max(adj_n, 1)) if (args.precision == "fp32" and args.config == CFG
                                                          and B == 32) else None
    roofline = {"bound": "mfma", "achieved": round(achieved, 2), "peak": peak, "unit": "TFLOP/s",
                "frac": round(achieved / peak, 4), "traffic": None if traffic is None else round(traffic),
                "traffic_source": None if traffic is None else
                ("stored rocprofv3 reading (profiles/k_seg_grad_counters.json: FETCH_SIZE + WRITE_SIZE per "
                 "dispatch, each scaled by its reading for a plain 1 GiB copy), used because its kernel-source "
                 "hash matches this build; not measured in this run"),
                "kernel": flops[args.precision]["kernel"], "avg_launch_ms": round(adj_ms / max(adj_n, 1), 4),
                "cgemm_8d3_tflops": round(flops[args.precision]["adjoint_8d3"] / adj_avg_s / 1e12, 2)}

    def path_flops(pr):
        return sum(v for k, v in flops[pr].items() if k not in ("adjoint_8d3", "kernel"))

    total_flops = path_flops(args.precision)
    stages = {k: round(v[0] / max(v[1], 1), 4) for k, v in head["stages"].items() if v[1]}

    extra = {}
    if not args.no_dense:
        # the same workload with the dense control kernels forced (the spin-chain
        # controls are Pauli strings, which the default path takes row by row)
        dn = leg(args.precision, args.steps, dense_controls=True)
        adn_ms, adn_n = dn["stages"]["adjoint"]
        extra["dense_controls"] = {"value": round(B * N / (dn["ms_per_step"] / 1e3), 1),
                                   "ms_per_step": round(dn["ms_per_step"], 3),
                                   "stages_ms": {k: round(v[0] / max(v[1], 1), 4) for k, v in dn["stages"].items()
                                                 if v[1]},
                                   "adjoint_frac": round(flops_dense["adjoint"] / (adn_ms / max(adn_n, 1) / 1e3) / 1e12
                                                         / peak, 4),
                                   "max_abs_dF": float(np.max(np.abs(dn["F"] - head["F"]))),
                                   "grad_err_rel": worst_rel_grad_err(dn["grad"], head["grad"])}
    if not args.no_fp64 and args.precision != "fp64":
        f64 = leg("fp64", max(2, args.steps // 4))
        v64 = B * N / (f64["ms_per_step"] / 1e3)
        extra["fp64"] = {"value": round(v64, 1), "ms_per_step": round(f64["ms_per_step"], 3),
                         "stages_ms": {k: round(v[0] / max(v[1], 1), 4) for k, v in f64["stages"].items() if v[1]},
                         "path_tflops": round(path_flops("fp64") / (f64["ms_per_step"] / 1e3) / 1e12, 2)}
        extra["speedup_vs_fp64"] = round(value / v64, 3)
        extra["max_abs_dF_fp32_vs_fp64"] = float(np.max(np.abs(head["F"] - f64["F"])))
    b3 = None
    if not args.no_bf16 and args.precision != "bf16x3" and 16 < d <= 64:
        b3 = leg("bf16x3", args.steps)
        v3 = B * N / (b3["ms_per_step"] / 1e3)
        adj3_ms, adj3_n = b3["stages"]["adjoint"]
        extra["bf16x3"] = {"value": round(v3, 1), "ms_per_step": round(b3["ms_per_step"], 3),
                           "stages_ms": {k: round(v[0] / max(v[1], 1), 4) for k, v in b3["stages"].items() if v[1]},
                           "adjoint_fp32_equiv_tflops": round(flops["bf16x3"]["adjoint_8d3"] / (adj3_ms / max(adj3_n, 1) / 1e3) / 1e12, 2),
                           # (Hermitian problems run the FP32 precision's split-FP16 kernels)
                           "adjoint_mfma_frac": round(flops["bf16x3"]["adjoint"] / (adj3_ms / max(adj3_n, 1) / 1e3)
                                                           / 1e12 / PEAK_TFLOPS["bf16x3"], 4),
                           "max_abs_dF_vs_fp32": float(np.max(np.abs(b3["F"] - head["F"]))),
                           "grad_err_vs_fp32": worst_rel_grad_err(b3["grad"], head["grad"])}
        if "fp64" in extra:
            extra["bf16x3"]["speedup_vs_fp64"] = round(v3 / extra["fp64"]["value"], 3)
    if not args.no_b1:
        b1 = qoc.Batch(batch.H0[:1], batch.Hc[:1], batch.u[:1], batch.dt, batch.V[:1])
        one = leg(args.precision, args.steps, 1, b1)
        extra["batch1"] = {"value": round(N / (one["ms_per_step"] / 1e3), 1),
                           "ms_per_step": round(one["ms_per_step"], 3), "step_time": one["step_time"]}
        for pr in ("fp64", "bf16x3"):
            if pr == args.precision or (pr == "fp64" and args.no_fp64) or \
                    (pr == "bf16x3" and (args.no_bf16 or not 16 < d <= 64)):
                continue
            o = leg(pr, args.steps, 1, b1)
            extra["batch1"][pr] = {"value": round(N / (o["ms_per_step"] / 1e3), 1),
                                   "ms_per_step": round(o["ms_per_step"], 3), "step_time": o["step_time"]}
        # the host-pointer entry point on the same problem: device allocation,
        # host-to-device copies, the path and the copy back, per call
        p0 = problems[0]
        qoc.gradient(p0.H0, p0.Hc, p0.u, p0.dt, p0.V, args.precision)
        t0 = time.perf_counter()
        calls = 5
        for _ in range(calls):
            qoc.gradient(p0.H0, p0.Hc, p0.u, p0.dt, p0.V, args.precision)
        host_ms = (time.perf_counter() - t0) / calls * 1e3
        extra["host_api_pcie_inclusive"] = {"value": round(N / (host_ms / 1e3), 1), "ms_per_call": round(host_ms, 3)}

    if serving is not None:
        extra["serving"] = serving
    if not args.no_state:
        extra["state_transfer"] = state_leg(qoc, torch, args.steps, args.warmup)
        print("[bench] state-transfer leg done", file=sys.stderr, flush=True)
    if not args.no_lindblad:
        extra["lindblad"] = lindblad_leg(qoc, torch, args.steps, args.warmup)
        print("[bench] Lindblad leg done", file=sys.stderr, flush=True)
    if not args.no_trm:
        extra["trm"] = trm_leg()
        print("[bench] trust-region leg done", file=sys.stderr, flush=True)

    cpu = None
    if not args.no_cpu:
        cpu, cpu1, ref = cpu_baseline()
        extra["cpu_baseline_1thread"] = cpu1
        if args.config == CFG:
            # the headline run's first problem is the oracle's sample
            g0 = head["grad"][0].cpu().numpy()
            extra["vs_oracle_problem0"] = {"abs_dF": float(abs(head["F"][0] - ref["F"])),
                                           "grad_err_rel_max": float(np.max(np.abs(g0 - ref["grad"]))
                                                                     / np.max(np.abs(ref["grad"])))}
            if b3 is not None:
                g3 = b3["grad"][0].cpu().numpy()
                extra["bf16x3"]["vs_oracle_problem0"] = {
                    "abs_dF": float(abs(b3["F"][0] - ref["F"])),
                    "grad_err_rel_max": float(np.max(np.abs(g3 - ref["grad"])) / np.max(np.abs(ref["grad"])))}

    out = {
        "metric": METRIC,
        "value": round(value, 1),
        "unit": "slice-steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"fp32": "f32", "fp64": "f64", "bf16x3": "bf16x3"}[args.precision],
        "data": "synthetic",
        "config": {"workload": f"{WORKLOADS[args.config]} GRAPE fwd+grad, d={d}, m={m}, N={N}, "
                               f"dt={problems[0].dt}, batch of {B} seeded problems",
                   "d": d, "m": m, "N": N, "batch": B, "precision": args.precision},
        "roofline": roofline,
        "cpu_baseline": None if cpu is None else {k: (round(v, 2) if isinstance(v, float) else v)
                                                  for k, v in cpu.items()},
        "path_tflops": round(total_flops / (ms / 1e3) / 1e12, 2),
        "step_time": head["step_time"],
        "stages_ms": stages,
    }
    out.update(extra)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
