"""Gradients of problems with squared slices (a slice norm bound above 1), whose
segments are spread over all workgroups: batches where only some problems have
such slices, more segments than workgroups and fewer, the serving engine,
checkpointed calls and the complex trace gradient.

A member of a batch has to give its results alone bit for bit, however its segments
are dealt out (and cut) there and here; against the oracle the tolerances of the
gradient path: FP64 |F - F_ref| <= 1e-10 F_ref and max|grad - ref| <= 1e-10 max|ref|,
FP32 1e-5 and 1e-4.
"""
import numpy as np
import pytest

import oracle
from oracle import trm as T
from workloads import Problem, make_random
from workloads.spin import make_random_monomial

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-4, "bf16x3": 1e-4}


def _theta(p):
    n1 = lambda H: np.abs(H).sum(axis=0).max()
    return p.dt * np.array([n1(p.H0) + sum(abs(p.u[j, k]) * n1(p.Hc[j]) for j in range(p.m)) for k in range(p.N)])


def _batch(d, m, N, thetas, mono=False):
    """One problem per entry of thetas, whose largest slice has that norm bound (one
    dt: amplitudes and drift take the scale)."""
    out = []
    for i, t in enumerate(thetas):
        p = (make_random_monomial if mono else make_random)(60 + i, d, m, N, 0.01)
        c = t / _theta(p).max()
        out.append(Problem(c * p.H0, p.Hc, c * p.u, p.dt, p.V))
    return out


def _run(probs, prec, **kw):
    import torch
    from paper_2208_12187_amd import qoc

    b = qoc.Batch.from_problems(probs)
    F, g = qoc.Runner(b.B, b.d, b.m, b.N, prec, **kw).gradient(b)
    torch.cuda.synchronize()
    return F.cpu().numpy(), g.cpu().numpy()


def _check(F, grad, ref, prec):
    assert abs(F - ref["F"]) <= (1e-10 * ref["F"] if prec == "fp64" else 1e-5)
    assert np.max(np.abs(grad - ref["grad"])) <= TOL[prec] * np.max(np.abs(ref["grad"]))


@pytest.mark.parametrize("d,m,N,prec", [(3, 2, 70, "fp64"), (16, 3, 70, "fp32"), (16, 3, 40, "fp64"), (30, 2, 70, "fp64"),
                                        (32, 3, 200, "fp32"), (32, 2, 70, "bf16x3"), (64, 2, 70, "fp32"), (51, 2, 70, "fp64"),
                                        (100, 2, 40, "fp32"), (128, 2, 30, "fp32")])
@pytest.mark.parametrize("mono", [False, True])
def test_some_problems_of_a_batch(gpu_lib, d, m, N, prec, mono):
    probs = _batch(d, m, N, [0.4, 1.5, 0.2, 0.9, 5.0, 0.3], mono)
    print(f"[squared] d={d} N={N} {prec} mono={mono}", flush=True)
    F, g = _run(probs, prec)
    for i, p in enumerate(probs):
        if i in (0, 1, 4):
            _check(F[i], g[i], oracle.grape_ref(p), prec)
        F1, g1 = _run([p], prec)
        assert F1[0] == F[i] and np.array_equal(g1[0], g[i]), f"problem {i}"


@pytest.mark.parametrize("d,N,B,prec", [(4, 1000, 6, "fp32"), (4, 1000, 6, "fp64"), (20, 700, 8, "fp64"),
                                        (20, 700, 8, "fp32"), (40, 600, 4, "fp64"), (40, 600, 5, "fp32"),
                                        (70, 300, 3, "fp32")])
def test_more_segments_than_workgroups(gpu_lib, d, N, B, prec):
    """Batches of more segments than the grid has workgroups, their members alone of
    fewer (which are cut into slices at 17 <= d <= 64)."""
    probs = _batch(d, 2, N, [2.0 + 0.1 * i for i in range(B)])
    print(f"[squared] d={d} N={N} B={B} {prec}", flush=True)
    F, g = _run(probs, prec)
    _check(F[B - 1], g[B - 1], oracle.grape_ref(probs[B - 1]), prec)
    for i in (0, B - 1):
        F1, g1 = _run([probs[i]], prec)
        assert F1[0] == F[i] and np.array_equal(g1[0], g[i]), f"problem {i}"


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_engine_with_squared_slices(gpu_lib, prec):
    """Requests with and without squared slices in one tick, bit for bit the host
    entry point's."""
    from paper_2208_12187_amd import qoc

    probs = []
    for d, N in ((2, 300), (16, 90), (16, 700), (27, 90), (32, 500), (64, 100), (50, 300), (100, 60), (128, 20)):
        probs += _batch(d, 2, N, [3.0, 0.5, 1.2])
    eng = qoc.Engine(prec, pool_bytes=8 << 30, host_bytes=128 << 20, max_active=64)
    try:
        ids = [eng.submit(p.H0, p.Hc, p.u, p.dt, p.V) for p in probs]
        F = {}
        while len(F) < len(ids):
            eng.step(wait=True)
            F.update(eng.poll())
        for i, p in zip(ids, probs):
            F1, g1 = qoc.gradient(p.H0, p.Hc, p.u, p.dt, p.V, prec, chunk=qoc.engine_chunk(p.d, p.N))
            assert F[i] == F1 and np.array_equal(eng.fetch(i), g1), (p.d, p.N)
    finally:
        eng.close()


@pytest.mark.parametrize("d,N,prec", [(16, 130, "fp64"), (32, 130, "fp32"), (64, 90, "fp64"), (64, 90, "fp32"), (128, 40, "fp32")])
def test_checkpointed(gpu_lib, d, N, prec):
    from paper_2208_12187_amd import qoc

    probs = _batch(d, 2, N, [1.7, 0.6])
    F, g = _run(probs, prec)
    Fc, gc = _run(probs, prec, hbm_budget=qoc.workspace_size(2, d, 2, N, prec) // 4)
    assert np.array_equal(F, Fc) and np.array_equal(g, gc)


@pytest.mark.parametrize("d,N,chunk,prec", [(16, 30, 0, "fp32"), (32, 50, 0, "fp32"), (60, 40, 0, "fp32"),
                                            (100, 30, 0, "fp32"), (40, 20, 0, "fp64"), (32, 50, 0, "bf16x3"),
                                            (20, 1300, 2, "fp32"), (20, 1300, 2, "bf16x3"), (40, 600, 2, "fp32"),
                                            (40, 600, 2, "bf16x3")])
def test_trace_gradient(gpu_lib, d, N, chunk, prec):
    """The complex derivative's two Hermitian parts, in slices cut out of their segments
    and (more segments than workgroups) in whole segments."""
    import torch
    from paper_2208_12187_amd import qoc

    probs = _batch(d, 2, N, [2.5, 0.5])
    b = qoc.Batch.from_problems(probs)
    print(f"[squared] trace gradient d={d} N={N} {prec}", flush=True)
    _, dg = qoc.Runner(2, d, 2, N, prec, chunk=chunk).trace_gradient(b)
    torch.cuda.synchronize()
    for p, x in zip(probs, dg.cpu().numpy()):
        _, dX = T.grape_xn_jacobian(p.H0, p.Hc, p.u, p.dt)
        ref = np.einsum("ab,jkab->jk", p.V.conj(), dX)
        assert np.max(np.abs(x - ref)) <= TOL[prec] * np.max(np.abs(ref))
