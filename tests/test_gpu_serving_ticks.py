"""Ticks of the serving engine with more work items than workgroups, so that a
persistent workgroup takes several in turn, against the host entry point with
the engine's chunk length (the same kernels on the same numbers: bit for bit)."""
import numpy as np
import pytest

from workloads import make_random

pytestmark = pytest.mark.gpu


def _replay(prec, probs, max_active):
    from paper_2208_12187_amd import qoc

    eng = qoc.Engine(prec, pool_bytes=6 << 30, host_bytes=256 << 20, max_active=max_active)
    try:
        ids = [eng.submit(p.H0, p.Hc, p.u, p.dt, p.V) for p in probs]
        F = {}
        while len(F) < len(ids):
            eng.step(wait=True)
            F.update(eng.poll())
        return [(F[i], eng.fetch(i)) for i in ids]
    finally:
        eng.close()


def _same(prec, probs, got):
    from paper_2208_12187_amd import qoc

    for i, (p, (F, grad)) in enumerate(zip(probs, got)):
        F1, g1 = qoc.gradient(p.H0, p.Hc, p.u, p.dt, p.V, prec, chunk=qoc.engine_chunk(p.d, p.N))
        assert F == F1 and np.array_equal(grad, g1), f"request {i}"


@pytest.mark.parametrize("d,m,n,prec", [(3, 2, 1100, "fp32"), (128, 14, 40, "fp32"), (100, 6, 70, "fp64")])
def test_targets_of_every_size_in_one_tick(gpu_lib, d, m, n, prec):
    """m + 2 items per request divide the grid (2048 and 256 workgroups), so that
    one workgroup prepares the targets of several requests in a row; their norms,
    which the preparation takes out, differ by powers of two."""
    probs = []
    for i in range(n):
        p = make_random(i % 7, d, m, 2, 0.01)
        probs.append(p.with_target(2.0 ** (i % 5 - 2) * p.V))
    print(f"[ticks] d={d} m={m} n={n} {prec}", flush=True)
    _same(prec, probs, _replay(prec, probs, n))
