"""The chunked chains of the state path (N >= 64, d <= 64) against the FP64 state
oracle and against the single chain that larger batches take.

Tolerances as for the state path: FP64 |F - F_ref| <= 1e-10 F_ref and max|grad - ref|
<= 1e-10 max|ref|; FP32 |F - F_ref| <= 1e-5 and max|grad - ref| <= 1e-4 max|ref|, and
the same between the two forms, which differ by their rounding only.
"""
import numpy as np
import pytest

import oracle
from workloads import StateProblem, make_state_random

pytestmark = pytest.mark.gpu

TOL = {"fp64": (1e-10, 1e-10), "fp32": (1e-5, 1e-4)}


def _check(F, g, ref, prec):
    assert abs(F - ref["F"]) <= TOL[prec][0] * (ref["F"] if prec == "fp64" else 1.0)
    assert np.max(np.abs(g - ref["grad"])) <= TOL[prec][1] * np.max(np.abs(ref["grad"]))


# around the rule's line, a last chunk of one slice (L = 3: 64, 67; L = 4: 101),
# more chunks than the totals kept in registers
@pytest.mark.parametrize("N", [63, 64, 67, 101])
@pytest.mark.parametrize("d,m,mono,prec", [(2, 1, True, "fp64"), (13, 3, False, "fp32"), (16, 20, True, "fp64"),
                                           (20, 2, False, "fp64"), (32, 4, True, "fp32"), (51, 2, False, "fp64"),
                                           (64, 14, True, "fp32"), (64, 3, True, "fp64")])
def test_chunked_chains(gpu_lib, d, m, mono, prec, N):
    from paper_2208_12187_amd import qoc

    p = make_state_random(500 + d, d, m, N, 0.02, monomial=mono)
    print(f"[state] chunks d={d} m={m} N={N} {prec}", flush=True)
    ref = oracle.state_ref(p)
    _check(*qoc.state_gradient(p.H0, p.Hc, p.u, p.dt, p.psi0, p.chi, prec), ref, prec)
    psiN = qoc.state_propagate(p.H0, p.Hc, p.u, p.dt, p.psi0, prec)
    assert np.max(np.abs(psiN - ref["psiN"])) <= TOL[prec][0]


@pytest.mark.parametrize("d,prec", [(5, "fp64"), (30, "fp32"), (64, "fp32")])
def test_chunks_of_long_slices(gpu_lib, d, prec):
    """Slices of 2^s parts (the largest norm bound of a slice is 1.5)."""
    from paper_2208_12187_amd import qoc

    q = make_state_random(600 + d, d, 2, 65, 1.0, monomial=True)
    n1 = lambda H: np.abs(H).sum(axis=0).max()
    theta = max(n1(q.H0) + sum(abs(q.u[j, k]) * n1(q.Hc[j]) for j in range(2)) for k in range(65))
    p = StateProblem(q.H0, q.Hc, q.u, 1.5 / theta, q.psi0, q.chi)
    assert qoc.slice_plan(p.H0, p.Hc, p.u, p.dt, prec)[:, 0].max() >= 1
    print(f"[state] chunks of long slices d={d} {prec}", flush=True)
    _check(*qoc.state_gradient(p.H0, p.Hc, p.u, p.dt, p.psi0, p.chi, prec), oracle.state_ref(p), prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_batches_beyond_the_chunked_ones(gpu_lib, prec):
    """65 problems (FP64: 33) of d = 40 run single chains, one less chunked ones."""
    import torch
    from paper_2208_12187_amd import qoc

    p = make_state_random(9, 40, 2, 70, 0.02)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    out = []
    for B in ((64, 65) if prec == "fp32" else (32, 33)):
        rep = lambda a: t(a)[None].expand(B, *a.shape).contiguous()
        b = qoc.StateBatch(rep(p.H0), rep(p.Hc), rep(p.u), p.dt, rep(p.psi0), rep(p.chi))
        F, g = qoc.StateRunner(B, 40, 2, 70, prec).gradient(b)
        torch.cuda.synchronize()
        F, g = F.cpu().numpy(), g.cpu().numpy()
        assert (F == F[0]).all() and (g == g[0]).all()
        out.append((F[0], g[0]))
    _check(*out[0], {"F": out[1][0], "grad": out[1][1]}, prec)
