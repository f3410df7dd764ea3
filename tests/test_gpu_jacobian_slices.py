"""The whole-Jacobian call on slices of any norm: their parts are doubled, s times
for 2^s parts, so that neither the work nor the shift by s bounds the norm.

Tolerance: exp(-i theta x) of a slice of norm theta has the condition number theta,
in the kernels and in the oracle alike, so a slice carries an error of theta times
the unit roundoff 2^-53 (2^-24), and N slices N of them; times 64 for the d terms of
each product's sums (d <= 64, products of errors of either sign) and the norm's
overestimate, and not less than the bound of well-scaled slices (1e-10 and 1e-4).
"""
import numpy as np
import pytest

from oracle import trm as T
from workloads import Problem, make_random
from workloads.spin import make_random_monomial

pytestmark = pytest.mark.gpu


def _at(p, theta):
    n1 = lambda H: np.abs(H).sum(axis=0).max()
    t = max(n1(p.H0) + sum(abs(p.u[j, k]) * n1(p.Hc[j]) for j in range(p.m)) for k in range(p.N))
    return Problem(p.H0, p.Hc, p.u, theta / t, p.V)


@pytest.mark.parametrize("theta", [1.9, 6.0, 50.0, 1e3, 1e6, 6e9])
@pytest.mark.parametrize("d,m,N,prec", [(2, 1, 3, "fp64"), (7, 3, 4, "fp64"), (16, 2, 5, "fp64"), (16, 3, 5, "fp32"),
                                        (32, 3, 3, "fp64"), (30, 1, 4, "fp32"), (64, 2, 3, "fp64"), (50, 3, 3, "fp32")])
def test_jacobian_of_long_slices(gpu_lib, d, m, N, prec, theta):
    import torch
    from paper_2208_12187_amd import qoc

    tol = max(1e-10 if prec == "fp64" else 1e-4, 64 * N * theta * 2.0 ** (-53 if prec == "fp64" else -24))
    if tol > 0.1:
        pytest.skip("no digit left at this precision")
    make = make_random_monomial if m == 2 else make_random
    p = make(500 + d, d, m, N, 0.01)
    # slices of one problem on both sides of theta = 1 (where s = 0 ends)
    p = _at(Problem(p.H0, p.Hc, p.u * np.linspace(1.0, 0.2, N), p.dt, p.V), theta)
    XN, dX = T.grape_xn_jacobian(p.H0, p.Hc, p.u, p.dt)
    J = torch.full((2 * d * d, m * N), 7.0, dtype=torch.float64, device="cuda")
    X = torch.empty((d, d), dtype=torch.complex128, device="cuda")
    print(f"[jacobian] d={d} m={m} N={N} {prec} theta={theta}", flush=True)
    qoc.JacobianRunner(d, m, N, prec).jacobian(qoc.Batch.from_problems([p]), J, X)
    torch.cuda.synchronize()
    J = J.cpu().numpy()
    ref = dX.transpose(2, 3, 0, 1).reshape(d * d, m * N)
    top = np.max(np.abs(ref))
    assert np.max(np.abs(X.cpu().numpy() - XN)) <= tol
    assert np.max(np.abs(J[:d * d] - ref.real)) <= tol * top
    assert np.max(np.abs(J[d * d:] - ref.imag)) <= tol * top
