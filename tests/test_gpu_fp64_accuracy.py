"""X_N in FP64 at d <= 16 against 80-bit arithmetic, at the rounding level.

Bound.  A number whose mantissa is log-uniform is rounded with an rms relative
error of 2^-52 sqrt((3 / 4) / (2 ln 2) / 12) = 0.425 2^-53.  A chain that rounds the
product once per slice at the size of its entries therefore carries, as a random
walk, a relative error of 0.425 2^-53 sqrt(N) in the Frobenius norm; a fifth more
is left for the errors of the products themselves, which scale with the slices'
norms (below 0.6 here), and of the carry (about 2 sqrt(N) of the N products).
Several problems are taken together, so that the mean square is sharp.  (Above
d = 16 the carry's products, in the three-product form, are larger than this.)
"""
import numpy as np
import pytest

from workloads.spin import heisenberg_drift, make_random, xy_controls

pytestmark = pytest.mark.gpu

CL, LD = np.clongdouble, np.longdouble


def _xn(H0, Hc, u, dt):
    """X_N in 80 bits: degree-18 Taylor polynomials at norms below 0.6 (0.6^19 / 19! < 2^-70)."""
    H0, Hc, u, dt = H0.astype(CL), Hc.astype(CL), u.astype(LD), LD(dt)
    d = H0.shape[0]
    eye = np.eye(d, dtype=CL)
    A = -1j * dt * (H0 + np.einsum("jk,jab->kab", u, Hc))
    assert np.abs(A).sum(axis=1).max() < 0.6
    P = eye + A / LD(18)
    for i in range(17, 0, -1):
        P = eye + (A @ P) / LD(i)
    X = eye
    for U in P:
        X = U @ X
    return X


def _problem(d, m, N, seed):
    rng = np.random.default_rng([seed, d])
    if m == 0:  # dense
        p = make_random(seed, d, 3, N, 0.01)
        return p.H0, p.Hc, p.u, 0.01
    nq = d.bit_length() - 1
    H0 = heisenberg_drift(rng.uniform(0.5, 1.5, nq - 1), rng.normal(0.0, 0.2, nq))
    return H0, np.stack(xy_controls(nq)), rng.normal(0.0, 0.5, (2 * nq, N)), 0.005


@pytest.mark.parametrize("d,m,N", [(16, 8, 1000), (16, 0, 800), (8, 6, 800)])
def test_xn_at_the_rounding_level(gpu_lib, d, m, N):
    from paper_2208_12187_amd import qoc

    e2 = []
    for seed in range(5):
        H0, Hc, u, dt = _problem(d, m, N, seed)
        ref = _xn(H0, Hc, u, dt)
        X = qoc.propagate(H0, Hc, u, dt, "fp64").astype(CL)
        e2.append(float((np.abs(X - ref) ** 2).sum() / (np.abs(ref) ** 2).sum()))
    rms, bound = np.sqrt(np.mean(e2)), 1.2 * 0.425 * 2.0 ** -53 * np.sqrt(N)
    print(f"[accuracy] d={d} m={m} N={N}: {rms:.3g}, bound {bound:.3g}", flush=True)
    assert rms <= bound
