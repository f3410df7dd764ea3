"""CPU pins of the split-FP16 arithmetic of the FP32 Hermitian path, emulated here in
NumPy independently of the kernels: a factor x is scaled by c = 2^12 and split into
hi = fp16(c x) and lo = fp16(c x - hi); a real product is
hi_a hi_b + hi_a lo_b + lo_a hi_b with FP32 accumulation, divided by c^2.

Bounds.  FP16 has 11 significant bits (unit roundoff 2^-11) down to 2^-14 and steps of
2^-24 below.  So |c x - hi| <= 2^-11 |c x|, and lo, rounded to 11 bits of that, leaves
|c x - hi - lo| <= 2^-22 |c x| where lo is normal and <= 2^-25 otherwise: in x,
max(2^-22 |x|, 2^-37).  Dropping lo_a lo_b and the two representation errors cost at
most 3 2^-22 |a||b| per term (up to 2^-33 of it), and FP32 accumulation of n terms
gamma_n = n 2^-24 / (1 - n 2^-24) times the sum of |terms|, of which there are 3 n.
"""
import numpy as np
import pytest

C = np.float32(4096.0)
TINY = 2.0 ** -37


def split(x):
    y = (C * np.asarray(x, dtype=np.float32)).astype(np.float32)
    hi = y.astype(np.float16)
    lo = (y - hi.astype(np.float32)).astype(np.float16)  # the difference is exact in FP32
    return hi.astype(np.float32), lo.astype(np.float32)


def prod3(a, b, acc):
    ah, al = split(a)
    bh, bl = split(b)
    f = lambda x: x.astype(acc)
    return (f(ah) @ f(bl) + f(al) @ f(bh) + f(ah) @ f(bh)) / (float(C) ** 2)


def cprod3(A, B, acc):
    Ar, Ai, Br, Bi = (x.astype(np.float32) for x in (A.real, A.imag, B.real, B.imag))
    return prod3(Ar, Br, acc) - prod3(Ai, Bi, acc) + 1j * (prod3(Ar, Bi, acc) + prod3(Ai, Br, acc))


def _herm(d, rng):
    H = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
    return (H + H.conj().T) / 2


def _unitary(d, rng):
    w, Q = np.linalg.eigh(_herm(d, rng))
    return (Q * np.exp(-1j * w)) @ Q.conj().T


def test_split_keeps_22_bits():
    rng = np.random.default_rng(0)
    x = np.concatenate([s * rng.standard_normal(20000) for s in (1.0, 1e-2, 1e-4, 1e-6, 1e-9)]).astype(np.float32)
    x = x[np.abs(x) <= 8.0]
    hi, lo = split(x)
    err = np.abs((hi.astype(np.float64) + lo) / float(C) - x)
    assert (err <= np.maximum(2.0 ** -22 * np.abs(x.astype(np.float64)), TINY)).all()
    big = np.abs(x) >= 2.0 ** -14  # lo normal
    assert (err[big] <= 2.0 ** -22 * np.abs(x[big])).all()


def test_split_of_the_edges():
    # zeros, the largest staged value, the smallest FP32 numbers, ties
    for x in (0.0, -0.0, 8.0, -8.0, 1e-38, 2.0 ** -36, 1.0 + 2.0 ** -11, 1.0 + 3 * 2.0 ** -11, 15.99):
        hi, lo = split(np.float32(x))
        assert np.isfinite(hi) and np.isfinite(lo)
        assert abs((float(hi) + float(lo)) / float(C) - np.float32(x)) <= max(2.0 ** -22 * abs(x), TINY)


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_complex_product_bound(d):
    rng = np.random.default_rng(d)
    A = (0.3 * _herm(d, rng) / np.sqrt(d)).astype(np.complex64)
    B = _unitary(d, rng).astype(np.complex64)
    ref = A.astype(np.complex128) @ B.astype(np.complex128)
    n = 2 * d
    absum = lambda f, g: np.abs(f.astype(np.float64)) @ np.abs(g.astype(np.float64))
    sre = absum(A.real, B.real) + absum(A.imag, B.imag)
    sim = absum(A.real, B.imag) + absum(A.imag, B.real)
    gam = 3 * n * 2.0 ** -24 / (1 - 3 * n * 2.0 ** -24)
    tiny = 2 * TINY * (np.abs(A).max() + np.abs(B).max()) * n
    for acc, extra in ((np.float64, 0.0), (np.float32, gam)):
        got = cprod3(A, B, acc)
        bound = lambda s: (3.01 * 2.0 ** -22 + 1.01 * extra) * s + tiny
        assert (np.abs(got.real - ref.real) <= bound(sre)).all()
        assert (np.abs(got.imag - ref.imag) <= bound(sim)).all()


@pytest.mark.parametrize("d", [16, 64, 128])
def test_every_staged_factor_stays_in_range(d):
    """The largest factors of the path: the degree-8 form's, the series' terms
    (2 |A|)^n / n! |Y| with |A| = 1, U - I and the products D Y of a conjugation, for
    a target that is all in one entry or spread evenly and just short of the next
    power of two.  All stay below 2^15, half of FP16's range."""
    rng = np.random.default_rng(1)
    H = _herm(d, rng)
    A = -1j * H / np.abs(H).sum(axis=0).max()     # |A|_1 = 1, the largest the plan lets through
    w, Q = np.linalg.eigh(1j * A)
    U = lambda t: (Q * np.exp(-1j * t * w)) @ Q.conj().T
    top = lambda M: float(C) * max(np.abs(M.real).max(), np.abs(M.imag).max())
    lim = 2.0 ** 15
    r = np.sqrt(177.0)
    x3 = 2 / 3
    x1, x2 = x3 * (1 + r) / 88, x3 * (1 + r) / 352
    x4, x5 = (-271 + 29 * r) / (315 * x3), 11 * (-1 + r) / (1260 * x3)
    x6, x7 = 11 * (-9 + r) / (5040 * x3), (89 - r) / (5040 * x3 * x3)
    A2 = A @ A
    A4 = A2 @ (x1 * A + x2 * A2)
    for M in (A, A2, x1 * A + x2 * A2, x3 * A2 + A4, x4 * np.eye(d) + x5 * A + x6 * A2 + x7 * A4, A @ A2):
        assert top(M) < lim
    one = np.zeros((d, d), dtype=complex)
    one[0, 1] = 1.999
    even = np.full((d, d), 1.999 / d, dtype=complex)
    for V in (one, even, 1.999 / np.sqrt(d) * _unitary(d, rng)):
        N = U(3.0) @ V
        Y = (N - N.conj().T) / 2j
        Z = Y
        for n in range(1, 30):
            assert top(Z) < lim
            Z = (A @ Z - Z @ A) / n
        for t in (0.5, 3.0, 50.0):
            D = U(t) - np.eye(d)
            assert top(D) < lim and top(D @ Y) < lim
