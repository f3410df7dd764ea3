"""Host-side checks of the bench's accounting of the segmented Hermitian path: the
orders follow the plan's rule, the product counts the kernels' loops, and each
dimension and precision is counted as the path that runs it."""
import math

import numpy as np
import pytest

import bench
from paper_2208_12187_amd import qoc
from workloads import make_config, make_random


def _at(p, theta):
    n1 = lambda H: np.abs(H).sum(axis=0).max()
    t = n1(p.H0) + np.abs(p.u).T @ np.array([n1(H) for H in p.Hc])
    p.dt = theta / float(t.max())
    return p, p.dt * t


def _tail(x, n, shift):
    """Remainder of sum x^k / (k + shift)! after the terms an n-product series takes."""
    k = n + 1 - shift
    return x ** k / math.factorial(n + 1) / (1 - x / (n + 2))


@pytest.mark.parametrize("d,prec", [(16, "fp64"), (64, "fp32"), (64, "fp64"), (100, "fp32")])
@pytest.mark.parametrize("theta", [1e-3, 0.1, 0.6, 0.95])
def test_orders_meet_the_remainder_bounds(d, prec, theta):
    p, th = _at(make_random(3, d, 2, 6, 0.01), theta)
    plan = qoc.slice_plan(p.H0, p.Hc, p.u, p.dt, prec, True)
    ur = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    for n, x in zip(bench.series_orders([p], plan, prec, d), 2 * th / 2.0 ** plan[:, 0]):
        n = int(n)
        need = [_tail(x, n, 0) <= ur * (1 + 1e-12)]
        spare = [n > 1 and _tail(x, n - 1, 0) <= ur * (1 - 1e-12)]
        if d > 64:  # Z's own series, of one term less
            need.append(_tail(x, n, 1) <= ur * (1 + 1e-12))
            spare.append(n > 1 and _tail(x, n - 1, 1) <= ur * (1 - 1e-12))
        assert all(need) and (n == 2 and d > 64 or not all(spare)), (n, x)


def _taylor(q):
    """Products of taylor_delta at d <= 64."""
    if q <= 3:
        return sum(1 for _ in range(q - 1, 0, -1))  # Horner
    n = 1                                           # A2
    if q <= 8:
        return n + 1 + (q > 4)                      # A2 B, then the degree-8 form's last
    n, t = n + 1, (q - 1) // 3                      # A3
    while t > 0:                                    # D_t + A3 R
        n, t = n + 1, t - 1
    return n


def _ps(q):
    """Products of the d = 128 exponential: X X, then one per digit and the last."""
    if q < 2:
        return 0
    if q == 2:
        return 1
    top = (q - 2) // 2
    return 1 + (top if q % 2 else top - 1) + 1


def _gradient(s, m, big, q, d):
    """Products of the gradient kernel on one slice."""
    if big:
        if s == 0:
            return max(m, 2)
        return max(m, 2) - 1 + _ps(q) + sum(2 + 1 for _ in range(s)) + 2
    n = m
    for j in range(s):
        n += 2 + (1 if j + 1 < s or d <= 16 else 0)
    return n + (2 if s else 0)


@pytest.mark.parametrize("d,prec", [(16, "fp32"), (16, "fp64"), (64, "fp32"), (64, "fp64"), (64, "bf16x3"), (128, "fp32")])
def test_product_counts_match_the_loops(d, prec, monkeypatch):
    for s in range(4):
        for q in range(1, 14):
            for m in (1, 2, 5, 12):
                monkeypatch.setattr(bench, "series_orders",
                                    lambda pr, pl, p, dd=64, m=m: np.array([m if dd <= 64 else max(m, 2)]))
                f = bench.series_flops(None, np.array([[s, q, q + 1]]), d, prec)
                big = d > 64
                g = 6.0 if prec == "fp64" else 24.0
                assert f["expm"] == g * d ** 3 * ((_ps(q) if big else _taylor(q)) + s), (s, q)
                assert f["adjoint"] == g * d ** 3 * _gradient(s, m, big, q, d), (s, q, m)
                assert f["adjoint_8d3"] == 8.0 * d ** 3 * _gradient(s, m, big, q, d)
                assert f["chain"] == (8.0 if d == 16 else 6.0) * d ** 3


@pytest.mark.parametrize("cfg,prec,kernel", [(2, "fp32", "k_seg_grad"), (2, "fp64", "k_seg_grad"), (3, "fp32", "k_seg_grad"),
                                             (3, "bf16x3", "k_seg_grad"), (4, "fp32", "k_seg_grad128"),
                                             (4, "fp64", "k_adjoint128")])
def test_each_workload_is_counted_as_the_path_that_runs_it(cfg, prec, kernel):
    p = make_config(cfg, N=6)
    plan = qoc.slice_plan(p.H0, p.Hc, p.u, p.dt, prec, True)
    f = bench.hermitian_flops([p], plan, p.d, p.m, prec)
    assert f["kernel"] == kernel
    if kernel == "k_adjoint128":
        assert f["adjoint"] == bench.slice_flops(plan, p.d, p.m, prec)["adjoint"]
        assert f["expm"] == 8.0 * p.d ** 3 * sum(_ps(int(q)) + int(s) for s, q, _ in plan)
    else:
        assert f["adjoint"] == bench.series_flops([p], plan, p.d, prec)["adjoint"]
