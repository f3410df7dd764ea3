"""Row tables of controls whose entries vanish in FP32: the tables are built from the
rounded entries, and so has to be the comparison of one control's columns with the
next one's (which then share entries of Z in the general generators' FP32 adjoint).

Tolerance: FP32 max|grad - ref| <= 1e-4 max|ref|, as for the rest of the FP32 path.
"""
import numpy as np
import pytest

from oracle import lindblad as LB

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [20, 32, 64, 100])
def test_entries_below_fp32_range(gpu_lib, d):
    from paper_2208_12187_amd import qoc

    rng = np.random.default_rng(d)
    N = 6
    G0 = 0.3 * (rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))) / np.sqrt(d)
    shift = np.roll(np.diag(rng.standard_normal(d) + 1j * rng.standard_normal(d)), 1, axis=1)
    # the first control's entries lie where the second one's do, but are 0 in FP32: rows
    # without an entry count at their own column
    Gc = np.stack([1e-60 * shift, shift, np.diag(rng.standard_normal(d))])
    u = rng.normal(0.0, 0.5, (3, N))
    T = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
    print(f"[row tables] d={d}", flush=True)
    F, grad = qoc.gradient(G0, Gc, u, 0.05, T, "fp32", generators=True)
    F0, _, ref, _ = LB.generator_gradient(G0, Gc, u, 0.05, T)
    assert abs(F - F0) <= 1e-4 * F0
    assert np.max(np.abs(grad - ref)) <= 1e-4 * np.max(np.abs(ref))
