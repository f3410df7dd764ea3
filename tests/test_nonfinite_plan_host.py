"""The slice plan of inputs that are not finite (no GPU): the _dev entry points never
read their inputs on the host, so the plan is what keeps such a slice from 2^60
steps.  Finite slices of the same problem keep their plans."""
import numpy as np
import pytest

from paper_2208_12187_amd import qoc
from workloads import make_random


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("d,prec", [(4, "fp64"), (40, "fp32"), (100, "fp32"), (100, "fp64")])
def test_no_squarings(d, prec, grad, bad):
    p = make_random(5, d, 2, 4, 0.5)
    ref = qoc.slice_plan(p.H0, p.Hc, p.u, p.dt, prec, grad)
    u = p.u.copy()
    u[1, 2] = bad
    plan = qoc.slice_plan(p.H0, p.Hc, u, p.dt, prec, grad)
    assert plan[2].tolist() == [0, 1, 2]
    assert np.array_equal(np.delete(plan, 2, 0), np.delete(ref, 2, 0))
    assert (ref[:, 0] > 0).any()
