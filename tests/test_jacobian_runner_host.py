"""JacobianRunner's buffers, with the library's launch replaced by a recorder
(no GPU): what it hands to the kernels has to stay alive after the call returns,
and what the kernels would write past is refused."""
import gc
import types
import weakref

import pytest
import torch

from paper_2208_12187_amd import qoc

D, M, N = 3, 2, 5


class _Recorder:
    """The real library except for the launch."""

    def __init__(self, real):
        self._real = real
        self.XN = None

    def __getattr__(self, name):
        return getattr(self._real, name)

    def qoc_jacobian_dev(self, d, m, N, H0, Hc, u, dt, J, ld, XN, ws, ws_bytes, opt):
        self.XN = XN
        return 0


@pytest.fixture
def setup(monkeypatch):
    rec = _Recorder(qoc.lib())
    monkeypatch.setattr(qoc, "lib", lambda: rec)
    r = qoc.JacobianRunner(D, M, N, "fp64", device="cpu")
    z = lambda *s: torch.zeros(s, dtype=torch.complex128)
    b = qoc.Batch(z(1, D, D), z(1, M, D, D), torch.zeros((1, M, N), dtype=torch.float64), 0.1)
    return rec, r, b, torch.zeros((2 * D * D, M * N + 1), dtype=torch.float64)


STREAM = types.SimpleNamespace(cuda_stream=0)


def test_every_buffer_of_a_call_outlives_it(setup, monkeypatch):
    """The kernels run after the call has returned, on a stream whose work the
    allocator does not know of: a buffer freed at return could be handed out
    again under them."""
    rec, r, b, J = setup
    made = []
    real = torch.empty

    def empty(*a, **k):
        t = real(*a, **k)
        made.append((weakref.ref(t), t.data_ptr()))
        return t

    monkeypatch.setattr(torch, "empty", empty)
    r.jacobian(b, J, stream=STREAM)
    gc.collect()
    assert rec.XN
    assert all(t() is not None for t, _ in made)
    assert rec.XN in {t().data_ptr() for t, _ in made} | {r.XN.data_ptr()}


@pytest.mark.parametrize("bad", [torch.zeros((D, D), dtype=torch.complex64), torch.zeros((D, D + 1), dtype=torch.complex128),
                                 torch.zeros((D, D), dtype=torch.complex128).T[:, ::2],
                                 torch.zeros((D, 2 * D), dtype=torch.complex128)[:, ::2]])
def test_a_buffer_for_xn_that_does_not_fit_is_refused(setup, bad):
    rec, r, b, J = setup
    with pytest.raises(ValueError):
        r.jacobian(b, J, XN=bad, stream=STREAM)
    assert rec.XN is None


def test_a_jacobian_elsewhere_is_refused(setup):
    rec, r, b, J = setup
    with pytest.raises(ValueError):
        r.jacobian(b, J.to("meta"), stream=STREAM)
    assert rec.XN is None
    X = torch.zeros((D, D), dtype=torch.complex128)
    r.jacobian(b, J, XN=X, stream=STREAM)
    assert rec.XN == X.data_ptr()


@pytest.mark.parametrize("name", ["fp64", "fp32"])
def test_precision_by_number(name):
    """As for Runner (and GrapeLSQ, which makes one of each): a name or its number."""
    a = qoc.JacobianRunner(D, M, N, name, device="cpu")
    b = qoc.JacobianRunner(D, M, N, qoc.PRECISIONS[name], device="cpu")
    assert a.ws_bytes == b.ws_bytes > 0
