"""Workspaces of the state path (no GPU): which batches are cut into chunks (the
chunk totals are part of the size), and which sizes a call accepts."""
import pytest

from paper_2208_12187_amd import qoc


def _totals(B, d, N, prec):
    """Bytes per problem beyond those of single chains (a batch far above the line)."""
    one = lambda b: qoc.state_workspace_size(b, d, 12, N, prec) / b
    return one(B) - one(4096)


@pytest.mark.parametrize("d,prec,last", [(16, "fp32", 512), (32, "fp32", 256), (64, "fp32", 64), (16, "fp64", 512),
                                         (32, "fp64", 96), (64, "fp64", 24)])
@pytest.mark.parametrize("N", [64, 500, 2000])
def test_batches_that_are_cut_into_chunks(d, prec, last, N):
    """Up to the batch at which single chains are as fast: at d = 64 in FP64 24
    problems gain a tenth from chunks and 32 lose one."""
    mat = 2 * d * d * (8 if prec == "fp64" else 4)
    chunks = -(-N // qoc.engine_chunk(d, N))
    for B in (1, last - 1, last):
        assert abs(_totals(B, d, N, prec) - chunks * mat) < 1024
    assert abs(_totals(last + 1, d, N, prec)) < 1024
    assert abs(_totals(1, d, 63, prec)) < 1024


def _launches(B, d, N, prec, ws_bytes):
    """Whether the call passes the check of its workspace.  Without a device it then
    ends with the device error of the descriptor upload, before any launch."""
    import ctypes

    import torch

    if torch.cuda.is_available():
        pytest.skip("host pointers stand in for device memory")
    L = qoc.lib()
    o = qoc.options(prec)
    buf = ctypes.create_string_buffer(4096)
    p = (ctypes.addressof(buf) + 255) // 256 * 256
    rc = L.qoc_state_gradient_dev(B, d, 12, N, p, p, p, 0.01, p, p, p, p, p, ws_bytes, ctypes.byref(o))
    assert rc in (-1, -5), L.qoc_last_error()
    return rc == -5


@pytest.mark.parametrize("d,prec,N,M", [(64, "fp32", 2000, 2000), (64, "fp64", 2000, 2000), (16, "fp32", 500, 500),
                                        (64, "fp32", 72, 73), (32, "fp64", 128, 129), (64, "fp64", 63, 64)])
def test_a_workspace_of_a_larger_call_is_accepted(d, prec, N, M):
    """A workspace sized for B problems of M slices serves every smaller batch of
    N <= M, whether those are cut into chunks or not."""
    for B in (1, 24, 25, 32, 64, 65, 200, 513, 600):
        size = qoc.state_workspace_size(B, d, 12, M, prec)
        for b in {b for b in (1, 2, B // 2, B - 1, B) if 1 <= b <= B}:
            assert _launches(b, d, N, prec, size), (B, b)
    # less than single chains take is refused
    assert not _launches(4096, d, N, prec, qoc.state_workspace_size(4096, d, 12, N, prec) - 1)
