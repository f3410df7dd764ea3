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
