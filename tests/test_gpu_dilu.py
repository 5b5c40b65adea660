"""The DILU second stage's pipelined kernels at the edges of their bricks
(8 x 8 x-lines): one brick and a remainder of one line in either direction,
bricks with a single line, single cells along x, and rows longer than a
brick's skew, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import assert_close, dev, upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (1, 9, 9), (2, 8, 8), (3, 9, 8), (5, 8, 9), (4, 17, 16), (33, 1, 10), (6, 20, 1), (15, 7, 25)]


@pytest.mark.parametrize("method", [rs.ABF, rs.FRS])
@pytest.mark.parametrize("dims", DIMS)
def test_dilu_brick_edges(dims, method):
    """FP64: factors bitwise (FRS leaves diagonal blocks that need pivoting),
    the apply within the parity tests' 1e-10.  FP32: the apply, repeated,
    bitwise, and within FP32 rounding of the FP64 one (the operands' 2^-24
    times the few hundred dependent operations of a cell's chain: 1e-4)."""
    p = synth.small(*dims, seed=23, sigma=1.5)
    A = oracle.assemble(p)
    Mo = oracle.CPR(A, method=method, smoother=rs.SM_DILU)
    B = upload(A)
    r = np.random.default_rng(9).standard_normal(4 * A.n)
    z = {}
    for prec in (64, 32):
        M = rs.cpr_setup(B, rs.decouple(B, method, prec), rs.cpr_opts(smoother=rs.SM_DILU))
        if prec == 64:
            assert np.array_equal(rs.cpr_smoother_get(M), Mo.dinv2())
        z[prec] = torch.empty(4 * A.n, dtype=torch.float64, device="cuda")
        rs.cpr_apply(M, dev(r), z[prec])
        again = torch.empty_like(z[prec])
        rs.cpr_apply(M, dev(r), again)
        assert torch.equal(again, z[prec])
    assert_close(z[64].cpu().numpy(), Mo.apply(r), 1e-10)
    assert_close(z[32].cpu().numpy(), z[64].cpu().numpy(), 1e-4)
