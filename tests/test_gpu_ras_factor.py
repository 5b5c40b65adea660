"""The RAS factorisation at the edges of its waves (16 x-lines each) and
passes (240 lines): bitwise against the oracle, with diagonal blocks that need
no pivoting (ABF scales them) and blocks that do (FRS)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (1, 16, 2), (2, 17, 3), (33, 15, 1), (20, 20, 10), (2, 240, 2), (3, 241, 2)]


@pytest.mark.parametrize("method", [rs.ABF, rs.FRS])
@pytest.mark.parametrize("dims", DIMS)
def test_ras_factors_bitwise(dims, method):
    A = oracle.assemble(synth.small(*dims, seed=29, sigma=1.5))
    Mo = oracle.CPR(A, method=method, smoother=rs.SM_RAS)
    B = upload(A)
    M = rs.cpr_setup(B, rs.decouple(B, method, 64), rs.cpr_opts(smoother=rs.SM_RAS))
    assert np.array_equal(rs.cpr_smoother_get(M), Mo.dinv2())
