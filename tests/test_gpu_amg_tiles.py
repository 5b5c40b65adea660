"""The fine-level independent-set rounds at the edges of their tiles (60 x 8 x
4 cells) and the two-launch scan past one workgroup (4096 entries): hierarchies
bitwise against the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 300), (60, 8, 4), (61, 9, 5), (59, 7, 3), (121, 1, 6), (2, 33, 9), (64, 8, 8), (16, 16, 17), (130, 17, 9)]


@pytest.mark.parametrize("sigma", [0.5, 2.0])
@pytest.mark.parametrize("dims", DIMS)
def test_hierarchy_bitwise(dims, sigma):
    A = oracle.assemble(synth.small(*dims, seed=37, sigma=sigma))
    Mo = oracle.CPR(A, smoother=rs.SM_BJ, coarse_n=8)
    B = upload(A)
    M = rs.cpr_setup(B, rs.decouple(B, rs.ABF, 64), rs.cpr_opts(smoother=rs.SM_BJ, coarse_n=8))
    ho = Mo.amg()
    assert rs.cpr_nlevels(M) == ho.nlevels
    for l in range(ho.nlevels):
        Lo, Lg = ho.level(l), rs.cpr_level(M, l)
        for k in ("n", "nnz", "rp", "ci", "a", "dl1") + (("agg",) if l < ho.nlevels - 1 else ()):
            assert np.array_equal(Lo[k], Lg[k]), (l, k)
