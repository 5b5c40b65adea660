"""Hierarchies past the sizes that one workgroup sets up (8192 rows), against the
oracle bit for bit: the fine level's independent-set tiles (60 x 8 x 4 cells) at
their edges, the two passes that grids filling less than a third of them take,
the two-launch scan, and a second level of more than 8192 rows."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

EDGES = [(60, 40, 4), (61, 41, 5), (59, 39, 7), (121, 9, 8), (120, 8, 9), (180, 16, 3), (130, 70, 1)]
THIN = [(20, 24, 20), (19, 24, 20), (1, 96, 100), (2, 70, 63), (9001, 1, 1), (1, 9001, 1), (1, 1, 9001), (33, 1, 260)]
SECOND = [(60, 60, 30), (80, 60, 20)]


@pytest.mark.parametrize("sigma", [0.5, 2.0])
@pytest.mark.parametrize("dims", EDGES + THIN + SECOND)
def test_hierarchy_bitwise(dims, sigma):
    A = oracle.assemble(synth.small(*dims, seed=37, sigma=sigma))
    ho = oracle.CPR(A, smoother=rs.SM_BJ, coarse_n=8).amg()
    if dims in SECOND:
        assert ho.level(1)["n"] > 8192
    B = upload(A)
    M = rs.cpr_setup(B, rs.decouple(B, rs.ABF, 64), rs.cpr_opts(smoother=rs.SM_BJ, coarse_n=8))
    assert rs.cpr_nlevels(M) == ho.nlevels
    for l in range(ho.nlevels):
        Lo, Lg = ho.level(l), rs.cpr_level(M, l)
        for k in ("n", "nnz", "rp", "ci", "a", "dl1") + (("agg",) if l < ho.nlevels - 1 else ()):
            assert np.array_equal(Lo[k], Lg[k]), (l, k)
