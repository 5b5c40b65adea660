"""The chained factorisation of RAS with overlap 1 at the edges of its launch
variants (96, 160 and 224 lines a layer, and one more of each) and of its rule
(170 layers, 85 of more than 160 lines, and one more of each), with one, two
and many layers, single columns and rows: the owned factors bitwise against the
oracle's, the apply (which uses all three stages' factors) as the overlapping
RAS tests compare it."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev, relerr, upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (1, 1, 2), (3, 96, 3), (3, 97, 2), (2, 160, 2), (2, 161, 3), (2, 224, 2), (2, 225, 2), (40, 3, 60),
        (5, 7, 130), (3, 5, 170), (3, 5, 171), (1, 161, 85), (1, 161, 86)]


@pytest.mark.parametrize("method", [rs.ABF, rs.FRS])
@pytest.mark.parametrize("dims", DIMS)
def test_chained_factors(dims, method):
    A = oracle.assemble(synth.small(*dims, seed=43, sigma=1.5))
    Mo = oracle.CPR(A, method=method, smoother=rs.SM_RAS1)
    B = upload(A)
    r = np.random.default_rng(13).standard_normal(4 * A.n)
    ref = Mo.apply(r)
    for prec, tol in ((64, 1e-10), (32, 1e-4)):
        M = rs.cpr_setup(B, rs.decouple(B, method, prec), rs.cpr_opts(smoother=rs.SM_RAS1))
        if prec == 64:
            assert np.array_equal(rs.cpr_smoother_get(M), Mo.dinv2())
        z = torch.empty(4 * A.n, dtype=torch.float64, device="cuda")
        rs.cpr_apply(M, dev(r), z)
        assert relerr(z.cpu().numpy(), ref) <= tol
