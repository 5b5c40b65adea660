"""The RAS sweeps at the edges of their strips (48 lines; 32 in FP64 while
every strip has a CU): one strip and a remainder of one line, columns fewer
and more than the eight that the backward sweep stores together, levels fewer
than the loads in flight, layers taller than 240 lines."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import assert_close, dev, upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (1, 49, 2), (7, 48, 2), (8, 49, 3), (9, 97, 2), (40, 16, 3), (17, 33, 1), (3, 65, 2), (2, 300, 2),
        (5, 96, 90)]


@pytest.mark.parametrize("smoother", [rs.SM_RAS, rs.SM_RAS1])
@pytest.mark.parametrize("dims", DIMS)
def test_ras_strip_edges(dims, smoother):
    """The apply in FP64 within the parity tests' 1e-10 of the oracle's (layer
    RAS) and of the FP32 one within FP32 rounding (2^-24 times the few hundred
    dependent operations of a cell's chain: 1e-4); repeated, bitwise."""
    p = synth.small(*dims, seed=41, sigma=1.5)
    A = oracle.assemble(p)
    B = upload(A)
    r = np.random.default_rng(11).standard_normal(4 * A.n)
    z = {}
    for prec in (64, 32):
        M = rs.cpr_setup(B, rs.decouple(B, rs.ABF, prec), rs.cpr_opts(smoother=smoother))
        z[prec] = torch.empty(4 * A.n, dtype=torch.float64, device="cuda")
        rs.cpr_apply(M, dev(r), z[prec])
        again = torch.empty_like(z[prec])
        rs.cpr_apply(M, dev(r), again)
        assert torch.equal(again, z[prec])
    if smoother == rs.SM_RAS:
        assert_close(z[64].cpu().numpy(), oracle.CPR(A, smoother=smoother).apply(r), 1e-10)
    assert_close(z[32].cpu().numpy(), z[64].cpu().numpy(), 1e-4)
