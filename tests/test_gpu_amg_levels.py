"""Levels set up by one workgroup (at most 8192 rows), the Galerkin rows by 16
lanes, and what is past either: the row limit and one more, levels that do not
coarsen, coarse rows of more than 16 and more than 32 columns (sigma 4), FP32.
Hierarchies bitwise against the oracle's, with the second level's strengths
and keys of several levels in them."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev, upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

CASES = [((64, 16, 8), 1.0, {}), ((2731, 3, 1), 1.0, {}), ((40, 40, 20), 4.0, {}), ((130, 17, 9), 4.0, {}),
         ((40, 40, 20), 4.0, dict(theta=0.8)), ((20, 20, 10), 2.0, dict(theta=0.95)), ((9, 2, 1), 0.0, {}),
         ((12, 12, 6), 1.0, dict(max_row_sum=0.0)), ((1, 1, 9), 1.0, {})]


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("dims,sigma,kw", CASES)
def test_levels_bitwise(dims, sigma, kw, prec):
    p = synth.small(*dims, seed=37, sigma=sigma)
    A = oracle.assemble(p)
    ho = oracle.CPR(A, smoother=rs.SM_BJ, coarse_n=8, **kw).amg()
    B = upload(A)
    M = rs.cpr_setup(B, rs.decouple(B, rs.ABF, prec), rs.cpr_opts(smoother=rs.SM_BJ, coarse_n=8, **kw))
    if prec == 32:                      # the FP32 decoupling rounds the pressure entries: a hierarchy of its own
        z = torch.empty(4 * A.n, dtype=torch.float64, device="cuda")
        rs.cpr_apply(M, dev(p.b), z)
        assert torch.isfinite(z).all()
        for l in range(rs.cpr_nlevels(M) - 1):
            L, C = rs.cpr_level(M, l), rs.cpr_level(M, l + 1)
            assert L["agg"].max() == C["n"] - 1 and C["rp"][-1] == C["nnz"]
            assert all((np.diff(C["ci"][C["rp"][i]:C["rp"][i + 1]]) > 0).all() for i in range(C["n"]))
        return
    assert rs.cpr_nlevels(M) == ho.nlevels
    for l in range(ho.nlevels):
        Lo, Lg = ho.level(l), rs.cpr_level(M, l)
        for k in ("n", "nnz", "rp", "ci", "a", "dl1") + (("agg",) if l < ho.nlevels - 1 else ()):
            assert np.array_equal(Lo[k], Lg[k]), (l, k)
