"""The Krylov solvers' one-launch reductions: vectors of a single pair of
entries, of one workgroup (512 pairs) and one more, of every workgroup exactly
(512 x 512 pairs) and beyond; Krylov spaces past 8 and 16 vectors."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev, relerr, upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (16, 16, 1), (257, 1, 1), (15, 17, 4), (128, 64, 16), (128, 64, 17)]


@pytest.mark.parametrize("solver", ["gmres", "bicgstab"])
@pytest.mark.parametrize("dims", DIMS)
def test_three_steps_match_oracle(dims, solver):
    """Three steps in FP64 against the oracle's: the dots differ in the order
    of their sums only (2^-53 sqrt(5e5), 1e-13, with room for the steps'
    cancellation: 1e-11); repeated, bitwise."""
    p = synth.small(*dims, seed=31)
    A = oracle.assemble(p)
    Mo = oracle.CPR(A, smoother=rs.SM_BJ)
    xo, io = (oracle.gmres if solver == "gmres" else oracle.bicgstab)(A, p.b, Mo, rtol=1e-13, maxit=3)
    B = upload(A)
    M = rs.cpr_setup(B, rs.decouple(B, rs.ABF, 64), rs.cpr_opts(smoother=rs.SM_BJ))
    solve, opts = (rs.gmres_solve, rs.gmres_opts) if solver == "gmres" else (rs.bicgstab_solve, rs.bicgstab_opts)
    xs = []
    for _ in range(2):
        x = torch.full((4 * A.n,), float("nan"), dtype=torch.float64, device="cuda")
        info = solve(B, M, dev(p.b), x, opts(rtol=1e-13, maxit=3, zero_guess=1), check=False)
        assert info["iters"] == io["iters"] and info["return"] == io["status"]
        xs.append(x)
    assert torch.equal(xs[0], xs[1])
    xg = xs[0].cpu().numpy()
    assert relerr(xg, xo) <= 1e-11
    true = np.linalg.norm(p.b - oracle.spmv(A, xg)) / np.linalg.norm(p.b)
    assert abs(true - info["relres"]) <= 1e-14 + 1e-12 * true


@pytest.mark.parametrize("maxit", [9, 17, 32])
def test_long_cycles(maxit):
    """Cycles whose passes run over more than 8 and 16 vectors: the rotations'
    estimate is the true residual to rounding (the basis stays orthogonal)."""
    p = synth.small(24, 20, 9, seed=33, sigma=2.0)
    A = oracle.assemble(p)
    B = upload(A)
    M = rs.cpr_setup(B, rs.decouple(B, rs.ABF, 64),
                     rs.cpr_opts(smoother=rs.SM_BJ, max_levels=1, lu_max=1, coarse_sweeps=1))
    x = torch.empty(4 * A.n, dtype=torch.float64, device="cuda")
    info = rs.gmres_solve(B, M, dev(p.b), x, rs.gmres_opts(restart=32, rtol=0.0, maxit=maxit, zero_guess=1),
                          check=False)
    assert info["iters"] == maxit and info["return"] == rs.RS_NOT_CONVERGED
    true = np.linalg.norm(p.b - oracle.spmv(A, x.cpu().numpy())) / np.linalg.norm(p.b)
    assert true < 1.0 and abs(true - info["est_relres"]) <= 1e-13 and abs(true - info["relres"]) <= 1e-13
