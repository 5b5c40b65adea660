"""Calls that meet the end of device memory: what they report, and that the
handle they ran on still works."""
import pytest
import torch

import synth
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

GiB = 1 << 30


def leave_free(target):
    """Take device memory until about `target` bytes of it are free."""
    torch.cuda.synchronize()
    rs.pool_trim()
    torch.cuda.empty_cache()
    held = []
    for _ in range(64):
        left = torch.cuda.mem_get_info()[0] - target
        if left < (4 << 20):
            break
        held.append(torch.empty(min(left, 16 * GiB) >> 21 << 21, dtype=torch.uint8, device="cuda"))
    return held


def test_gmres_restart_that_does_not_fit():
    """A longer restart runs out of memory after its basis has been allocated;
    the handle then solves with the former restart, and with a longer one that
    fits."""
    dp = rs.DeviceProblem(synth.small(64, 64, 60, seed=41))
    N, A = 4 * dp.n, dp.bsr()
    M = rs.cpr_setup(A, rs.decouple(A, rs.ABF, 64), rs.cpr_opts(smoother=rs.SM_RAS))
    x0, x1 = torch.zeros_like(dp.b), torch.zeros_like(dp.b)
    short = rs.gmres_opts(restart=4, rtol=1e-10)
    assert rs.gmres_solve(A, M, dp.b, x0, short)["return"] == 0
    basis, z = 8 * N * 33, 8 * N * 32
    # room for the basis and for half of the preconditioned vectors; what the
    # short restart held (9 vectors) comes back to the pool meanwhile
    held = leave_free(basis + z // 2 - 9 * 8 * N)
    info = rs.gmres_solve(A, M, dp.b, x1, rs.gmres_opts(restart=32, rtol=1e-10), check=False)
    assert info["return"] == -3
    assert rs.gmres_solve(A, M, dp.b, x1, short)["return"] == 0
    assert torch.equal(x0, x1)
    del held
    torch.cuda.empty_cache()
    assert rs.gmres_solve(A, M, dp.b, x1, rs.gmres_opts(restart=32, rtol=1e-10))["return"] == 0
