"""Calls that meet the end of device memory: what they report, and that the
handle they ran on still works."""
from contextlib import contextmanager

import pytest
import torch

import synth
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

GiB = 1 << 30


def test_dilu_refuses_a_grid_before_it_takes_memory():
    """A column of 2^25 cells in FP64, where the set-up takes 2^25 - 4."""
    nz = 1 << 25
    rp, ci = rs.pattern(1, 1, nz)
    vals = torch.zeros(16 * ci.numel(), dtype=torch.float64, device="cuda").view(-1, 16)
    row = torch.repeat_interleave(torch.arange(nz, device="cuda"), torch.diff(rp).long())
    vals[ci == row] = torch.eye(4, dtype=torch.float64, device="cuda").reshape(1, 16)
    del row
    A = rs.bsr_create(1, 1, nz, rp, ci, vals.view(-1))
    D = rs.decouple(A, rs.ABF, 64)
    before = sum(rs.pool_usage())
    with pytest.raises(rs.RsError) as e:
        rs.cpr_setup(A, D)
    assert e.value.status == -1
    assert sum(rs.pool_usage()) == before
    del A, D, rp, ci, vals
    torch.cuda.empty_cache()
    rs.pool_trim()


def take(target):
    """Blocks of device memory that leave about `target` bytes free."""
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


@pytest.fixture(scope="module")
def small_card():
    """Most of the device's memory taken once for all the tests below."""
    held = take(24 * GiB)
    yield
    held.clear()
    torch.cuda.empty_cache()


@contextmanager
def free_memory(target):
    held = take(target)
    try:
        yield
    finally:
        held.clear()
        torch.cuda.empty_cache()
        rs.pool_trim()


def test_gmres_restart_that_does_not_fit(small_card):
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
    with free_memory(basis + z // 2 - 9 * 8 * N):
        info = rs.gmres_solve(A, M, dp.b, x1, rs.gmres_opts(restart=32, rtol=1e-10), check=False)
        assert info["return"] == -3
        assert rs.gmres_solve(A, M, dp.b, x1, short)["return"] == 0
        assert torch.equal(x0, x1)
    assert rs.gmres_solve(A, M, dp.b, x1, rs.gmres_opts(restart=32, rtol=1e-10))["return"] == 0


@pytest.mark.parametrize("use", ["gmres", "bicgstab", "apply"])
@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("dims", [(96, 96, 64), (100, 136, 64)])
def test_dilu_without_room_for_the_brick_order(small_card, dims, prec, use):
    """DILU where memory ends half a copy of its blocks short of what it takes
    with room to spare, at the solve or at the set-up: it goes without the copy
    (which is a matter of order only), to the same result.  Bricks of 8 x 4 lines
    and of 8 x 8."""
    dp = rs.DeviceProblem(synth.small(*dims, seed=41))
    n, A = dp.n, dp.bsr()
    D = rs.decouple(A, rs.ABF, prec)

    def run(x):
        M = rs.cpr_setup(A, D)
        if use == "gmres":
            assert rs.gmres_solve(A, M, dp.b, x, rs.gmres_opts(restart=32, zero_guess=1, rtol=1e-10))["return"] == 0
        elif use == "bicgstab":
            assert rs.bicgstab_solve(A, M, dp.b, x, rs.bicgstab_opts(zero_guess=1, rtol=1e-10))["return"] == 0
        else:
            rs.cpr_apply(M, dp.b, x)
        return M

    x0, x1 = torch.empty_like(dp.b), torch.empty_like(dp.b)
    before = rs.pool_usage()[0]
    M = run(x0)
    taken, copy = rs.pool_usage()[0] - before, prec // 8 * 7 * 16 * n
    del M
    # (at the set-up its temporaries, about 110 bytes a cell, come on top)
    with free_memory(taken - copy // 2 + (110 * n if use == "apply" else 0)):
        M = run(x1)
        assert torch.equal(x0, x1)
