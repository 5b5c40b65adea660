"""The Galerkin product with a thread per coarse row (more than 262144 of them),
from the grid and from a CSR level: every entry is the sum of the finer level's
entries in row order, so adding those one after another gives the same bits."""
import numpy as np
import pytest
import torch

from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu


def system(nx, ny, nz, sigma):
    """Diagonal blocks on the 7-point pattern: an M-matrix in every unknown.
    sigma 0: coupled strongly along z and weakly across it, so that aggregates
    are short columns and two levels have many rows; else log-normal weights,
    which give long coarse rows."""
    rp, ci = rs.pattern(nx, ny, nz)
    n, g = nx * ny * nz, torch.Generator(device="cuda").manual_seed(47)
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.diff(rp).long())
    w = torch.rand(ci.numel(), dtype=torch.float64, device="cuda", generator=g) + 0.5
    step = (ci - row).abs()
    if sigma:
        w = torch.exp(sigma * torch.randn(ci.numel(), dtype=torch.float64, device="cuda", generator=g))
    else:
        w[step < nx * ny] *= 0.02
    w[step == 0] = 0.0
    v = -w
    v[step == 0] = 1e-3 + torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, row, w)
    return rp, ci, (v[:, None] * torch.eye(4, dtype=torch.float64, device="cuda").reshape(1, 16)).reshape(-1)


def assert_product(F, C):
    agg, nc = F["agg"], C["n"]
    row = np.repeat(np.arange(F["n"]), np.diff(F["rp"]))
    I, J = agg[row], agg[F["ci"]]
    on = (I >= 0) & (J >= 0)
    crow = np.repeat(np.arange(nc), np.diff(C["rp"]))
    ckey = torch.as_tensor(crow * nc + C["ci"]).cuda()
    assert (ckey[1:] > ckey[:-1]).all()
    key = torch.as_tensor(I[on].astype(np.int64) * nc + J[on]).cuda()
    at = torch.searchsorted(ckey, key)
    assert torch.equal(ckey[at], key)                  # no entry is missing
    at = at.cpu().numpy()
    assert np.bincount(at, minlength=C["nnz"]).min() > 0   # and none is made up
    assert np.array_equal(np.bincount(at, F["a"][on], C["nnz"]), C["a"])
    l1 = np.bincount(crow, np.abs(C["a"]), nc)
    diag = C["a"][C["ci"] == crow]
    assert np.array_equal(C["dl1"], np.where(diag < 0, -l1, l1))


@pytest.mark.parametrize("dims,sigma", [((170, 170, 170), 0.0), ((140, 150, 130), 4.0)])
def test_thread_per_coarse_row(dims, sigma):
    rp, ci, vals = system(*dims, sigma)
    A = rs.bsr_create(*dims, rp, ci, vals)
    D = rs.bsr_attach_decouple(A, vals, rs.FRS, 64)    # rows of diagonal blocks: the pressure rows as they are
    M = rs.cpr_setup(A, D, rs.cpr_opts(smoother=rs.SM_BJ))
    L = [rs.cpr_level(M, l) for l in range(2 if sigma else 3)]
    assert all(l["n"] > 262144 for l in L)
    for F, C in zip(L, L[1:]):
        assert_product(F, C)
    if sigma:
        assert np.diff(L[1]["rp"]).max() > 16          # past the list that a thread keeps in LDS
    del M, D, A
    rs.pool_trim()
