"""The assembly, gradient and transpose kernels at the edges of their tiles
(16 x 4 x 4 cells of a workgroup, 16 cells of a workgroup in a row): single
cells along an axis, one past a tile in each direction, ragged remainders,
against the oracle; every pointer aligned to a double only."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import assert_close, dev, upload
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (1, 7, 3), (16, 4, 4), (17, 5, 5), (33, 3, 9), (5, 1, 6), (15, 9, 1)]


def _odd(a, dtype=torch.float64):
    """The values on a pointer that is 8 but not 16 bytes aligned."""
    a = torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).reshape(-1)
    buf = torch.empty(a.numel() + 1, dtype=dtype, device="cuda")
    buf[1:] = a.cuda()
    return buf[1:]


@pytest.mark.parametrize("dims", DIMS)
def test_assembly_and_gradient_tiles(dims):
    nx, ny, nz = dims
    p = synth.small(nx, ny, nz, seed=31, sigma=1.5)
    n = p.n
    A = oracle.assemble(p)
    rp, _ = rs.pattern(nx, ny, nz)
    wc, wu = dev(p.well_cell, torch.int32), dev(p.well_u)
    logk, Mf, Mb, B = _odd(p.logk), _odd(p.Mf), _odd(p.Mb), _odd(p.B)
    vals = _odd(np.zeros(16 * A.nnzb))
    rs.assemble(nx, ny, nz, logk, p.kvkh, p.tscale, Mf, Mb, B, p.dt, wc, wu, rp, vals)
    # the products and sums of the definition; exp may differ by an ulp
    ref = A.v.reshape(-1)
    assert np.abs(vals.cpu().numpy() - ref).max() <= 1e-14 * np.abs(ref).max()
    rng = np.random.default_rng(5)
    lam, x = rng.standard_normal(4 * n), rng.standard_normal(4 * n)
    G = _odd(np.zeros(16 * A.nnzb))
    H = upload(A)
    rs.grad_vals(H, _odd(lam), _odd(x), G)
    rows = np.repeat(np.arange(n), np.diff(A.rp))
    Gref = -lam.reshape(n, 4)[rows][:, :, None] * x.reshape(n, 4)[A.ci][:, None, :]
    assert np.array_equal(G.cpu().numpy().reshape(-1, 4, 4), Gref)
    g = _odd(np.zeros(n))
    rs.grad_logk(nx, ny, nz, logk, p.kvkh, p.tscale, Mf, Mb, wc, wu, rp, G, g)
    # 100 roundings of a sum over a cell's faces, relative to its largest terms
    gref = oracle.grad_logk(p, lam, x)
    assert_close(g.cpu().numpy(), gref, 100 * 2.0 ** -52 * 10)


@pytest.mark.parametrize("attached", [False, True])
@pytest.mark.parametrize("dims", DIMS)
def test_transpose_tiles(dims, attached):
    """A^T lambda = w through the adjoint solve, with A's own copy and with
    attached values: the true residual of the transposed system."""
    p = synth.small(*dims, seed=33, sigma=1.0)
    A = oracle.assemble(p)
    H = upload(A)
    if attached:
        vals = dev(A.v.reshape(-1))
        D = rs.bsr_attach_decouple(H, vals, rs.ABF, 64)
    w = np.random.default_rng(7).standard_normal(4 * A.n)
    lam = torch.zeros(4 * A.n, dtype=torch.float64, device="cuda")
    info = rs.adjoint_solve(H, dev(w), lam, opts=rs.gmres_opts(rtol=1e-11, maxit=200))
    assert info["return"] == 0
    res = np.linalg.norm(w - A.dense().T @ lam.cpu().numpy())
    assert res <= 2e-11 * np.linalg.norm(w)
