"""Coarsest inverse at the edges of its register tiles (108, 156, 192, 224 and
256 rows): against LAPACK on matrices that pivot, the order of a tie, and a
matrix that holds a NaN."""
import numpy as np
import pytest
import torch

from gpu_util import dev
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu


def _inverse(a):
    x = torch.full(a.shape, 7.0, dtype=torch.float64, device="cuda")
    rs.dense_inverse(dev(np.ascontiguousarray(a)), x)
    return x.cpu().numpy()


@pytest.mark.parametrize("n", [5, 31, 110, 158, 191, 192, 193, 208, 223, 224, 225, 240, 255, 256])
def test_against_lapack(n):
    rng = np.random.default_rng(n)
    D = rng.standard_normal((n, n)) + np.diag(n + rng.random(n))
    for A in (D[rng.permutation(n)], D[::-1], rng.standard_normal((n, n))):
        X = _inverse(A)
        bound = 1e-14 * n * np.linalg.cond(A)        # n steps, each within a few units of 2^-53
        assert np.abs(A @ X - np.eye(n)).max() <= bound
        ref = np.linalg.inv(A)
        assert np.abs(X - ref).max() <= bound * np.abs(ref).max()


@pytest.mark.parametrize("n", [192, 224, 256])
def test_ties_and_permutations(n):
    """Entries of equal magnitude everywhere (powers of two and small whole
    numbers, so exact), and a permutation, whose inverse is its transpose."""
    H = np.array([[1.0]])
    while H.shape[0] * 2 <= n:
        H = np.block([[H, H], [H, -H]])
    m = H.shape[0]
    A = np.eye(n)
    A[:m, :m] = H
    want = np.eye(n)
    want[:m, :m] = H / m
    assert np.array_equal(_inverse(A), want)
    P = np.eye(n)[np.random.default_rng(n).permutation(n)]
    assert np.array_equal(_inverse(P), P.T)


@pytest.mark.parametrize("n", [40, 110, 180, 220, 250, 256])
def test_nan_and_zero_are_refused(n):
    for v in (np.nan, 0.0):
        A = np.eye(n) * 2.0
        A[:, n // 2] = v
        with pytest.raises(rs.RsError):
            _inverse(A)
        with pytest.raises(rs.RsError):
            _inverse(np.full((n, n), v))
