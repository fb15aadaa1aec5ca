"""Diagonal blocks of the Cholesky solve at the edges of their 16 x 16 parts.

Systems without refinement, so that the factorisation itself is what is
checked. A = M^T M + D I with small integer M, x a vector of small integers:
A and b = A x are exact in FP64, so x is the exact solution. The conditioning
of A is at most 1 + ||M||^2 / D (about 6 for these M), and a solve through
Cholesky factors and inverted diagonal blocks is within a small multiple of
D kappa(A) eps of x: the bound is 8 D kappa eps ||x||.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _solve(A, b, lam, refine):
    from paper_2206_01580_amd import sorf
    alpha, info = sorf.solve(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), lam, refine)
    torch.cuda.synchronize()
    return alpha.cpu().numpy(), int(info.item())


@pytest.mark.parametrize("D", [1, 2, 15, 16, 17, 31, 33, 112, 113, 127, 129, 143, 145, 257])
def test_factorisation_without_refinement(D):
    rng = np.random.default_rng(D)
    M = rng.integers(-1, 2, size=(D, D)).astype(np.float64)
    A = M.T @ M + D * np.eye(D)
    x = rng.integers(-9, 10, size=D).astype(np.float64)
    x[0] = 5.0
    a, info = _solve(np.tril(A), A @ x, 0.0, 0)
    assert info == 0
    bound = 8 * D * np.linalg.cond(A) * 2.0 ** -53 * np.linalg.norm(x)
    assert np.linalg.norm(a - x) <= bound, (np.linalg.norm(a - x), bound)


@pytest.mark.parametrize("row", [0, 15, 16, 40, 63, 64, 127, 128, 143, 144, 209])
def test_first_bad_pivot_is_reported(row):
    """Two rows with a negative diagonal: info is the first one's number, wherever
    it lies in its part, and the padding past the matrix never counts."""
    D = 210
    A = np.eye(D)
    A[row, row] = -2.0
    A[D - 1, D - 1] = -1.0
    _, info = _solve(A, np.ones(D), 0.0, 0)
    assert info == row + 1
