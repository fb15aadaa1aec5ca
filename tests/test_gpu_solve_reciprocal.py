"""GPU: the factorisation alone (no refinement) is accurate to a few roundings.

512 systems of two equations in one block-diagonal matrix: zeros stay exact, so each is
solved by itself. [[a, b], [b, c]] with b^2 = 1e-8 a c and right-hand side (1, 0): the
second unknown is -(b / a) / sqrt(d) / sqrt(d), d = c - b^2 / a, a chain of products
without a sum that matters (d is c to 1e-8). With u = 2^-53 and a reciprocal and a
reciprocal square root good to 2 u, its relative error is at most 2 u (1 / a), u (b times
it), 2 x (2 u + u) (the two roots, each times something, their errors equal), u (d) and
3 u (the products of the sweeps): 13 u. Errors spread evenly over these ranges and
independent, the root's counted as one of 4 u, have a root mean square of
sqrt((4 + 1 + 16 + 2 + 1 + 3) / 3) u = 3 u; the 512 values are held to 4 u.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_two_equations_many_times():
    from paper_2206_01580_amd import sorf
    rng = np.random.default_rng(4)
    n = 512
    a, c = rng.uniform(1, 4, n), rng.uniform(1, 4, n)
    b = 1e-4 * np.sqrt(a * c) * rng.choice([-1.0, 1.0], n)
    G = np.zeros((2 * n, 2 * n))
    i = 2 * np.arange(n)
    G[i, i], G[i + 1, i], G[i + 1, i + 1] = a, b, c
    y = np.tile([1.0, 0.0], n)
    x = sorf.Solver(2 * n)(torch.from_numpy(G).cuda(), torch.from_numpy(y).cuda(), 0.0, n_refine=0)
    torch.cuda.synchronize()
    x = x.cpu().numpy()[1::2].astype(np.longdouble)
    a, b, c = (v.astype(np.longdouble) for v in (a, b, c))
    exact = -b / (a * c - b * b)
    err = (np.abs(x / exact - 1)).astype(np.float64) * 2.0 ** 53
    assert err.max() <= 13
    assert np.sqrt((err ** 2).mean()) <= 4
