"""GPU: sorf_projection_fit on samples whose Gram matrix has entries of very different
size: features far down the FP32 range, and remainders of low-rank samples that are
rounding only. The results are finite and as good as for any other sample.

Bounds as for coinciding values: columns orthonormal to 1e-6, squared singular values
within 4 d_rep eps64 of the largest, residuals of G u = s^2 u within the FP32 rounding
of u, 2^-22 of the largest.
"""
import math

import numpy as np
import pytest
import torch

from oracle import fchl19_oracle as FO

pytestmark = pytest.mark.gpu

ENERGY = dict(n2=23, n3=22, eta2=0.27, eta3=5.6, N2=2.78, N3=2.1, c3=60.1, zeta=math.pi, rcut=6.0)
WATER = np.array([[0.0, 0.0, 0.117], [0.0, 0.757, -0.467], [0.0, -0.757, -0.467]])


def water(centre):
    """FCHL19 rows of one atom of 120 jittered water molecules (elements O = 0, H = 1)."""
    rng = np.random.default_rng(11)
    R = (WATER[None] + 0.05 * rng.standard_normal((120, 3, 3))).reshape(-1, 3).astype(np.float32)
    rho, _ = FO.fchl19(R, np.tile(np.array([0, 1, 1], np.int32), 120), 3 * np.arange(121), 2, ENERGY)
    return rho.numpy().astype(np.float32)[centre::3]


def make(kind):
    rng = np.random.default_rng(0)
    if kind == "subnormal":     # three features below the smallest normal FP32 number
        X = rng.standard_normal((50, 6))
        X[:, 3:] *= 1e-40
    elif kind == "graded":      # from 1 down to 1e-38
        X = rng.standard_normal((60, 40)) * 10.0 ** -np.linspace(0, 38, 40)
    elif kind == "small":       # rank 20 at 1e-32: the remainder is rounding, 1e-80
        X = np.repeat(rng.standard_normal((20, 40)), 3, axis=0) * 1e-32
    elif kind == "large":       # rank 20 at 1e35
        X = np.repeat(rng.standard_normal((20, 40)), 3, axis=0) * 1e35
    elif kind == "tail":        # rank 1 with a Gaussian tail
        X = rng.standard_normal((30, 1)) * np.exp(-0.05 * np.arange(60.0) ** 2)
    else:
        return water(int(kind[-1]))
    return X.astype(np.float32)


@pytest.mark.parametrize("kind", ["subnormal", "graded", "small", "large", "tail", "water0", "water1"])
def test_range(kind):
    from paper_2206_01580_amd import sorf
    X = make(kind)
    n_pca = min(32, X.shape[1])
    U, sv = sorf.projection_fit(torch.from_numpy(X).cuda(), n_pca)
    torch.cuda.synchronize()
    U, sv = U.double().cpu().numpy(), sv.cpu().numpy()
    assert np.isfinite(U).all() and np.isfinite(sv).all()
    unit = float(np.abs(X).max())   # the bounds below are relative: keep numpy's side in range
    G = (X / np.float64(unit)).T @ (X / np.float64(unit))
    lam = np.sort(np.linalg.eigvalsh(G))[::-1][:n_pca].clip(0)
    sv = sv / unit
    assert np.abs(U.T @ U - np.eye(n_pca)).max() < 1e-6
    assert np.abs(sv ** 2 - lam).max() <= 4 * X.shape[1] * 2.0 ** -52 * lam[0]
    assert np.abs(G @ U - U * sv ** 2).max() <= 2.0 ** -22 * lam[0]
