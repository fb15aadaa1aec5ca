"""GPU: sorf_projection_fit where singular values coincide in clusters that begin and end
at, before and after the 16 rows that one workgroup orthonormalises, for factors in LDS
and in memory.

Bounds as for other coinciding values: columns orthonormal to 1e-6, squared singular
values within 4 d_rep eps64 of the largest, residuals of G u = s^2 u within the FP32
rounding of u, 2^-22 of the largest.
"""
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def sample(d_rep, clusters, seed=5):
    """Rows whose Gram matrix has each value of `clusters` [(value, count)] count times."""
    values = np.concatenate([[v] * c for v, c in clusters])
    rng = np.random.default_rng(seed)
    B, _ = np.linalg.qr(rng.standard_normal((d_rep, len(values))))
    return np.ascontiguousarray(values[:, None] * B.T, np.float32)


@pytest.mark.parametrize("d_rep,clusters,n_pca", [
    (40, [(3.0, 16), (2.0, 1)], 17),                   # one whole panel
    (40, [(3.0, 1), (2.0, 16), (1.0, 2)], 19),         # one row later
    (64, [(4.0, 15), (3.0, 2), (2.0, 17), (1.0, 3)], 37),
    (90, [(4.0, 5), (3.0, 5), (2.0, 38), (1.0, 1)], 48),   # several clusters in a panel, three panels
    (129, [(2.0, 128)], 128),
    (129, [(2.0, 100)], 129),                          # and the null space
    (1024, [(2.0, 40), (1.0, 30)], 75),
    (1025, [(3.0, 3), (2.0, 40), (1.0, 30)], 75),      # rows of a panel in memory
], ids=str)
def test_clusters(d_rep, clusters, n_pca):
    from paper_2206_01580_amd import sorf
    X = sample(d_rep, clusters)
    U, sv = sorf.projection_fit(torch.from_numpy(X).cuda(), n_pca)
    torch.cuda.synchronize()
    U, sv = U.double().cpu().numpy(), sv.cpu().numpy()
    G = X.astype(np.float64).T @ X.astype(np.float64)
    lam = np.sort(np.linalg.eigvalsh(G))[::-1][:n_pca].clip(0)
    assert np.abs(U.T @ U - np.eye(n_pca)).max() < 1e-6
    assert np.abs(sv ** 2 - lam).max() <= 4 * d_rep * 2.0 ** -52 * lam[0]
    assert np.abs(G @ U - U * sv ** 2).max() <= 2.0 ** -22 * lam[0]


def test_a_large_cluster_is_shared_out():
    """All 720 vectors of samples of rank 100, 620 of them of one value: at most 20 times the
    time of samples of full rank (more than 100 times when one workgroup has the cluster)."""
    from paper_2206_01580_amd import sorf

    def best(n):
        g = torch.Generator(device="cuda")
        g.manual_seed(n)
        X = torch.randn((n, 720), generator=g, device="cuda")
        out = []
        for _ in range(3):
            torch.cuda.synchronize()
            t = time.perf_counter()
            sorf.projection_fit(X, 720)
            torch.cuda.synchronize()
            out.append(time.perf_counter() - t)
        return min(out)

    assert best(100) <= 20 * best(1000)
