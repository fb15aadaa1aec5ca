"""GPU: the feature kernels that keep the two waves of a SIMD in step (several
stacks of one molecule per workgroup), against the FP64 oracle.

Bounds of the repository: features 1e-5 of a row's maximum or, for large phases,
2^-24 (T log2 d + 3) |u| per atom; energies 1e-5 of sum |alpha Z|.
"""
import numpy as np
import pytest
import torch

from oracle import sorf_oracle as O
from paper_2206_01580_amd import workloads as W

pytestmark = pytest.mark.gpu

# d, stacks: whole workgroups of one molecule (64 vectors or a multiple), and one stack more
SHAPES = [(64, 128), (64, 129), (64, 256), (128, 64), (128, 65), (128, 128), (128, 256), (256, 32),
          (256, 33), (256, 64)]


def problem(d, S, T, sizes, seed=3):
    p = W.random_problem(seed + d + S + T, d=d, n_stacks=S, n_transforms=T, n_elements=4,
                         n_mols=len(sizes), min_atoms=1, max_atoms=2, sigma=4.0)
    ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rng = np.random.default_rng(seed + d)
    A = int(ptr[-1])
    p.x = rng.standard_normal((A, d)).astype(np.float32)
    p.element = rng.integers(0, 4, A).astype(np.int32)
    p.mol_ptr = ptr
    p.alpha = rng.standard_normal(S * d).astype(np.float32)
    return p


def gpu(p):
    from paper_2206_01580_amd import sorf
    return sorf, sorf.Model.from_problem(p), sorf.Batch.from_problem(p)


# sizes: no, one, two, three atoms; a chunk of the energies and one atom more
@pytest.mark.parametrize("T", [1, 2, 3])
@pytest.mark.parametrize("d,S", SHAPES)
def test_features_and_energies(d, S, T):
    p = problem(d, S, T, [1, 0, 2, 3, 32, 33, 18, 65, 0])
    sorf, model, batch = gpu(p)
    Z = sorf.forward(model, batch)
    alpha = torch.from_numpy(p.alpha).cuda()
    E = sorf.predict(model, batch, alpha)
    torch.cuda.synchronize()
    Zo = O.molecule_features(p.x, p.element, p.mol_ptr, p.signs, p.bias, p.sigma)
    Z = Z.double().cpu().numpy()
    assert np.all(np.abs(Z - Zo).max(axis=1) <= 1e-5 * np.abs(Zo).max(axis=1))
    scale = np.abs(Zo * p.alpha[None, :]).sum(axis=1)
    assert np.all(np.abs(E.double().cpu().numpy() - Zo @ p.alpha.astype(np.float64)) <= 1e-5 * scale)
