"""GPU: the feature kernels that keep the two waves of a SIMD in step (several
stacks of one molecule per workgroup), against the FP64 oracle.

Bounds of the repository: features 1e-5 of a row's maximum or, for large phases,
2^-24 (T log2 d + 3) |u| per atom; energies 1e-5 of sum |alpha Z|; gradients 1e-5
of an atom's largest entry; forces 1e-5 of a molecule's largest.
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


def problem(d, S, T, sizes, seed=3, with_J=False):
    p = W.random_problem(seed + d + S + T, d=d, n_stacks=S, n_transforms=T, n_elements=4,
                         n_mols=len(sizes), min_atoms=1, max_atoms=2, sigma=4.0)
    ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rng = np.random.default_rng(seed + d)
    A = int(ptr[-1])
    p.x = rng.standard_normal((A, d)).astype(np.float32)
    p.element = rng.integers(0, 4, A).astype(np.int32)
    p.mol_ptr = ptr
    p.alpha = rng.standard_normal(S * d).astype(np.float32)
    if with_J:
        jsz = np.asarray(sizes) * d * 3 * np.asarray(sizes)
        p.J_ptr = np.concatenate([[0], np.cumsum(jsz)]).astype(np.int64)
        p.J = (0.1 * rng.standard_normal(int(p.J_ptr[-1]))).astype(np.float32)
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


@pytest.mark.parametrize("T", [1, 2, 3])
@pytest.mark.parametrize("d,S", SHAPES + [(2, 3), (16, 200), (32, 7), (64, 4), (128, 16), (128, 48),
                                          (512, 9), (1024, 5)])
def test_gradients_and_forces(d, S, T):
    """dE/dx with and without weights, energies with dE/dx, energies with forces: one result."""
    p = problem(d, S, T, [1, 0, 2, 5, 9], with_J=True)
    sorf, model, batch = gpu(p)
    alpha = torch.from_numpy(p.alpha).cuda()
    dE = torch.linspace(-1.0, 2.0, batch.n_mols, device="cuda")
    g = sorf.backward(model, batch, alpha)
    gw = sorf.backward(model, batch, alpha, dE=dE)
    E, g2 = sorf.EnergyGrad(model)(batch, alpha)
    Ef, F = sorf.predict(model, batch, alpha, torch.from_numpy(p.J).cuda(),
                         torch.from_numpy(p.J_ptr).cuda())
    torch.cuda.synchronize()
    assert torch.equal(g, g2)
    if d >= 64:   # one kernel, one order of summation
        assert torch.equal(E, Ef)
    a64 = p.alpha.astype(np.float64)
    go = O.grad_x(p.x, p.element, p.mol_ptr, p.signs, p.bias, p.sigma, a64)
    top = np.abs(go).max(axis=1, keepdims=True)
    assert np.all(np.abs(g.double().cpu().numpy() - go) <= 1e-5 * top)
    mol = np.repeat(np.arange(batch.n_mols), np.diff(p.mol_ptr))
    w = dE.double().cpu().numpy()[mol][:, None]
    assert np.all(np.abs(gw.double().cpu().numpy() - w * go) <= 1e-5 * np.abs(w) * top + 1e-30)
    Zo = O.molecule_features(p.x, p.element, p.mol_ptr, p.signs, p.bias, p.sigma)
    scale = np.abs(Zo * p.alpha[None, :]).sum(axis=1)
    assert np.all(np.abs(E.double().cpu().numpy() - Zo @ a64) <= 1e-5 * scale)
    Fo = O.forces(go, p.J, p.J_ptr, p.mol_ptr)
    F = F.double().cpu().numpy()
    for m in range(batch.n_mols):
        s = slice(3 * p.mol_ptr[m], 3 * p.mol_ptr[m + 1])
        if p.mol_ptr[m + 1] > p.mol_ptr[m]:
            assert np.abs(F[s] - Fo[s]).max() <= 1e-5 * np.abs(Fo[s]).max()


@pytest.mark.parametrize("S", [64, 100, 128])
def test_a_batch_of_any_size_gives_the_same_bits(S):
    """One wave per atom (5000 atoms) and several (the first 50 of them)."""
    p = problem(128, S, 3, [50, 4950])
    sorf, model, batch = gpu(p)
    alpha = torch.from_numpy(p.alpha).cuda()
    few = sorf.Batch(batch.x[:50].contiguous(), batch.element[:50].contiguous(), batch.mol_ptr[:2].contiguous())
    E, g = sorf.EnergyGrad(model)(batch, alpha)
    E1, g1 = sorf.EnergyGrad(model)(few, alpha)
    torch.cuda.synchronize()
    assert torch.equal(g[:50], g1) and torch.equal(E[:1], E1)
