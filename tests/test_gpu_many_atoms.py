"""GPU: calls with more atoms or molecules than the workgroups of one launch (HIP takes
fewer than 2^32 threads in one): the last ones, and those on both sides of a launch's
end, have bitwise the results they have in a small batch.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def model(S, T, seed):
    from paper_2206_01580_amd import sorf
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    signs = torch.randint(-2 ** 31, 2 ** 31, (2, T, S, 2), generator=g, device="cuda").to(torch.int32)
    bias = torch.rand((2, S * 64), generator=g, device="cuda") * 6.28
    return sorf.Model(64, S, T, 2, 4.0, signs, bias), torch.randn(S * 64, generator=g, device="cuda")


def atoms(n, seed):
    """n molecules of one atom."""
    from paper_2206_01580_amd import sorf
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return sorf.Batch(torch.randn((n, 64), generator=g, device="cuda"),
                      torch.randint(0, 2, (n,), generator=g, device="cuda").to(torch.int32),
                      torch.arange(n + 1, device="cuda", dtype=torch.int64))


def some(batch, idx):
    from paper_2206_01580_amd import sorf
    return sorf.Batch(batch.x[idx].contiguous(), batch.element[idx].contiguous(),
                      torch.arange(len(idx) + 1, device="cuda", dtype=torch.int64))


def test_gradients():
    """2^23 + 3 atoms, 257 stacks of 64: a workgroup of 512 threads each."""
    from paper_2206_01580_amd import sorf
    n = 2 ** 23 + 3
    m, alpha = model(257, 1, 1)
    b = atoms(n, 2)
    idx = torch.tensor([0, 2 ** 22 - 1, 2 ** 22, 2 ** 23 - 1, 2 ** 23, n - 1], device="cuda")
    few = some(b, idx)
    dE = torch.linspace(-1.0, 2.0, n, device="cuda")
    E, g = sorf.EnergyGrad(m)(b, alpha)
    E1, g1 = sorf.EnergyGrad(m)(few, alpha)
    assert torch.equal(g[idx], g1) and torch.equal(E[idx], E1)
    del E, g
    g = sorf.backward(m, b, alpha, dE=dE)
    g1 = sorf.backward(m, few, alpha, dE=dE[idx].contiguous())
    assert torch.equal(g[idx], g1)


def test_energies():
    """2^18 + 5 molecules, 4096 stacks of 64: 8.6 million workgroups of 512 threads."""
    from paper_2206_01580_amd import sorf
    n = 2 ** 18 + 5
    m, alpha = model(4096, 1, 3)
    b = atoms(n, 4)
    idx = torch.tensor([0, 2 ** 17 - 1, 2 ** 17, 2 ** 18 - 1, 2 ** 18, n - 1], device="cuda")
    E = sorf.predict(m, b, alpha)
    E1 = sorf.predict(m, some(b, idx), alpha)
    assert torch.equal(E[idx], E1)
