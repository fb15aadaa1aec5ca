"""Atoms of molecules above 64 atoms (a workgroup of 16 waves per atom) at the
edges of that kernel's split: the smallest such molecule, one element, element
pairs that span many lane groups and several chunks of pairs, radial bins that
leave threads over, that exceed a wave, and more than there are threads. Held
to the oracle with the bound of the other representation tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2206_01580_amd import workloads as W
from test_gpu_fchl19 import PRM, check

pytestmark = pytest.mark.gpu

CASES = {
    "smallest": ([65, 3], 5, PRM, 1.0),
    "one-element-many-groups": ([90], 1, PRM, 1.0),      # one pair of elements, 2 chunks
    "sixteen-elements": ([70], 16, PRM, 1.0),            # 136 element pairs, parts within one
    "few-neighbours": ([66], 5, PRM, 6.0),               # fewer pairs than lane groups
    "bins-2": ([68], 3, dict(PRM, n3=2), 1.0),           # 512 groups of 2
    "bins-70": ([67], 2, dict(PRM, n3=70), 1.0),
    "bins-1100": ([65], 1, dict(PRM, n3=1100), 1.0),     # more bins than threads
    "beside-small-ones": ([29, 80, 1, 64, 65], 4, PRM, 1.0),
}


@pytest.mark.parametrize("case", list(CASES))
def test_large_molecules_match_oracle(case):
    sizes, E, prm, stretch = CASES[case]
    rng = np.random.default_rng(len(case))
    R = W.host_geometries(sizes, seed=sum(sizes) + E) * stretch
    el = rng.integers(0, E, size=sum(sizes)).astype(np.int32)
    ptr = np.r_[0, np.cumsum(sizes)].astype(np.int64)
    print(f"{case}: max row error / row scale {check(R, el, ptr, E, prm):.2e}")


@pytest.mark.parametrize("E", [5, 10])   # rows staged in LDS, and above what is staged
def test_small_molecule_gradients_independent_of_the_wave_count(E):
    """Up to 256 molecules take 16 waves each, more take four: the same bits."""
    from test_gpu_fchl19 import F, gpu_grad
    sizes = ([1, 2, 4, 5, 15, 16, 17, 32, 33, 63, 64] * 24)[:260]
    rng = np.random.default_rng(E)
    R = W.host_geometries(sizes, seed=7).astype(np.float32)
    el = rng.integers(0, E, size=sum(sizes)).astype(np.int32)
    ptr = np.r_[0, np.cumsum(sizes)].astype(np.int64)
    g = rng.standard_normal((sum(sizes), F.fchl19_size(E, PRM["n2"], PRM["n3"]))).astype(np.float32)
    many = gpu_grad(R, el, ptr, E, PRM, g)
    n = int(ptr[22])
    few = gpu_grad(R[:n], el[:n], ptr[:23], E, PRM, g[:n])
    assert np.isfinite(many).all()
    assert np.array_equal(many[:n], few)


@pytest.mark.parametrize("n", [1024, 1025, 1100])
def test_gather_beyond_one_pass_of_the_workgroup(n):
    """Molecules around 1024 atoms, one piece of 64 atoms a wave and two: sampled
    rows against a small molecule that holds the same neighbourhoods (a
    stretched chain: atom i sees atoms i - 3 .. i + 3). The chain's triples are
    nearly collinear, where a gradient in FP32 has no 1e-5 to hold; the
    gradient's gather is the same code, and the 1260-atom test holds it."""
    from test_gpu_fchl19 import F, gpu_rho
    rng = np.random.default_rng(n)
    step = PRM["rcut"] / 3.4
    R = np.zeros((n, 3))
    R[:, 0] = np.arange(n) * step
    R += rng.uniform(-0.1, 0.1, size=R.shape)
    R = R.astype(np.float32)
    el = rng.integers(0, 3, size=n).astype(np.int32)
    rho = gpu_rho(R, el, np.array([0, n]), 3, PRM)
    for i in (0, 5, 63, 64, 127, 128, n // 2, 1000, n - 1):
        a, b = max(0, i - 8), min(n, i + 9)
        ref, _ = F.fchl19(R[a:b].astype(np.float64), el[a:b], np.array([0, b - a]), 3, PRM)
        ref = ref.numpy()[i - a]
        assert np.abs(rho[i] - ref).max() <= 2e-5 * np.abs(ref).max(), i
