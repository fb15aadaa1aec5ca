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
