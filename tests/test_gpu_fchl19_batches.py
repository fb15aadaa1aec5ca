"""GPU: atoms of molecules above 64 atoms take a workgroup of 16 waves each while the call
has at most 256 atoms and of eight otherwise. A molecule's rows and gradients are bitwise
the same in both, wherever it stands in the batch.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2206_01580_amd import workloads as W
from test_gpu_fchl19 import PRM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,E,prm,stretch", [
    (65, 5, PRM, 1.0), (90, 1, PRM, 1.0), (70, 16, PRM, 1.0), (66, 5, PRM, 6.0),
    (256, 3, PRM, 1.0), (68, 3, dict(PRM, n3=2), 1.0), (67, 2, dict(PRM, n3=70), 1.0),
    (65, 2, dict(PRM, n3=257), 1.0), (65, 1, dict(PRM, n3=512), 1.0), (65, 1, dict(PRM, n3=513), 1.0),
    (80, 4, dict(PRM, n3=22), 0.8)], ids=str)
def test_same_bits(n, E, prm, stretch):
    from paper_2206_01580_amd import sorf
    rng = np.random.default_rng(n + E)
    R = (W.host_geometries([n], seed=n) * stretch).astype(np.float32)
    el = rng.integers(0, E, size=n).astype(np.int32)
    other = (W.host_geometries([200, 3, 100], seed=1)).astype(np.float32)
    other_el = rng.integers(0, E, size=303).astype(np.int32)
    p = sorf.fchl19_params(**prm)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()   # noqa: E731
    alone = dev(R), dev(el), dev(np.array([0, n], np.int64))
    batch = (dev(np.concatenate([other[:203], R, other[203:]])),
             dev(np.concatenate([other_el[:203], el, other_el[203:]])),
             dev(np.cumsum([0, 200, 3, n, 100]).astype(np.int64)))
    rho1 = sorf.fchl19(*alone, E, p)
    rho2 = sorf.fchl19(*batch, E, p)
    assert torch.isfinite(rho2).all()
    assert torch.equal(rho1, rho2[203:203 + n])
    g = torch.from_numpy(rng.standard_normal(tuple(rho2.shape)).astype(np.float32)).cuda()
    d1 = sorf.fchl19_backward(*alone, E, g[203:203 + n].contiguous(), p)
    d2 = sorf.fchl19_backward(*batch, E, g, p)
    assert torch.isfinite(d2).all()
    assert torch.equal(d1, d2[203:203 + n])
