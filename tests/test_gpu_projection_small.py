"""The projection of few atoms (one bucketing launch, tiles of 32 columns and
stages of 64 k) gives every row the bits that it has in a large batch, and
agrees with the plain product, at the edges of its stages and tiles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_rep,d,E", [(720, 128, 5), (128, 720, 5), (64, 32, 1), (65, 33, 3),
                                       (15, 2, 2), (68, 36, 7)])
def test_few_rows_have_the_bits_of_a_large_batch(d_rep, d, E):
    from paper_2206_01580_amd import sorf
    g = torch.Generator().manual_seed(d_rep + d)
    n = 40000
    rho = torch.randn(n, d_rep, generator=g).cuda()
    U = torch.randn(E, d_rep, d, generator=g).cuda()
    el = torch.randint(0, E, (n,), generator=g, dtype=torch.int32).cuda()
    many = sorf.project(rho, el, U)
    ref = torch.empty(n, d, dtype=torch.float64)
    scale = torch.empty(n, d, dtype=torch.float64)
    rho64, U64, el_h = rho.double().cpu(), U.double().cpu(), el.cpu()
    for e in range(E):
        rows = (el_h == e).nonzero().flatten()[:400]
        ref[rows] = rho64[rows] @ U64[e]
        scale[rows] = rho64[rows].abs() @ U64[e].abs()
    for k in (1, 2, 33, 129, 1000):
        few = sorf.project(rho[:k].contiguous(), el[:k].contiguous(), U)
        torch.cuda.synchronize()
        assert torch.equal(few, many[:k]), k
    k = 129
    # an FP32 sum of d_rep products: at most d_rep roundings of 2^-24
    err = (many[:k].double().cpu() - ref[:k]).abs()
    assert torch.all(err <= d_rep * 2.0 ** -24 * scale[:k])
