"""Gram products of rows that lie far apart: an operand's leading dimension so
large that four rows span more than 4 GB."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2005_09534_amd import polfed
    c = polfed.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def far():
    """Memory of 13 rows, 0.18 G values apart (18.7 GB); 3 x 8 x 0.18 G > 2^32."""
    import torch
    ld = 180_000_003
    M = torch.zeros(12 * ld + 64, dtype=torch.float64, device="cuda")
    yield M, ld
    del M
    torch.cuda.empty_cache()


# less than four rows, a whole load of eight and a remainder; one column (no
# pairs), a pair that straddles the end, several tiles
@pytest.mark.parametrize("n,p,q", [(4, 2, 1), (3, 1, 3), (13, 33, 17), (13, 64, 40), (8, 1, 20)])
@pytest.mark.parametrize("which", ["X", "Y"])
def test_gram_of_far_rows(ctx, far, n, p, q, which):
    import torch
    M, ld = far
    rng = np.random.default_rng(n + p + q)
    Xh, Yh = rng.standard_normal((n, p)), rng.standard_normal((n, q))
    X, Y = torch.from_numpy(Xh).cuda(), torch.from_numpy(Yh).cuda()
    A = (X if which == "X" else Y)
    F = M.as_strided((n, A.shape[1]), (ld, 1))
    F.copy_(A)
    G = ctx.gram(F, Y) if which == "X" else ctx.gram(X, F)
    S = torch.empty((p, q), dtype=torch.float64, device="cuda")
    ctx.gram_static(F if which == "X" else X, Y if which == "X" else F, S)
    torch.cuda.synchronize()
    F.zero_()
    # sums of n products: at most n eps of the sum of their sizes
    bound = 2.3e-16 * (n + 4) * (np.abs(Xh).T @ np.abs(Yh))
    assert (np.abs(G.cpu().numpy() - Xh.T @ Yh) <= bound).all()
    assert torch.equal(G, S)
