"""The tall update around the ends of its blocks of k, for every number of
column tiles and both workgroup sizes."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2005_09534_amd import polfed
    c = polfed.Context(0)
    yield c
    c.close()


# sums without staging (up to 8), one, two and three blocks of 16 and of 32, and
# the limits from which few rows take blocks of 32 (128) and 64 (256)
@pytest.mark.parametrize("p", [3, 4, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64, 65, 97, 127, 128, 161,
                               255, 256, 257, 320])
@pytest.mark.parametrize("q", [1, 15, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("n", [37, 65541])
def test_update_around_its_blocks(ctx, n, p, q):
    import torch
    rng = np.random.default_rng([n, p, q])
    X, C, Y = (rng.standard_normal(s) for s in ((n, p + 1), (p, q + 2), (n, q + 3)))
    Xt, Ct, Yt = (torch.from_numpy(a).cuda() for a in (X, C, Y))
    ctx.update(Xt[:, :p], Ct[:, :q], Yt[:, :q], alpha=-1.5, beta=0.5)
    got = Yt.cpu().numpy()
    # p products and two more terms: at most (p + 4) eps of the sum of their sizes
    ref = -1.5 * (X[:, :p] @ C[:, :q]) + 0.5 * Y[:, :q]
    size = 1.5 * (np.abs(X[:, :p]) @ np.abs(C[:, :q])) + 0.5 * np.abs(Y[:, :q])
    assert (np.abs(got[:, :q] - ref) <= 2.3e-16 * (p + 4) * size).all()
    assert np.array_equal(got[:, q:], Y[:, q:])
