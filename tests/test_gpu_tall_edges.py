"""Gram and update products at the edges of their tiles: odd and single columns,
leading dimensions past the width, rows that fill no tile, and values that are
not finite staying in their own row or column of the result."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pf():
    from paper_2005_09534_amd import polfed
    return polfed


@pytest.fixture(scope="module")
def ctx(pf):
    c = pf.Context(0)
    yield c
    c.close()


def _block(n, p, pad, seed):
    """n x p block inside rows of p + pad, and its values."""
    import torch
    M = torch.from_numpy(np.random.default_rng(seed).standard_normal((n, p + pad))).cuda()
    return M[:, :p], M[:, :p].cpu().numpy()


SHAPES = [(n, p, q) for n in (1, 7, 65, 3432) for p, q in
          [(1, 1), (2, 1), (1, 17), (3, 64), (31, 16), (33, 17), (65, 33), (100, 31), (129, 63)]]


@pytest.mark.parametrize("n,p,q", SHAPES + [(70001, 129, 33), (70001, 16, 64), (70001, 20, 5)])
@pytest.mark.parametrize("pad", [0, 3])
def test_gram_and_update_edges(ctx, n, p, q, pad):
    X, Xh = _block(n, p, pad, 1)
    Y, Yh = _block(n, q, pad, 2)
    # sums of n (p) products: at most n eps (p eps) of the sum of their sizes
    G = ctx.gram(X, Y).cpu().numpy()
    assert (np.abs(G - Xh.T @ Yh) <= 2.3e-16 * (n + 4) * (np.abs(Xh).T @ np.abs(Yh))).all()
    import torch
    C = torch.from_numpy(np.random.default_rng(3).standard_normal((p, q))).cuda()
    for alpha, beta in ((1.0, 0.0), (-0.5, 2.0)):
        Z = Y.clone() if pad == 0 else torch.cat([Y, Y[:, :1]], 1)[:, :q]
        Zh = Z.cpu().numpy()
        U = ctx.update(X, C, Z, alpha=alpha, beta=beta).cpu().numpy()
        Ch = C.cpu().numpy()
        size = abs(alpha) * (np.abs(Xh) @ np.abs(Ch)) + abs(beta) * np.abs(Zh)
        assert (np.abs(U - (alpha * (Xh @ Ch) + beta * Zh)) <= 2.3e-16 * (p + 4) * size).all()


@pytest.mark.parametrize("n,p,q", [(65, 33, 17), (70001, 129, 33)])
def test_not_finite_stays_in_its_column(ctx, n, p, q):
    X, Xh = _block(n, p, 0, 1)
    Y, Yh = _block(n, q, 0, 2)
    X[n - 1, p - 1] = float("nan")
    Y[n - 1, q - 1] = float("inf")
    G = ctx.gram(X, Y).cpu().numpy()
    ref = Xh.T @ Yh
    bound = 2.3e-16 * (n + 4) * (np.abs(Xh).T @ np.abs(Yh))
    assert (np.abs(G - ref) <= bound)[:-1, :-1].all()
    assert np.isnan(G[-1]).all() and not np.isfinite(G[:, -1]).any()
    import torch
    C = torch.from_numpy(np.random.default_rng(3).standard_normal((p, q))).cuda()
    Z = torch.zeros((n, q), dtype=torch.float64, device="cuda")
    U = ctx.update(X, C, Z).cpu().numpy()
    assert np.isnan(U[-1]).all() and np.isfinite(U[:-1]).all()
