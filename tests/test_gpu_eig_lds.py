"""The one-workgroup Jacobi at its edges: odd and even sizes up to the
largest, scaled far from 1, both sizes of its rotation log, and the entropies'
block launch on blocks of every size."""

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


@pytest.mark.parametrize("n", [2, 5, 32, 63, 95, 96, 97, 127, 128])
@pytest.mark.parametrize("scale", [1.0, 1e100, 1e-100])
def test_lds_jacobi_edges(ctx, n, scale):
    import torch
    A = np.random.default_rng(n).standard_normal((n, n))
    A = scale * (A + A.T)
    w, V = (x.cpu().numpy() for x in ctx.sym_eig(torch.from_numpy(A).cuda()))
    norm = np.abs(A).sum(axis=1).max()
    # each of ~10 sweeps of n rounds rotates with errors of a few eps: n eps
    # times a constant; 1e-12 is 35 n eps at n = 128
    assert np.abs(w - np.linalg.eigvalsh(A)).max() <= 1e-12 * norm
    assert np.abs(A @ V - V * w).max() <= 1e-12 * norm
    assert np.abs(V.T @ V - np.eye(n)).max() <= 1e-12


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 64, 65, 66, 128])
@pytest.mark.parametrize("kind", ["full", "diagonal", "rank one", "pairs"])
def test_lds_jacobi_log(ctx, n, kind):
    """Both sizes of the rotation log at their edges, rounds of identities, and
    equal eigenvalues."""
    import torch
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n))
    A = A + A.T
    if kind == "diagonal":
        A = np.diag(np.diag(A))
    elif kind == "rank one":
        A = np.ones((n, n))
    elif kind == "pairs":
        A = np.kron(np.eye((n + 1) // 2), np.array([[1.0, 2.0], [2.0, 1.0]]))[:n, :n]
    w, V = (x.cpu().numpy() for x in ctx.sym_eig(torch.from_numpy(A.copy()).cuda()))
    norm = max(np.abs(A).sum(axis=1).max(), 1e-300)
    # as above
    assert np.all(np.diff(w) >= 0)
    assert np.abs(w - np.linalg.eigvalsh(A)).max() <= 1e-12 * norm
    assert np.abs(A @ V - V * w).max() <= 1e-12 * norm
    assert np.abs(V.T @ V - np.eye(n)).max() <= 1e-12


@pytest.mark.parametrize("L,nvec,cuts", [(2, 1, [0, 1]), (4, 3, [0, 3]), (6, 2, [5]),
                                         (10, 130, [0, 1, 2, 3, 4]), (18, 2, [0, 8])])
def test_entropies_of_random_vectors(ctx, pf, L, nvec, cuts):
    """Against singular values; 650 pairs are more than one chunk of 512."""
    import torch
    V = np.random.default_rng(L).standard_normal((pf.dim(L), nvec))
    V /= np.linalg.norm(V, axis=0)
    S = ctx.entanglement(L, torch.from_numpy(V).cuda(), cuts)
    h = L // 2
    s = np.array([x for x in range(1 << L) if bin(x).count("1") == h])
    for c, x in enumerate(cuts):
        t = ((s >> x) | (s << (L - x))) & ((1 << L) - 1)
        psi = np.zeros((nvec, 1 << h, 1 << h))
        psi[:, t >> h, t & ((1 << h) - 1)] = V.T
        lam = np.linalg.svd(psi, compute_uv=False) ** 2
        ref = -np.sum(np.where(lam > 1e-300, lam * np.log(np.maximum(lam, 1e-300)), 0.0), axis=1)
        # lambda errors of ~100 eps, times -ln lambda <= 40, over <= 512 values
        assert np.abs(S[:, c] - ref).max() <= 1e-10
