"""The step by segments against the step kernel with incremental ranks.

Both add a row's bonds in the same order, so the results are equal bit for
bit.  Lengths cover every number of high sites a kernel is built for, widths
every piece size and number of slices.
"""

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


def _both(ctx, L, s, prec, call):
    """call() by segments and by the step kernel."""
    saved = ctx.get_step_shape(L, s, prec)
    Y = call()
    try:
        ctx.set_step_shape(L, s, prec, *saved[:5], 1)
        Z = call()
    finally:
        ctx.set_step_shape(L, s, prec, *saved)
    return Y, Z


@pytest.mark.parametrize("L,J2,prec,s", [
    (L, J2, prec, s) for L in (16, 18, 20) for J2 in (0.0, 0.7) for prec in (0, 1)
    for s in (1, 2, 4, 8, 64) if not (prec == 0 and s == 4)
] + [(22, 0.0, 1, 32), (22, 0.7, 0, 16), (24, 0.0, 0, 8), (24, 0.7, 1, 4), (26, 0.0, 1, 16),
     (26, 0.7, 0, 2), (28, 0.0, 0, 1), (28, 0.7, 1, 2)])
def test_segments_equal_step_kernel(ctx, pf, L, J2, prec, s):
    import torch
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, J2, 0.9, workloads.fields(L, 2.0, L))
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    X = torch.randn((pf.dim(L), s), generator=g, device="cuda",
                    dtype=torch.float64 if prec == 0 else torch.float32)
    for K in ((1, 2, 9) if L <= 20 else (2,)):
        for sigma in (0.0, 0.031):  # odd coefficients zero, and none
            Y, Z = _both(ctx, L, s, prec,
                         lambda: ctx.apply_filter(m, -40.0, 40.0, sigma, K, X))
            assert torch.equal(Y, Z), (K, sigma)


def test_infinities_stay_where_the_step_kernel_has_them(ctx, pf):
    import torch
    from paper_2005_09534_amd import workloads
    L, s = 16, 4
    m = pf.make_model(L, 1.0, 0.7, 0.9, workloads.fields(L, 2.0, L))
    X = torch.from_numpy(workloads.random_block(pf.dim(L), s, 3)).cuda()
    X[7, 0] = float("inf")
    X[12000, 1] = float("nan")
    Y, Z = _both(ctx, L, s, 0, lambda: ctx.apply_filter(m, -40.0, 40.0, 0.031, 2, X))
    assert torch.equal(torch.isnan(Y), torch.isnan(Z))
    ok = ~torch.isnan(Z)
    assert torch.equal(Y[ok], Z[ok])


@pytest.mark.parametrize("L,J2,nvec,nmom", [(16, 0.0, 1, 31), (16, 0.7, 3, 32), (18, 0.0, 70, 9),
                                            (22, 0.7, 40, 80)])  # (more steps than one final sum)
def test_moments_by_segments(ctx, pf, L, J2, nvec, nmom):
    """The sums a segment step leaves against those of separate launches: the
    same terms in another order, n nvec of them of at most 1 (in units of
    mu_0), so within a few eps sqrt(n nvec) of each other; 1e-12 is 10 times
    that for the largest."""
    import numpy as np
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, J2, 0.9, workloads.fields(L, 2.0, L))
    S = 1
    while S < nvec and S < 64:
        S *= 2
    saved = ctx.get_step_shape(L, S, 0)
    mu = ctx.dos_moments(m, -40.0, 40.0, nmom, nvec=nvec, seed=5)
    try:
        ctx.set_step_shape(L, S, 0, *saved[:5], 1)
        ref = ctx.dos_moments(m, -40.0, 40.0, nmom, nvec=nvec, seed=5)
    finally:
        ctx.set_step_shape(L, S, 0, *saved)
    assert mu[0] == 1.0
    assert np.abs(mu - ref).max() <= 1e-12


# an eighth of every slice to an XCD, and whole slices (64 and more of them);
# one slice a block (rows of X and Y used in place) and several
@pytest.mark.parametrize("lengths,R,prec,s,J2", [((16, 18), 4, 1, 4, 0.0), ((16,), 17, 0, 8, 0.7),
                                                 ((16, 14, 18), 5, 0, 2, 0.0)])
def test_batch_by_segments_equals_single_solves(ctx, pf, lengths, R, prec, s, J2):
    import numpy as np
    from paper_2005_09534_amd import workloads
    Ls = [lengths[r % len(lengths)] for r in range(R)]
    models = [pf.make_model(L, 1.0, J2, 1.0, workloads.fields(L, 3.0, 70 + r))
              for r, L in enumerate(Ls)]
    kw = dict(precision=prec, block_size=s, target=0.1, window_factor=4.0)
    b = ctx.solve_batch(models, 4, **kw)
    for r in (0, R - 1):
        one = ctx.solve(models[r], 4, vectors=False, **kw)
        assert b["status"][r] == one["status"] == 0
        # both within 1e-8 ||H|| in residual; eigenvalue errors are second order
        assert np.abs(one["E"] - b["E"][r]).max() <= 1e-10 * one["info"]["normH"]
