"""The filter of a short chain in one launch against the step kernel.

Both do the same operations in the same order, so the results are equal bit
for bit; a step shape with incremental ranks keeps the step kernel (a launch
a step).  The tile form (L = 16, FP32) runs only in batches of at least 128
columns: there a batch is compared with its members' own solves.
"""

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


# one row a thread in one wave and in 16, two rows, four; both bond sets
@pytest.mark.parametrize("L,J2", [(4, 0.0), (6, 0.7), (10, 0.0), (12, 0.0), (12, 0.7), (14, 0.0),
                                  (14, 0.7)])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("s", [1, 64])
def test_resident_equals_step_kernel(ctx, pf, L, J2, prec, s):
    import torch
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, J2, 0.9, workloads.fields(L, 2.0, L))
    X = torch.from_numpy(workloads.random_block(pf.dim(L), s, 3)).cuda()
    X = X if prec == 0 else X.float()
    saved = ctx.get_step_shape(L, s, prec)
    # (orders around the number of steps of one launch on the shortest block)
    orders = [0, 1, 2, 3, 40] + ([16383, 16384, 16385] if s == 1 and L == 12 else [])
    for K in orders:
        for sigma in (0.0, 0.031):  # odd coefficients zero, and none
            Y = ctx.apply_filter(m, -20.0, 20.0, sigma, K, X)
            try:
                ctx.set_step_shape(L, s, prec, *saved[:5], 1)
                Z = ctx.apply_filter(m, -20.0, 20.0, sigma, K, X)
            finally:
                ctx.set_step_shape(L, s, prec, *saved)
            assert torch.equal(Y, Z), (K, sigma)


def test_infinities_stay_where_the_step_kernel_has_them(ctx, pf):
    import torch
    from paper_2005_09534_amd import workloads
    L, s = 10, 2
    m = pf.make_model(L, 1.0, 0.0, 0.9, workloads.fields(L, 2.0, L))
    X = torch.from_numpy(workloads.random_block(pf.dim(L), s, 3)).cuda()
    X[7, 0] = float("inf")
    X[100, 1] = float("nan")
    saved = ctx.get_step_shape(L, s, 0)
    Y = ctx.apply_filter(m, -20.0, 20.0, 0.031, 2, X)
    try:
        ctx.set_step_shape(L, s, 0, *saved[:5], 1)
        Z = ctx.apply_filter(m, -20.0, 20.0, 0.031, 2, X)
    finally:
        ctx.set_step_shape(L, s, 0, *saved)
    assert torch.equal(torch.isnan(Y), torch.isnan(Z))
    ok = ~torch.isnan(Z)
    assert torch.equal(Y[ok], Z[ok])


@pytest.mark.parametrize("J2", [0.0, 0.7])
def test_tile_form_batch_equals_single_solves(ctx, pf, J2):
    from paper_2005_09534_amd import workloads
    L, R, nev = 16, 16, 6
    models = [pf.make_model(L, 1.0, J2, 1.0, workloads.fields(L, 3.0, 50 + r)) for r in range(R)]
    kw = dict(precision=1, block_size=8, target=0.2)  # 16 x 8 columns
    b = ctx.solve_batch(models, nev, **kw)
    assert b["status"] == [0] * R
    for r in (0, 7, 15):
        one = ctx.solve(models[r], nev, vectors=False, **kw)
        # both are within their residual bar 1e-8 ||H||, and an eigenvalue's
        # error is second order in it
        assert np.abs(one["E"] - b["E"][r]).max() <= 1e-10 * one["info"]["normH"]
        assert b["resid"][r].max() <= 1e-8 * one["info"]["normH"]
