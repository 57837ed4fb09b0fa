"""Edges of the filter's paths: coefficients that are zero, and blocks that are
aligned no better than their elements."""

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


@pytest.mark.parametrize("L,s", [(12, 2), (16, 1), (16, 8), (18, 2)])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("K", [1, 3])
def test_zero_leading_coefficient_drops_values_that_are_not_finite(ctx, pf, L, s, prec, K):
    """sigma = 0, odd order: c_K = 0, and the recurrence starts from zero
    whatever X holds.  What is not finite in X spreads to the rows where the
    step kernel has it, not one bond further."""
    import torch
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, 0.0, 0.9, workloads.fields(L, 2.0, L))
    X = torch.from_numpy(workloads.random_block(pf.dim(L), s, 3)).cuda()
    X = X if prec == 0 else X.float()
    X[7, 0] = float("inf")
    X[100, s - 1] = float("nan")
    Y = ctx.apply_filter(m, -40.0, 40.0, 0.0, K, X)
    saved = ctx.get_step_shape(L, s, prec)
    try:
        ctx.set_step_shape(L, s, prec, *saved[:5], 1)
        Z = ctx.apply_filter(m, -40.0, 40.0, 0.0, K, X)
    finally:
        ctx.set_step_shape(L, s, prec, *saved)
    ok = torch.isfinite(Z)
    assert torch.equal(torch.isfinite(Y), ok) and int((~ok).sum()) > 0
    assert torch.equal(Y[ok], Z[ok])


def _shifted(A):
    """A's values in memory that starts one element past an aligned address."""
    import torch
    B = torch.empty(A.numel() + 1, dtype=A.dtype, device=A.device)[1:].view(A.shape)
    B.copy_(A)
    assert B.is_contiguous() and B.data_ptr() % 16 == A.element_size()
    return B


# the whole filter in one launch, rows of one slice used in place, blocks packed
# into slices
@pytest.mark.parametrize("L,prec,s", [(12, 0, 4), (12, 1, 1), (16, 0, 1), (16, 0, 2), (16, 0, 8),
                                      (16, 1, 2), (16, 1, 4), (16, 1, 16), (18, 0, 2)])
@pytest.mark.parametrize("J2", [0.0, 0.7])
def test_blocks_aligned_as_their_elements(ctx, pf, L, prec, s, J2):
    import torch
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, J2, 0.9, workloads.fields(L, 2.0, L))
    X = torch.from_numpy(workloads.random_block(pf.dim(L), s, 3)).cuda()
    X = X if prec == 0 else X.float()
    for K in (1, 5):
        Y = ctx.apply_filter(m, -40.0, 40.0, 0.031, K, X)
        Z = _shifted(torch.zeros_like(X))
        ctx.apply_filter(m, -40.0, 40.0, 0.031, K, _shifted(X), out=Z)
        assert torch.equal(Y, Z), K
