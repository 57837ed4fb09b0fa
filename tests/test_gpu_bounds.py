"""The spectral bounds: short chains in one launch, longer ones by segments,
and the product with H by segments where the block is one slice."""

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


def _both(ctx, L, s, prec, call):
    """call() by the tables and by the step kernel with incremental ranks."""
    saved = ctx.get_step_shape(L, s, prec)
    Y = call()
    try:
        ctx.set_step_shape(L, s, prec, *saved[:5], 1)
        Z = call()
    finally:
        ctx.set_step_shape(L, s, prec, *saved)
    return Y, Z


# one row in the last tile and less than one tile (n = 6, 20, 70), one, two and
# four rows a thread (n = 252, 924, 3432), segments from n = 12870 on, their sums
# through one more launch (L = 24)
# (J2 needs L >= 6)
@pytest.mark.parametrize("J2,L", [(0.0, 4)] + [
    (J2, L) for J2 in (0.0, 0.7) for L in (6, 8, 10, 12, 14, 16, 18, 20)] + [(0.7, 24)])
def test_bounds_equal_the_step_kernel_run(ctx, pf, L, J2):
    """A few steps, before rounding has grown: every bound within steps * n
    roundings of the spectrum's width of the other run's."""
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, J2, 0.9, workloads.fields(L, 2.0, L))
    for steps in (1, 2, 5):
        a, b = _both(ctx, L, 1, 0, lambda: np.array(ctx.bounds(m, steps)))
        width = max(1.0, abs(b[0]), abs(b[1]))
        # entries of T each to about sqrt(n) eps |H|, through up to 5 steps
        # that divide by beta (about |H| / 10 at the smallest here)
        # (one step has no residual bounds: nan from both)
        np.testing.assert_allclose(a, b, rtol=0, atol=1e5 * 2.3e-16 * width, equal_nan=True)
        assert np.all(np.isfinite(a)) or steps == 1


@pytest.mark.parametrize("L", [10, 12, 14, 16])
def test_bounds_hold_the_spectrum(ctx, pf, L):
    """200 steps: E0, E1 are the extremes to rounding (|H| n eps)."""
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, 0.4, 0.9, workloads.fields(L, 1.5, L))
    a, b = _both(ctx, L, 1, 0, lambda: np.array(ctx.bounds(m, 200)))
    n = pf.dim(L)
    assert abs(a[0] - b[0]) <= n * 2.3e-16 * abs(b[0])
    assert abs(a[1] - b[1]) <= n * 2.3e-16 * abs(b[0])


@pytest.mark.parametrize("L,J2,prec,s", [
    (L, J2, prec, s) for L in (14, 16, 20) for J2 in (0.0, 0.7)
    for prec, s in ((0, 1), (0, 2), (1, 1), (1, 2), (1, 4), (0, 4), (1, 8))
] + [(22, 0.7, 0, 64), (24, 0.0, 0, 1)])
def test_apply_h_equals_the_step_kernel(ctx, pf, L, J2, prec, s):
    import torch
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, J2, 0.9, workloads.fields(L, 2.0, L))
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    X = torch.randn((pf.dim(L), s), generator=g, device="cuda",
                    dtype=torch.float64 if prec == 0 else torch.float32)
    Y, Z = _both(ctx, L, s, prec, lambda: ctx.apply_h(m, X))
    assert torch.equal(Y, Z)
