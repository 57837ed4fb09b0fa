"""Products with H in column slices over the XCDs (blocks beyond the L2 caches)
against unsliced ones: an entry that asks for one slice, whatever the library
would choose, and the step kernel with incremental ranks.  Equal bit for bit."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pf():
    from paper_2005_09534_amd import polfed
    return polfed


# 512- and 256-byte rows in four, two and one slices, in either precision, and
# rows of 128 bytes (never sliced); blocks of 25 MB (never sliced) to 1.4 GB;
# entries that ask for one, two and more slices than there are
@pytest.mark.parametrize("L,J2,prec,s", [
    (18, 0.7, 0, 64), (20, 0.7, 0, 64), (20, 0.0, 0, 64), (20, 0.7, 0, 32), (20, 0.7, 1, 64),
    (20, 0.7, 0, 16), (22, 0.7, 0, 64), (22, 0.0, 0, 64), (22, 0.7, 1, 64), (22, 0.0, 1, 64),
    (22, 0.7, 0, 32), (24, 0.7, 0, 32), (24, 0.0, 0, 64)])
def test_sliced_products_equal_unsliced(pf, L, J2, prec, s):
    import torch
    from paper_2005_09534_amd import workloads
    m = pf.make_model(L, 1.0, J2, 0.9, workloads.fields(L, 2.0, L))
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    X = torch.empty((pf.dim(L), s), device="cuda",
                    dtype=torch.float64 if prec == 0 else torch.float32).normal_(generator=g)
    ctx = pf.Context(0)
    try:
        Y = ctx.apply_h(m, X)
        shape = ctx.get_step_shape(L, s, prec)
        for rank, slices in ((0, 1), (1, 1), (0, 2), (0, 8), (1, 4), (0, 1)):
            ctx.set_step_shape(L, s, prec, *shape[:5], rank, slices)
            assert torch.equal(ctx.apply_h(m, X), Y), (rank, slices)
    finally:
        ctx.close()
