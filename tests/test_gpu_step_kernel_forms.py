"""What still runs on the step kernel by rows: the Clenshaw filter with
incremental ranks or the stored pattern (in graphs, in column slices), the
forward form, and products of wide blocks with any launch shape.  Every one is
compared bit for bit with the launches that the library chooses by itself,
which add the same terms in the same order."""

import pytest

torch = pytest.importorskip("torch")

from paper_2005_09534_amd import autotune, workloads  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pf():
    from paper_2005_09534_amd import polfed
    return polfed


@pytest.fixture
def ctx(pf):
    c = pf.Context(0)
    yield c
    c.close()


def _chain(pf, L, J2, s, prec, seed=3):
    m = pf.make_model(L, 1.0, J2, 0.9, workloads.fields(L, 2.0, L))
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    X = torch.empty((pf.dim(L), s), device="cuda",
                    dtype=torch.float32 if prec else torch.float64).normal_(generator=g)
    return m, X


@pytest.mark.parametrize("rank,slices", [(1, 1), (1, 4), (2, 1), (2, 2)])
@pytest.mark.parametrize("L,J2,prec", [(14, 0.0, 0), (14, 0.7, 1), (16, 0.7, 0)])
def test_clenshaw_graphs_of_the_step_kernel(ctx, pf, L, J2, prec, rank, slices):
    """Captured and replayed several times, with eager work and waits between
    the replays, other orders and other buffers in turn."""
    s = 8
    m, X = _chain(pf, L, J2, s, prec)
    _, X2 = _chain(pf, L, J2, s, prec, seed=4)
    ref = {(K, i): ctx.apply_filter(m, -40.0, 40.0, 0.1, K, x) for K in (16, 61)
           for i, x in enumerate((X, X2))}
    shape = ctx.get_step_shape(L, s, prec)
    ctx.set_step_shape(L, s, prec, *shape[:5], rank, slices)
    Y = [torch.empty_like(X), torch.empty_like(X)]
    for graphs in (True, False):
        ctx.set_graphs(graphs)
        for K, i, rep in [(61, 0, 0), (61, 0, 1), (61, 0, 2), (16, 0, 0), (16, 1, 1), (61, 1, 0),
                          (61, 1, 1), (61, 0, 3)]:
            Y[i].fill_(float("nan"))
            ctx.apply_filter(m, -40.0, 40.0, 0.1, K, (X, X2)[i], out=Y[i])
            _ = (X * 2).sum().item()
            assert torch.equal(Y[i], ref[K, i]), (graphs, K, i, rep)


@pytest.mark.parametrize("prec,s,J2", [(0, 8, 0.0), (0, 4, 0.7), (1, 32, 0.7), (1, 8, 0.0)])
def test_shapes_of_products_and_the_forward_form(ctx, pf, prec, s, J2):
    """Every launch shape with the rank tables, where it is read: H X of a block
    of more than one slice, and the forward form."""
    L = 14
    m, X = _chain(pf, L, J2, s, prec)
    H = ctx.apply_h(m, X)
    ctx.set_filter_form(pf.FORM_FORWARD)
    F = ctx.apply_filter(m, -40.0, 40.0, 0.1, 12, X)
    shapes = [sh for sh in autotune.SHAPES if sh[5] == 0 and sh[6] in (1, 4)]
    assert {sh[0] for sh in shapes} == {256, 512, 1024} and {sh[3] for sh in shapes} == {0, 1}
    for sh in shapes:
        ctx.set_step_shape(L, s, prec, *sh)
        assert torch.equal(ctx.apply_h(m, X), H), sh
        assert torch.equal(ctx.apply_filter(m, -40.0, 40.0, 0.1, 12, X), F), sh


@pytest.mark.parametrize("prec,slices", [(0, 4), (1, 2)])
def test_sliced_clenshaw_of_the_longest_workload(ctx, pf, prec, slices):
    """L = 26, 64 columns, slice-major: 16 FP64 columns a slice, 32 in FP32."""
    L, s = 26, 64
    m, X = _chain(pf, L, 0.0, s, prec)
    Y = ctx.apply_filter(m, -40.0, 40.0, 0.013, 3, X)
    ctx.set_step_shape(L, s, prec, 256 if prec == 0 else 512, 2, 2, 1, 0, 1, slices)
    assert torch.equal(ctx.apply_filter(m, -40.0, 40.0, 0.013, 3, X), Y)
    del X, Y
    torch.cuda.empty_cache()
