"""The batched filters (shared launches of the batched solve) against the
filters of the same chains one by one: the same operations in the same order
on weights rounded the same way, so the results are equal bit for bit."""

import ctypes

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


def _batch(ctx, pf, models, E, sigma, K, X):
    """Y of the batched launches for lists of one entry a member."""
    import torch
    R = len(models)
    Y = [torch.full_like(x, float("nan")) for x in X]
    D, LL, VP = ctypes.c_double * R, ctypes.c_longlong * R, ctypes.c_void_p * R
    prec = 0 if X[0].dtype == torch.float64 else 1
    ctx._check(pf.LIB.polfed_test_filter_batch(
        ctx.h, ctypes.c_int(R), (pf.Model * R)(*models), D(*[-e for e in E]), D(*E), D(*sigma),
        LL(*K), ctypes.c_int(prec), ctypes.c_int(X[0].shape[1]), VP(*[x.data_ptr() for x in X]),
        VP(*[y.data_ptr() for y in Y])), "test_filter_batch")
    return Y


def _members(pf, lengths, J2, s, prec):
    import torch
    from paper_2005_09534_amd import workloads
    models, X, E = [], [], []
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    for r, L in enumerate(lengths):
        h = workloads.fields(L, 2.0, 40 + r)
        models.append(pf.make_model(L, 1.0, J2, 0.9, h))
        X.append(torch.randn((pf.dim(L), s), generator=g, device="cuda",
                             dtype=torch.float64 if prec == 0 else torch.float32))
        E.append((1.0 + J2) * L * 0.5 + 0.5 * float(np.abs(h).sum()))
    return models, X, E


def _compare(ctx, pf, lengths, orders, J2, s, prec):
    import torch
    models, X, E = _members(pf, lengths, J2, s, prec)
    # odd coefficients zero, and none
    sigma = [(0.0, 0.031, -0.2)[r % 3] for r in range(len(lengths))]
    Y = _batch(ctx, pf, models, E, sigma, orders, X)
    for r in range(len(lengths)):
        Z = ctx.apply_filter(models[r], -E[r], E[r], sigma[r], orders[r], X[r])
        assert torch.equal(Y[r], Z), (r, lengths[r], orders[r])


# lengths of the one-launch filter (12, 14) and of the segments (16 .. 20), each
# of several orders: none, one, odd and even, the longest not the first.  One
# slice (rows of X and Y used in place) and several; few slices in all (an eighth
# of each to an XCD) and 64 and more (whole slices)
@pytest.mark.parametrize("J2", [0.0, 0.7])
@pytest.mark.parametrize("prec,s", [(0, 1), (0, 2), (0, 4), (0, 32), (1, 1), (1, 2), (1, 4), (1, 8),
                                    (1, 64)])
def test_batch_equals_single_filters(ctx, pf, J2, prec, s):
    lengths = [16, 12, 18, 16, 14, 16, 20, 14, 18]
    orders = [5, 4, 12, 0, 7, 1, 3, 0, 2]
    _compare(ctx, pf, lengths, orders, J2, s, prec)


def test_batch_of_many_members(ctx, pf):
    lengths = [16, 18] * 10
    _compare(ctx, pf, lengths, [(7 * r) % 11 for r in range(20)], 0.0, 8, 0)


# FP32, L = 16, from 128 columns on: the tile form, orders around the number of
# steps of one launch (16384)
@pytest.mark.parametrize("J2", [0.0, 0.7])
def test_tile_form_equals_single_filters(ctx, pf, J2):
    orders = [0, 1, 2, 3, 40, 41, 16383, 16384, 16385, 16386, 9, 10, 11, 12, 13, 32769]
    _compare(ctx, pf, [16] * 16, orders, J2, 8, 1)
