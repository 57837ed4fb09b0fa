"""What the autotuner's search compares: shapes that take the rank tables by
the forward form, whose steps they shape; the Clenshaw filter, which takes none
of them, does not choose among them.  A context that counts and answers with
set times stands in for the library (no GPU)."""

import random

import pytest

from paper_2005_09534_amd import autotune, workloads
from paper_2005_09534_amd import polfed as pf

CURRENT = (256, 1, 8, 1, 0, 0, 1)


class _Ctx:
    """seconds(shape, form) of a filter; tables under Clenshaw: one time and
    noise of 20 %, whatever the shape."""

    def __init__(self, forward, clenshaw, form=pf.FORM_CLENSHAW, current=CURRENT):
        self.shape, self.filter_form = current, form
        self.forward, self.clenshaw = forward, clenshaw
        self.rng = random.Random(5)
        self.calls = []

    def get_step_shape(self, L, nvec, precision):
        return self.shape

    def set_step_shape(self, L, nvec, precision, *sh):
        self.shape = tuple(sh)

    def set_filter_form(self, form):
        self.filter_form = form

    def apply_filter(self, m, E0, E1, sigma, K, X, out=None):
        self.calls.append((self.shape, self.filter_form))

    def filter_stats(self, reset=True):
        if self.filter_form == pf.FORM_FORWARD:
            t = self.forward(self.shape)
        else:
            t = self.clenshaw(self.shape)
            if self.shape[5] == 0:
                t *= self.rng.uniform(0.8, 1.2)
        return dict(gpu_s=t, launches=1.0, bytes=1e9)


@pytest.fixture(autouse=True)
def _no_gpu(monkeypatch):
    monkeypatch.setattr(autotune, "_random_block", lambda n, width, precision: (None, None),
                        raising=False)


def _forward(best):
    return lambda sh: 1.0 + 0.1 * sum(a != b for a, b in zip(sh, best))


@pytest.mark.parametrize("best", [(512, 2, 2, 0, 1, 0, 1), (1024, 4, 1, 1, 1, 0, 1)])
def test_tables_are_chosen_by_the_form_that_takes_them(best):
    ctx = _Ctx(_forward(best), lambda sh: 0.5 if sh[5] == 0 else 2.0)
    cache = {}
    sh, gbs = autotune.tune_shape(ctx, workloads.chain(12, 2.0, 1), 8, 0, cache=cache)
    assert sh == best and gbs > 0 and ctx.shape == best
    assert ctx.filter_form == pf.FORM_CLENSHAW
    assert cache[autotune._key("shape", 12, 0.0, 0, 8)][:7] == list(best)
    # under Clenshaw one shape with the tables, the winner
    assert {s for s, f in ctx.calls if f == pf.FORM_CLENSHAW and s[5] == 0} == {best}


def test_the_shape_in_force_stays_where_all_are_equal():
    ctx = _Ctx(lambda sh: 1.0, lambda sh: 0.5 if sh[5] == 0 else 2.0)
    assert autotune.tune_shape(ctx, workloads.chain(12, 2.0, 1), 8, 0)[0] == CURRENT
    assert ctx.shape == CURRENT


def test_another_rank_mode_wins_by_its_clenshaw_filter():
    best = (512, 2, 2, 0, 1, 1, 4)
    ctx = _Ctx(_forward(CURRENT), lambda sh: 0.5 if sh[5] == 0 else _forward(best)(sh) * 0.3)
    assert autotune.tune_shape(ctx, workloads.chain(12, 2.0, 1), 8, 0)[0] == best
    # and the tables where they are in force and no more than the margin behind
    near = _Ctx(_forward(CURRENT), lambda sh: 0.5 if sh[5] == 0 else 0.99 * 0.5 * 0.8)
    assert autotune.tune_shape(near, workloads.chain(12, 2.0, 1), 8, 0, margin=0.6)[0] == CURRENT


def test_forward_form_in_force_compares_all_by_it():
    best = (512, 2, 2, 0, 1, 2, 1)
    ctx = _Ctx(_forward(best), lambda sh: 1 / 0, form=pf.FORM_FORWARD)
    assert autotune.tune_shape(ctx, workloads.chain(12, 2.0, 1), 8, 0)[0] == best
    assert ctx.filter_form == pf.FORM_FORWARD


def test_given_shapes_are_all_timed():
    given = [(256, 1, 8, 1, 0, 0, 2), (512, 1, 2, 1, 0, 0, 4), (256, 1, 4, 1, 0, 1, 2)]
    ctx = _Ctx(_forward(given[1]), lambda sh: 0.5 if sh[5] == 0 else 2.0)
    assert autotune.tune_shape(ctx, workloads.chain(12, 2.0, 1), 8, 0, shapes=given)[0] == given[1]
    assert set(given) <= {s for s, _ in ctx.calls}


def test_blocks_of_a_batch_are_timed_once_each(monkeypatch):
    """The batched filters take no launch shape: a width's sample batch runs to
    warm up and once timed, and no shape is set or kept."""
    import torch
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)

    class Batch:
        runs, blocks = [], []

        def get_batch_shape(self, L, nvec, precision):
            return CURRENT[:5] + (1,)

        def solve_batch(self, models, nev, block_size, precision, vectors):
            self.runs.append(block_size)
            return dict(status=[pf.OK] * len(models))

        def set_block_size(self, L, precision, nev, block_size):
            self.blocks.append(block_size)

        def set_batch_shape(self, *a):
            raise AssertionError("a batch shape was set")

    ctx, shapes, blocks = Batch(), {}, {}
    chains = [workloads.chain(12, 2.0, r) for r in range(3)]
    best = autotune.tune_block(ctx, chains, 20, 1, widths=(4, 8), cache=blocks, shape_cache=shapes)
    assert ctx.runs == [4, 4, 8, 8] and shapes == {}
    assert best[0] in (4, 8) and ctx.blocks == [best[0]]
    assert blocks[autotune._key("block", 12, 0.0, 1, 20)][0] == best[0]
