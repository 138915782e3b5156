"""GPU parity of the plain fused path where its kernels hand over to one another:
the ways its groups leave (staged and merged, through the device table by the
merge kernel or by the finalize kernel), the join index's kinds by key count, and
the memory that each call leaves empty for the next, after calls of other sizes,
repeated keys and too small outputs."""
import numpy as np
import pytest
import torch

import datagen
import oracle
from paper_2608_13696_amd import rel
from tests.gpu_util import assert_groups_equal, gpu_groups, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = rel.Context(0)
    yield c
    c.close()


def _plan(capacity=0, placement="auto"):
    return rel.Plan(capacity, rel.PLACE[placement], rel.PLACE["global"], 0, 0)


def _check(ctx, T, plan=None, stats=True):
    fact, dim = to_dev(T)
    want, ws = oracle.run_tables(T)
    out, st = ctx.filter_join_agg(fact, dim, T.day_lt, T.group_by, plan=plan or _plan(), stats=stats)
    assert ctx.sync() == 0
    assert_groups_equal(gpu_groups(out), want, str(T.meta))
    if stats:
        assert (st["rows_passed"], st["join_matches"], st["groups"]) == (ws["rows_passed"], ws["join_matches"], ws["groups"])


def _tables(n, m, by, prios, flags, seed, stride=1, grp=None):
    T = datagen.make_tables(n, m, seed, group_by=by, fk_domain=m + m // 7 + 1, grp_card=grp)
    rng = np.random.default_rng(seed)
    T.prio = rng.integers(-prios // 2, prios - prios // 2, size=m).astype(np.int8)
    T.flag = rng.integers(-flags // 2, flags - flags // 2, size=n).astype(np.int8)
    T.pk, T.fk = T.pk * stride, T.fk * stride
    return T


# 262144 rows: the merge kernel ends the call; more: 1024-thread workgroups and a finalize kernel
@pytest.mark.parametrize("n", [1, 1023, 60_001, 262_144, 262_145, 700_003])
@pytest.mark.parametrize("prios,flags", [(5, 3), (8, 5), (40, 12), (200, 10), (256, 256)])
def test_group_counts_and_stages(ctx, n, prios, flags):
    """15 groups to more than the LDS table, a stage or (60001 rows) the staged total holds."""
    _check(ctx, _tables(n, 15_000, "prio_flag", prios, flags, n), stats=n % 2 == 1)


@pytest.mark.parametrize("m", [1, 65_535, 65_536, 65_537, 150_001])
@pytest.mark.parametrize("stride", [1, 2, 30])
@pytest.mark.parametrize("by", ["prio_flag", "fk", "dim_grp"])
def test_index_kinds(ctx, m, stride, by):
    _check(ctx, _tables(120_003, m, by, 5, 3, m + stride, stride, grp=m // 3 + 1))


def test_memory_left_empty(ctx):
    """One context through calls of different sizes and kinds, among them failing ones."""
    rng = np.random.default_rng(9)
    for k in range(24):
        n, m = int(np.exp(rng.uniform(3, 13))), int(np.exp(rng.uniform(1, 12)))
        by = ["prio_flag", "fk", "dim_grp"][k % 3]
        T = _tables(n, m, by, int(rng.integers(2, 250)), int(rng.integers(2, 9)), 100 + k, [1, 1, 50][k % 5 % 3], grp=m)
        _check(ctx, T)
        fact, dim = to_dev(T)
        if k % 4 == 0 and m > 1:  # a repeated key
            dim["pk"][m - 1] = dim["pk"][0]
            with pytest.raises(rel.RelError) as e:
                ctx.filter_join_agg(fact, dim, T.day_lt, by, plan=_plan())
            assert e.value.status == rel.DUPLICATE_KEY
        elif k % 4 == 2:  # an output for one group
            out, _ = ctx.filter_join_agg(fact, dim, T.day_lt, by, plan=_plan(), stats=False, out_cap=1)
            bits = ctx.sync()
            want, _ = oracle.run_tables(T)
            assert int(out.n_groups) == want["key"].size and bits == (rel.DEV_OVERFLOW if want["key"].size > 1 else 0)


def test_planned_tables_that_are_too_small(ctx):
    T = _tables(200_003, 50_000, "dim_grp", 5, 3, 3, grp=40_000)
    fact, dim = to_dev(T)
    for placement in ("global", "lds"):
        plan = _plan(100, placement)
        with pytest.raises(rel.RelError) as e:
            ctx.filter_join_agg(fact, dim, T.day_lt, "dim_grp", plan=plan)
        assert e.value.status == rel.OVERFLOW
        plan.allow_fallback = 1
        _check(ctx, T, plan)
        _check(ctx, T)
