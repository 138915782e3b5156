"""GPU parity of the planned partitioned form, whose partial sums by group are
partitioned and summed in LDS: group counts around the bins' and tables' sizes,
chunks that fill up, hot keys and hot groups, bins cut into pieces, too small
plans and outputs, and other calls between."""
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


def _tables(n, m, seed, grp, hot=0.0, negative=False):
    """`grp`: group count, or an array of the dim rows' groups; `hot`: the share of rows with one key."""
    T = datagen.make_tables(n, m, seed, day_lt=1300, group_by="dim_grp", grp_card=max(1, min(m, 9)))
    r = np.random.default_rng(seed)
    T.grp = (grp if isinstance(grp, np.ndarray) else r.integers(0, grp, m)).astype(np.int32)
    if negative:
        T.grp = (T.grp - np.int32(2**30)) * 2
    if hot:
        T.fk[r.random(n) < hot] = T.pk[m // 2]
    return T


def _check(ctx, T, capacity, groups="global", **kw):
    fact, dim = to_dev(T)
    plan = rel.Plan(capacity, rel.PLACE[groups], rel.PLACE["partitioned"], 0, 0)
    out, st = ctx.filter_join_agg(fact, dim, T.day_lt, T.group_by, plan=plan, **kw)
    ora, ost = oracle.run_tables(T)
    assert_groups_equal(gpu_groups(out), ora, f"n={T.n} m={T.m} capacity={capacity}")
    assert [st[x] for x in ("rows_passed", "join_matches", "groups")] == [ost[x] for x in ("rows_passed", "join_matches", "groups")]


@pytest.mark.parametrize("n,m,groups", [(1, 1, 1), (300, 70, 70), (5000, 2047, 1), (40_000, 9000, 513), (200_000, 50_000, 50_000),
                                        (1_000_000, 250_000, 2), (1_000_003, 260_001, 70_000), (600_000, 500_000, 500_000)])
def test_sizes(ctx, n, m, groups):
    for hot in (0.0, 0.6):
        T = _tables(n, m, n + m, groups, hot, negative=hot > 0)
        for capacity in (max(groups, 600), 4 * groups + 2000):
            _check(ctx, T, capacity)


def test_plan_that_misjudges_the_groups(ctx):
    """Far too many groups expected, and too few: a bin's LDS table overflows into the device table, and that one
    into the error (or the plain run) that an undersized plan gives."""
    T = _tables(500_000, 120_000, 5, 60_000)
    _check(ctx, T, 10_000_000)
    _check(ctx, T, 33_000)  # (65536 slots in the device table)
    fact, dim = to_dev(T)
    plan = rel.Plan(1000, rel.PLACE["global"], rel.PLACE["partitioned"], 0, 0)
    with pytest.raises(rel.RelError) as e:
        ctx.filter_join_agg(fact, dim, T.day_lt, T.group_by, plan=plan)
    assert e.value.status == rel.OVERFLOW
    plan = rel.Plan(1000, rel.PLACE["global"], rel.PLACE["partitioned"], 1, 0)
    out, st = ctx.filter_join_agg(fact, dim, T.day_lt, T.group_by, plan=plan)
    assert st["fell_back"] == 1
    assert_groups_equal(gpu_groups(out), oracle.run_tables(T)[0], "fallback")
    _check(ctx, T, 60_000)


def test_hot_group_and_keys_without_rows(ctx):
    m = 300_000
    grp = np.arange(m) % 3000
    grp[::2] = 7  # half of the dim keys in one group: its bin is cut into pieces
    T = _tables(900_000, m, 6, grp)
    T.fk[::3] = -5
    _check(ctx, T, 3000)
    T.day_lt = -1  # nothing passes
    _check(ctx, T, 3000)


def test_other_calls_between_and_small_output(ctx):
    """The device table is left empty for the plain path, which shares it, and the other way round."""
    T = _tables(400_000, 100_000, 8, 40_000)
    P = _tables(30_000, 7000, 9, 5000)
    fact, dim = to_dev(P)
    for capacity in (40_000, 33_000, 100_000):
        _check(ctx, T, capacity)
        out, _ = ctx.filter_join_agg(fact, dim, P.day_lt, P.group_by)
        assert_groups_equal(gpu_groups(out), oracle.run_tables(P)[0], "plain between")
    fact, dim = to_dev(T)
    plan = rel.Plan(40_000, rel.PLACE["global"], rel.PLACE["partitioned"], 0, 0)
    with pytest.raises(rel.RelError) as e:
        ctx.filter_join_agg(fact, dim, T.day_lt, T.group_by, plan=plan, out_cap=1000)
    assert e.value.status == rel.CAPACITY
    _check(ctx, T, 40_000)


@pytest.mark.parametrize("m,groups", [(40_000, 30), (100_000, 30_000), (20_000, 9000)])  # 64 partitions and more; fewer
@pytest.mark.parametrize("price,qty", [((90_000, 10_500_000), (1, 51)), ((-5, 5), (-3, 1)), ((2**32 - 3, 2**32 + 3), (0, 1)),
                                       ((-(2**40), 2**40), (-(2**31), 2**31)), ((-(2**63), 2**63), (7, 8)),
                                       ((2**62, 2**62 + 1000), (-(2**31), -(2**31) + 5))])
def test_value_ranges(ctx, m, groups, price, qty):
    """Rows of one word where the values' ranges allow, of 16 bytes where they don't; few groups and many."""
    T = _tables(150_000, m, 12, groups, negative=True)
    r = np.random.default_rng(m)
    T.pk = (T.pk.astype(np.int64) * 7 - 3000).astype(np.int32)  # keys of both signs
    T.fk = T.pk[r.integers(0, m, T.n)]
    T.fk[::10] = r.integers(-(2**31), 2**31, len(T.fk[::10])).astype(np.int32)
    T.price_cents = r.integers(price[0], price[1] - 1, T.n, dtype=np.int64, endpoint=True)
    T.qty = r.integers(qty[0], qty[1], T.n, dtype=np.int64).astype(np.int32)
    for placement in ("global", "lds"):
        _check(ctx, T, groups, placement)


def test_repeated_key_is_reported(ctx):
    T = _tables(50_000, 20_000, 10, 9000)
    T.pk[15_000] = T.pk[3]
    fact, dim = to_dev(T)
    plan = rel.Plan(9000, rel.PLACE["global"], rel.PLACE["partitioned"], 0, 0)
    with pytest.raises(rel.RelError) as e:
        ctx.filter_join_agg(fact, dim, T.day_lt, T.group_by, plan=plan)
    assert e.value.status == rel.DUPLICATE_KEY
    _check(ctx, _tables(50_000, 20_000, 11, 9000), 9000)
