"""A dim key that occurs twice, and that many fact rows have: the call reports it,
its other outputs are right, and so is the next call's."""
import numpy as np
import pytest
import torch

import datagen
import oracle
from paper_2608_13696_amd import rel
from tests.gpu_util import assert_groups_equal, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = rel.Context(0)
    yield c
    c.close()


def _tables(n, m, by, seed, span=None):
    T = datagen.make_tables(n, m, seed, day_lt=1800, group_by=by, grp_card=max(1, min(m, 5)))
    r = np.random.default_rng(seed)
    T.pk = r.permutation(m).astype(np.int32)
    if span is not None:
        a = r.integers(0, span, m)
        a[0], a[m - 1] = 0, span - 1
        if by == "dim_grp":
            T.grp = a.astype(np.int32)
        else:
            T.prio = a.astype(np.int8)
    T.fk = T.pk[r.integers(0, m, n)].astype(np.int32)
    return T


# In turn: one chunk of groups and the table in LDS (the two rows' values or'ed name a group past the last), a table
# in device memory, numbered attributes, several chunks; (prio, flag); GROUP BY fk with one chunk and several.
@pytest.mark.parametrize("by,m,span,attrs", [("dim_grp", 2000, 5, (2, 3)), ("dim_grp", 2000, 300, (254, 255)),
                                             ("dim_grp", 100_000, 300, (254, 255)), ("dim_grp", 4000, 60_000, (20_000, 45_000)),
                                             ("dim_grp", 30_000, 20_000, (8191, 16_383)), ("prio_flag", 900, 5, (2, 3)),
                                             ("prio_flag", 900, 28, (15, 16)), ("fk", 500, None, None), ("fk", 9000, None, None)])
def test_hot_repeated_key_in_a_batch(ctx, by, m, span, attrs):
    bad, good = _tables(20_000, m, by, 3 + m, span), _tables(15_000, 700, "dim_grp", 4 + m, 90)
    a, b = m // 3, m // 2
    if attrs:
        (bad.grp if by == "dim_grp" else bad.prio)[[a, b]] = attrs
    key = bad.pk[b]
    bad.fk[::2] = bad.pk[a]
    bad.fk[1::4] = bad.pk[m // 4]
    dev = [to_dev(T) for T in (bad, good)]
    dev[0][1]["pk"][b] = int(bad.pk[a])
    batch = rel.Batch(ctx, [(f, d, T.day_lt, T.group_by, 0) for (f, d), T in zip(dev, (bad, good))], way="whole")
    for repeated in (True, True, False):
        if not repeated:
            dev[0][1]["pk"][b] = int(key)
        batch.run()
        if repeated:
            with pytest.raises(rel.RelError) as e:
                batch.sync()
            assert e.value.status == rel.DUPLICATE_KEY
        else:
            batch.sync()
            assert_groups_equal(rel.sorted_groups(batch.outs[0].host()), oracle.run_tables(bad)[0], "without the repeated key")
        assert_groups_equal(rel.sorted_groups(batch.outs[1].host()), oracle.run_tables(good)[0], "beside a repeated key")
    batch.close()
    assert ctx.sync() == 0


def _one_partition(keys):
    """int32 keys whose hashes in the partitioned join are 0, 1, ..: all in one partition."""
    inv = pow(2654435769, -1, 2**32)
    return (np.arange(keys, dtype=np.uint64) * np.uint64(inv) & np.uint64(2**32 - 1)).astype(np.uint32).view(np.int32)


# A key in several chunks of a partition's dim keys gives each of them a partial sum of the same rows: more partial
# sums than fact rows, and (8M rows) than there are chunks of memory for.
@pytest.mark.parametrize("n,m,keys", [(1, 6000, 1), (100, 200_000, 1), (100, 40_000, 3), (3000, 300_000, 700), (5000, 8_000_000, 1000)])
def test_key_in_many_chunks_of_a_planned_join(n, m, keys):
    pk = _one_partition(keys)
    T = datagen.make_tables(n, m, 7 + m, day_lt=2556, group_by="dim_grp", grp_card=9)
    T.pk, T.fk = np.resize(pk, m), np.resize(pk, n)
    T.grp = (np.arange(m) % 5000).astype(np.int32)
    fact, dim = to_dev(T)
    good = _tables(9000, 2500, "dim_grp", 8, 2000)
    good.day_lt = T.day_lt
    plan = lambda: rel.Plan(6000, rel.PLACE["global"], rel.PLACE["partitioned"], 0, 0)  # noqa: E731
    c = rel.Context(0)  # (with no memory of an earlier, larger call)
    with pytest.raises(rel.RelError) as e:
        c.filter_join_agg(fact, dim, T.day_lt, "dim_grp", plan=plan())
    assert e.value.status == rel.DUPLICATE_KEY
    gf, gd = to_dev(good)
    out, _ = c.filter_join_agg(gf, gd, good.day_lt, "dim_grp", plan=plan())
    assert_groups_equal(rel.sorted_groups(out.host()), oracle.run_tables(good)[0], "the next call")
    c.close()
