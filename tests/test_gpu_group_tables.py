"""GPU parity of plain LDS calls whose groups go to the device table: which the streaming workgroups put there, which only
the merge finds no room for, tables far larger than the groups, outputs that are too small, and the next call."""
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


def _tables(n, groups, clustered, seed):
    """`clustered`: a row's group grows with the row, so that a workgroup meets few of them."""
    m = max(groups, 16)
    T = datagen.make_tables(n, m, seed, day_lt=2400, group_by="dim_grp", grp_card=groups)
    r = np.random.default_rng(seed)
    T.pk = r.permutation(m).astype(np.int32)
    T.grp = (T.pk % groups).astype(np.int32)
    T.fk = (np.arange(n, dtype=np.int64) * m // n if clustered else r.integers(0, m, n)).astype(np.int32)
    return T


# 65536 rows: 256-thread workgroups; 262144: the merge kernel ends the call
@pytest.mark.parametrize("n", [900, 20_000, 65_536, 65_537, 262_144, 262_145])
@pytest.mark.parametrize("groups,capacity", [(30, 30), (600, 600), (3000, 3000), (3000, 500_000), (40_000, 600_000)])
def test_groups_in_the_device_table(ctx, n, groups, capacity):
    for clustered in (False, True):
        T = _tables(n, groups, clustered, n + groups)
        fact, dim = to_dev(T)
        want, ws = oracle.run_tables(T)
        plan = rel.Plan(capacity, rel.PLACE["lds"], rel.PLACE["global"], 0, 0)
        for stats in (True, False):
            out, st = ctx.filter_join_agg(fact, dim, T.day_lt, "dim_grp", plan=plan, stats=stats)
            assert ctx.sync() == 0
            assert_groups_equal(gpu_groups(out), want, f"n={n} groups={groups} capacity={capacity} clustered={clustered}")
            assert not stats or st["groups"] == ws["groups"] and st["join_matches"] == ws["join_matches"]


@pytest.mark.parametrize("n", [20_000, 200_000])
def test_output_for_fewer_groups(ctx, n):
    T = _tables(n, 5000, False, 3)
    fact, dim = to_dev(T)
    want = oracle.run_tables(T)[0]
    plan = rel.Plan(20_000, rel.PLACE["lds"], rel.PLACE["global"], 0, 0)
    out, _ = ctx.filter_join_agg(fact, dim, T.day_lt, "dim_grp", plan=plan, stats=False, out_cap=100)
    assert ctx.sync() == rel.DEV_OVERFLOW and int(out.n_groups) == want["key"].size
    out, _ = ctx.filter_join_agg(fact, dim, T.day_lt, "dim_grp", plan=plan, stats=False)
    assert ctx.sync() == 0
    assert_groups_equal(gpu_groups(out), want, "the next call")
