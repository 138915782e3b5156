"""GPU parity of batches whose instances go either way, one workgroup each or by
tables in device memory: chosen from their sizes, all by the tables, all whole."""
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


@pytest.mark.parametrize("sizes", [[(1000, 600_000), (1000, 100), (250_000, 40)], [(3, 2)], [(30_000, 7500)] * 20 + [(200_000, 3000)],
                                   [(5000, 1250)] * 40, [(2048, 1024), (2049, 1025), (400_000, 200_000)]])
def test_both_ways(ctx, sizes):
    tables, insts = [], []
    for i, (n, m) in enumerate(sizes):
        by = ("dim_grp", "prio_flag", "fk")[i % 3]
        T = datagen.make_tables(n, m, 50 + i, day_lt=1400, group_by=by, fk_domain=m + m // 5 + 1, grp_card=max(1, m // 3))
        tables.append(T)
        insts.append((*to_dev(T), T.day_lt, by, 0))
    want = [oracle.run_tables(T) for T in tables]
    for way in ("auto", "shared", "whole"):
        b = rel.Batch(ctx, insts, way=way)
        for run in range(2):
            b.run()
            st = b.sync()
            for i, (ora, ost) in enumerate(want):
                what = f"{way} run {run} instance {i} {sizes[i]}"
                assert_groups_equal(rel.sorted_groups(b.outs[i].host()), ora, what)
                assert [st[i][x] for x in ("rows_passed", "join_matches", "groups")] == [ost[x] for x in ("rows_passed", "join_matches", "groups")], what
        b.close()

