"""GPU parity of the plain fused path over dim sides of few keys, on both sides of the
number of fact rows from which their index is no hash table any more."""
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


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1])
@pytest.mark.parametrize("m,stride", [(1, 1), (2, 1), (2, 40), (5, 2), (100, 1), (1001, 2), (4000, 30), (65_536, 1), (65_536, 3)])
def test_few_dim_keys(ctx, n, m, stride):
    T = datagen.make_tables(n, m, m + stride, day_lt=1500, group_by="prio_flag", fk_domain=m + m // 3 + 1, grp_card=7)
    r = np.random.default_rng(m)
    T.pk, T.fk = T.pk * stride - 3, T.fk * stride - 3
    T.prio = r.integers(-3, 3, m).astype(np.int8)
    T.grp = r.integers(-5, 300, m).astype(np.int32)
    fact, dim = to_dev(T)
    for by in ("prio_flag", "dim_grp", "fk"):
        T.group_by = by
        plan = rel.Plan(0, rel.PLACE["auto"], rel.PLACE["global"], 0, 0)
        out, st = ctx.filter_join_agg(fact, dim, T.day_lt, by, plan=plan)
        want, ws = oracle.run_tables(T)
        assert_groups_equal(gpu_groups(out), want, f"n={n} m={m} stride={stride} {by}")
        assert (st["rows_passed"], st["join_matches"]) == (ws["rows_passed"], ws["join_matches"])
    if m > 1:
        dim["pk"][m - 1] = dim["pk"][0]
        with pytest.raises(rel.RelError) as e:
            ctx.filter_join_agg(fact, dim, T.day_lt, "prio_flag", plan=plan)
        assert e.value.status == rel.DUPLICATE_KEY
