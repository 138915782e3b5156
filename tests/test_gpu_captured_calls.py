"""Calls recorded into a graph, on a context whose tables are smaller than theirs:
what a recorded call leaves to be done has not been done for an eager call before
the first replay, and every replay and every eager call between them is right."""
import numpy as np
import pytest
import torch

import datagen
import oracle
from paper_2608_13696_amd import rel
from tests.gpu_util import assert_groups_equal, gpu_groups, to_dev

pytestmark = pytest.mark.gpu


def _tables(n, m, by, seed):
    T = datagen.make_tables(n, m, seed, day_lt=1800, group_by=by, fk_domain=m + 3, grp_card=7)
    T.prio = np.random.default_rng(seed).integers(-3, 3, m).astype(np.int8)
    return T


# (all scratch allocations hold at least 4 KB: the recorded call's tables fit, but are larger than the first call's)
@pytest.mark.parametrize("by,n0,m0,n1,m1", [("fk", 5000, 20, 5000, 100), ("prio_flag", 10, 20, 31, 100), ("dim_grp", 5000, 9, 5000, 30)])
def test_plain_call_recorded_before_its_size_ran(by, n0, m0, n1, m1):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        c = rel.Context(0, stream=s)
        small, large = _tables(n0, m0, by, 1), _tables(n1, m1, by, 2)
        dev = [to_dev(T) for T in (small, large)]
        want = [oracle.run_tables(T)[0] for T in (small, large)]

        def call(i):
            return c.filter_join_agg(*dev[i], (small, large)[i].day_lt, by, stats=False)[0]

        assert_groups_equal(gpu_groups(call(0)), want[0], "first")
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            out = call(1)
        assert_groups_equal(gpu_groups(call(1)), want[1], "eager, before a replay")
        for k in range(4):
            out.n_groups.fill_(-1)
            g.replay()
            assert_groups_equal(gpu_groups(out), want[1], f"replay {k}")
            assert_groups_equal(gpu_groups(call(k % 2)), want[k % 2], f"eager after replay {k}")
        assert c.sync() == 0
        c.close()


@pytest.mark.parametrize("hint", [0, 40])
def test_groupby_recorded_before_its_size_ran(hint):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        c = rel.Context(0, stream=s)
        r = np.random.default_rng(5)
        data = [(r.integers(-4, 4, n), r.integers(-99, 99, n), r.integers(-9, 9, n).astype(np.int32)) for n in (10, 31)]
        dev = [[torch.from_numpy(a).cuda() for a in d] for d in data]
        want = [oracle.groupby_agg(*d) for d in data]

        def call(i):
            return c.groupby_agg(*dev[i], capacity_hint=hint and (4, 20)[i])

        assert_groups_equal(gpu_groups(call(0)), want[0], "first")
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            out = call(1)
        assert_groups_equal(gpu_groups(call(1)), want[1], "eager, before a replay")
        for k in range(4):
            out.n_groups.fill_(-1)
            g.replay()
            assert_groups_equal(gpu_groups(out), want[1], f"replay {k}")
            assert_groups_equal(gpu_groups(call(k % 2)), want[k % 2], f"eager after replay {k}")
        assert c.sync() == 0
        c.close()
