"""The join placement that a plan asks for under a hot key, between the two limits on its groups."""
import numpy as np
import pytest
import torch

from paper_2608_13696_amd import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,share,groups,plain", [(2_000_000, 0.03, 1600, True), (8_400_000, 0.03, 1600, False), (8_400_000, 0.2, 1600, True),
                                                  (33_000_000, 0.1, 1600, False), (33_000_000, 0.3, 1600, True), (8_400_000, 0.03, 900, True),
                                                  (2_000_000, 0.3, 3000, False), (2_000_000, 0.0, 900, False)])
def test_plain_join_under_a_hot_key(n, share, groups, plain):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(1)
    ints = lambda k, hi, dt=torch.int32: torch.randint(0, hi, (k,), generator=g, device="cuda", dtype=dt)  # noqa: E731
    m = 100_000
    fk = ints(n, m)
    fk[torch.rand(n, generator=g, device="cuda") < share] = 7
    fact = {"fk": fk, "day": ints(n, 2557)}
    dim = {"pk": torch.randperm(m, generator=g, device="cuda", dtype=torch.int32), "prio": None,
           "grp": torch.arange(m, device="cuda", dtype=torch.int32) % groups}
    ctx = rel.Context(0)
    # a network that gives 0: as many groups as the sketch estimates (1566 for 1600, 919 for 900, 2711 for 3000)
    p = rel.Planner(ctx, np.zeros(6914), np.zeros(40), np.ones(40), 0.0)
    plan, _ = p.plan(fact, dim, 1200, "dim_grp", ints(256, n, torch.int64), ints(256, m, torch.int64))
    assert (plan.join_placement == rel.PLACE["global"]) == plain, plan.group_capacity
    p.close()
    ctx.close()
