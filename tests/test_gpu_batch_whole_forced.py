"""The edges of the instances that one workgroup takes whole, where the estimate of
what is faster would send some of them to the shared tables."""
import functools

import pytest

from paper_2608_13696_amd import rel
from tests import test_gpu_batch_whole as edges
from tests.test_gpu_batch_whole import ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def whole(monkeypatch):
    monkeypatch.setattr(rel, "Batch", functools.partial(rel.Batch, way="whole"))


@pytest.mark.parametrize("m", [1, 63, edges.RANK_ROWS - 1, edges.RANK_ROWS, edges.RANK_ROWS + 1, 6000])
def test_group_attribute_ranges(ctx, m):  # noqa: F811
    edges.test_group_attribute_ranges(ctx, m)


def test_rows_tiles_and_empty(ctx):  # noqa: F811
    edges.test_rows_tiles_and_empty(ctx)


@pytest.mark.parametrize("by", ["fk", "prio_flag"])
def test_keys_and_tables(ctx, by):  # noqa: F811
    edges.test_keys_and_tables(ctx, by)


def test_changed_inputs_and_hints(ctx):  # noqa: F811
    edges.test_both_ways_and_changed_inputs(ctx)
    edges.test_wide_groups_behind_a_small_hint(ctx)


@pytest.mark.parametrize("m", [40, 6000, 100_000])
def test_repeated_key_is_reported(ctx, m):  # noqa: F811
    edges.test_repeated_key_is_reported(ctx, m)
