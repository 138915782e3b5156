"""GPU parity of the stand-alone group-by on each of its ways (LDS tables, the
device table, partitioned rows) and at the sizes where it changes between them:
row counts, group counts with and without a hint, hot keys, keys that crowd one
bin, the empty-slot key, and outputs or tables that are too small."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_13696_amd import rel
from tests.gpu_util import assert_groups_equal, gpu_groups

pytestmark = pytest.mark.gpu
MIN = np.iinfo(np.int64).min


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = rel.Context(0)
    yield c
    c.close()


def _rows(key, seed):
    rng = np.random.default_rng(seed)
    price = rng.integers(-(2 ** 62), 2 ** 62, size=key.size, dtype=np.int64)
    qty = rng.integers(-(2 ** 31), 2 ** 31, size=key.size, dtype=np.int64).astype(np.int32)
    return price, qty


def _check(ctx, key, sel=None, hint=0, seed=0):
    price, qty = _rows(key, seed)
    D = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731
    g = ctx.groupby_agg(D(key), D(price), D(qty), D(sel), capacity_hint=hint)
    assert ctx.sync() == 0
    assert_groups_equal(gpu_groups(g), oracle.groupby_agg(key, price, qty, sel))


def _bin(key):
    """The 32-bit hash whose top bits choose a key's bin."""
    k = key.astype(np.uint64)
    x = (k & np.uint64(0xFFFFFFFF)) ^ (((k >> np.uint64(32)) * np.uint64(0x85EBCA6B)) & np.uint64(0xFFFFFFFF))
    return (x * np.uint64(2654435769)) & np.uint64(0xFFFFFFFF)


# 7168-row tiles; partitioned from 65536 rows with a hint and 131072 without
@pytest.mark.parametrize("n", [1, 1023, 65_535, 65_536, 71_680, 71_681, 131_071, 131_072, 300_007])
@pytest.mark.parametrize("groups", [1, 300, 513, 40_000])
@pytest.mark.parametrize("hinted", [False, True])
def test_sizes_and_group_counts(ctx, n, groups, hinted):
    rng = np.random.default_rng(n + groups)
    keys = rng.integers(MIN, -(MIN + 1), size=groups, dtype=np.int64)
    keys[0] = MIN  # the empty-slot marker is a key like any other
    key = keys[rng.integers(0, groups, size=n)]
    sel = np.flatnonzero(rng.random(n) < 0.6).astype(np.int32) if n % 2 else None
    _check(ctx, key, sel, groups if hinted else 0, seed=n)


@pytest.mark.parametrize("hinted", [False, True])
def test_every_row_its_own_group(ctx, hinted):
    n = 1_000_003
    _check(ctx, np.random.default_rng(1).permutation(n).astype(np.int64) * (1 << 33), None, n if hinted else 0)


@pytest.mark.parametrize("share", [0.3, 0.97])
def test_hot_keys(ctx, share):
    """One key with most rows: its bin is cut into pieces of 32768 rows."""
    rng = np.random.default_rng(2)
    key = rng.integers(0, 50_000, size=400_001, dtype=np.int64)
    key[rng.random(key.size) < share] = 77
    _check(ctx, key, None, 50_000)
    _check(ctx, key)


@pytest.mark.parametrize("crowd_rows", [30_000, 200_000])  # within one piece; cut into several
def test_keys_that_crowd_one_bin(ctx, crowd_rows):
    """More groups in one bin than its LDS table holds: the rest go to the device table. (Without a hint: the device
    table hashes such keys side by side too, and a table sized from a hint gives up after 256 probe steps.)"""
    rng = np.random.default_rng(3)
    pool = rng.integers(MIN, -(MIN + 1), size=12_000_000, dtype=np.int64)
    crowd = pool[_bin(pool) >> np.uint64(21) == 5]
    assert crowd.size > 4500
    rest = pool[:140_000]
    key = np.concatenate([crowd[rng.integers(0, crowd.size, size=crowd_rows)], rest])
    key = key[rng.permutation(key.size)]
    _check(ctx, key)


def test_small_outputs_and_tables_overflow(ctx):
    n = 200_000
    key = np.arange(n, dtype=np.int64)
    price, qty = _rows(key, 4)
    d = [torch.from_numpy(a).cuda() for a in (key, price, qty)]
    g = ctx.groupby_agg(*d, capacity_hint=n, out_cap=1000)
    assert ctx.sync() == rel.DEV_OVERFLOW and int(g.n_groups) == n
    ctx.groupby_agg(*d, capacity_hint=1000)  # a table for 1000 groups
    assert ctx.sync() == rel.DEV_OVERFLOW
    _check(ctx, key, None, n)  # and none of it stays behind
