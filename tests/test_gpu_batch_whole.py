"""GPU parity of the batched form at the edges of the instances that one workgroup
takes whole: the group arrays' capacity, numbered attributes, chunks, the join
table's places and widths, what is left to the shared tables, and both ways in
one batch."""
import numpy as np
import pytest
import torch

import datagen
import oracle
from paper_2608_13696_amd import rel
from tests.gpu_util import assert_groups_equal, to_dev

pytestmark = pytest.mark.gpu

CAP, RANK_ROWS = 7168, 5120  # groups of one chunk; dim rows that may have their attributes numbered


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = rel.Context(0)
    yield c
    c.close()


def _instance(n, m, by, seed, span=None, low=0, gap=1, kmin=0, outside=True):
    """Dim keys kmin, kmin + gap, ...; attributes over exactly [low, low + span)."""
    T = datagen.make_tables(n, m, seed, day_lt=1800, group_by=by, grp_card=max(1, min(m, 5)))
    r = np.random.default_rng(seed)
    T.pk = (kmin + gap * r.permutation(m)).astype(np.int32)
    if span is not None:
        a = low + r.integers(0, span, m)
        if m > 1:
            a[0], a[m - 1] = low, low + span - 1
        if by == "dim_grp":
            T.grp = a.astype(np.int32)
        else:
            T.prio = a.astype(np.int8)
    T.fk = (T.pk[r.integers(0, m, n)] if m else r.integers(-5, 5, n)).astype(np.int32)
    if outside and n > 8:  # keys that match nothing, next to the range and as far off as there are
        T.fk[:: max(n // 7, 1)] = np.int32(kmin - 1 if kmin > np.iinfo(np.int32).min else kmin + gap * m)
        T.fk[1 :: max(n // 5, 1)] = np.iinfo(np.int32).min if kmin > np.iinfo(np.int32).min else np.iinfo(np.int32).max
        T.fk[2 :: max(n // 6, 1)] = np.iinfo(np.int32).max if kmin < 2**30 else np.iinfo(np.int32).min
    return T


def _run(ctx, tables, hints=None, runs=2, change=None):
    insts = []
    for i, T in enumerate(tables):
        fact, dim = to_dev(T)
        insts.append((fact, dim, T.day_lt, T.group_by, hints[i] if hints else 0))
    b = rel.Batch(ctx, insts)
    for run in range(runs):
        if change and run:
            change(tables, insts)
        for out in b.outs:
            out.key.fill_(-7)
            out.n_groups.fill_(-1)
        b.run()
        st = b.sync()
        for i, T in enumerate(tables):
            ora, ost = oracle.run_tables(T)
            what = f"run {run} instance {i} n={T.n} m={T.m} group_by={T.group_by}"
            assert_groups_equal(rel.sorted_groups(b.outs[i].host()), ora, what)
            assert [st[i][x] for x in ("rows_passed", "join_matches", "groups")] == \
                [ost[x] for x in ("rows_passed", "join_matches", "groups")], what
    b.close()


@pytest.mark.parametrize("m", [1, 63, RANK_ROWS - 1, RANK_ROWS, RANK_ROWS + 1, 6000])
def test_group_attribute_ranges(ctx, m):
    spans = [1, 3, 4, 15, 16, 255, 256, CAP - 1, CAP, CAP + 1, 2 * CAP, 3 * CAP + 5, 65535, 65536, 1 << 20]
    _run(ctx, [_instance(9001 + i, m, "dim_grp", 100 + i, span=s, low=(-70000 if i % 2 else 12345))
               for i, s in enumerate(spans) if m > 1 or s == 1])


def test_rows_tiles_and_empty(ctx):
    tables = [_instance(n, m, by, 7 + n + m, span=40)
              for by in ("dim_grp", "prio_flag") for n in (1, 4095, 4096, 4097, 12289) for m in (2, 5000)]
    for n, m in ((0, 10), (50, 0), (0, 0)):
        T = datagen.make_tables(n, m, 11 + n + m, day_lt=900, group_by="dim_grp", grp_card=7)
        if T.grp is None:
            T.grp = np.zeros(0, np.int32)
        tables.append(T)
    _run(ctx, tables)


@pytest.mark.parametrize("by", ["fk", "prio_flag"])
def test_keys_and_tables(ctx, by):
    lim = np.iinfo(np.int32)
    span = None if by == "fk" else 256
    low = -128
    tables = [_instance(9000, m, by, 30 + i, span=span if m > 256 else (None if by == "fk" else 3), low=low, gap=gap, kmin=k0)
              for i, (m, gap, k0) in enumerate([
                  (CAP, 1, 0), (CAP + 1, 1, -3), (CAP // 2, 2, 0), (2000, 3, 5), (20, 1, lim.min), (20, 1, lim.max - 19),
                  (2, 2**31 - 1, -2), (9, 4, -16), (8, 4, -16), (30000, 2, -30000), (100_000, 1, 17), (60_000, 2, 4)])]
    _run(ctx, tables)


def test_both_ways_and_changed_inputs(ctx):
    """Large instances beside small ones, some of which are left to the shared tables; the columns
    change between replays, and with them what an instance is taken by."""
    tables = [_instance(400_000, 50_000, "dim_grp", 50, span=30_000), _instance(300_000, 70_000, "fk", 51)]
    tables += [_instance(2000 + 37 * i, 600, by, 60 + i, span=span, gap=gap)
               for i, (by, span, gap) in enumerate([("dim_grp", 9, 1), ("dim_grp", 200_000, 1), ("dim_grp", 9, 50), ("fk", None, 1),
                                                    ("fk", None, 7), ("prio_flag", 5, 1), ("dim_grp", 60_000, 1)])]

    def change(tables, insts):
        for T, (_, dim, *_rest) in zip(tables[2:], insts[2:]):
            if T.group_by == "dim_grp":
                T.grp = (T.grp.astype(np.int64) // 3 * (1 if T.grp.max() > 100 else 30_000)).astype(np.int32)
                dim["grp"].copy_(torch.from_numpy(T.grp))

    _run(ctx, tables, runs=3, change=change)


def test_wide_groups_behind_a_small_hint(ctx):
    """A hint that promises few groups of a wide attribute range: no spill memory was laid out for them."""
    tables = [_instance(20_000, 6000, "dim_grp", 80, span=50_000), _instance(20_000, 6000, "dim_grp", 81, span=9)]
    tables[0].grp = (tables[0].grp // 10_000 * 10_000).astype(np.int32)
    _run(ctx, tables, hints=[16, 16])


@pytest.mark.parametrize("m", [40, 6000, 100_000])
def test_repeated_key_is_reported(ctx, m):
    T = _instance(9000, m, "dim_grp", 90, span=300)
    T.pk[m // 2] = T.pk[m // 3]
    fact, dim = to_dev(T)
    b = rel.Batch(ctx, [(fact, dim, T.day_lt, T.group_by, 0)])
    b.run()
    with pytest.raises(rel.RelError) as e:
        b.sync()
    assert e.value.status == rel.DUPLICATE_KEY
    b.close()
    assert ctx.sync() == 0
