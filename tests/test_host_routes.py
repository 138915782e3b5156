"""Which kernels a call launches, and how wide, at the sizes where the choice changes (without a GPU)."""
import os

import pytest

from tests import hoststub

pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(hoststub.ROOT, "paper_2608_13696_amd", "librel.so")),
                                reason="librel.so not built")


@pytest.fixture
def host(tmp_path_factory):
    return lambda body: hoststub.run(tmp_path_factory, body)


def test_whoever_reads_the_group_table_is_as_wide_as_the_table(host):
    """Groups that did not fit LDS are in the device table: no single workgroup may have to go through a large one."""
    host("""
    c = new_ctx()
    lds = lambda cap: rel.Plan(cap, rel.PLACE["lds"], rel.PLACE["global"], 0, 0)
    for n, m, by, plan in ((1000, 500, "prio_flag", None), (60_000, 15_000, "prio_flag", None), (262_144, 15_000, "prio_flag", None),
                           (262_145, 15_000, "prio_flag", None), (5000, 100_000, "dim_grp", lds(250_000)),
                           (250_000, 100_000, "dim_grp", lds(500_000)), (250_000, 100_000, "dim_grp", lds(600_000)),
                           (10_000, 100, "dim_grp", lds(100_000_000))):
        kernels()
        assert query(c, n, m, by, plan) == 0
        slots = 16
        while slots < 2 * (plan.group_capacity if plan else min(n, 65536)):
            slots *= 2
        grid = {part: g for name, g in kernels() for part in ("k_group_merge", "k_finalize") if part in name}
        assert "k_group_merge" in grid
        reader = 4 * grid["k_finalize"] if "k_finalize" in grid else grid["k_group_merge"] - 1  # (8192 slots of a finalize workgroup's ticket)
        assert reader * 8192 >= slots, (n, plan and plan.group_capacity, grid)
    """)


@pytest.mark.parametrize("by", ["prio_flag", "dim_grp"])
def test_small_dim_side_of_a_large_fact_side_is_a_dense_array(host, by):
    """Its range is looked for (k_key_minmax) where the rows that probe it are many; a hash table is built at once."""
    host(f"""
    c = new_ctx()
    for n, m, dense in ((60_000, 65_536, False), (1 << 21, 65_536, False), ((1 << 21) + 1, 1, True), (30_000_000, 16_000, True),
                        (60_000, 65_537, True), (30_000_000, 0, False)):
        kernels()
        assert query(c, n, m, {by!r}) == 0
        names = kernels()
        assert launched(names, "k_key_minmax") == dense and launched(names, "k_join_build") == (not dense), (n, m)
    """)


def test_batch_work_items_are_no_smaller_than_pays(host):
    """Instances that go by shared tables: about one item of rows per CU, unless the tuning asks for fewer rows."""
    host("""
    def grid(k, n, m):
        c = new_ctx()
        items = (rel.BatchItem * k)()
        for it in items:
            it.fact, it.dim, it.q, it.out, it.group_capacity = fact(n), dim(m), rel.Query(1000, rel.GROUP_BY["dim_grp"]), groups(n), 300
        tune = (rel.BatchTuning * 1)(rel.BatchTuning(31, 4, 256, 512, 65536, 0))
        kernels()
        assert L.rel_batch_create(c, items, k, tune, 1, P(ctypes.c_void_p())) == 0
        names = kernels()
        probe = [g for name, g in names if "k_batch_probe" in name]
        build = [g for name, g in names if "k_batch_build" in name]
        return launched(names, "k_batch_whole"), probe and probe[0], build and build[0]
    assert grid(1, 300_000, 75_000) == (False, 147, 74)      # 2048 rows, 1024 keys
    assert grid(4, 1_000_000, 1000) == (False, 248, 4)       # 15625 rows, rounded up to whole steps
    assert grid(1, 60_000_000, 1000)[1] == 916               # the tuning's 65536
    """)


def test_batch_work_items_are_a_share_of_what_their_kernel_takes(host):
    """A bucket's instances are one kernel's, and rows of many groups cost more than others: instances of another size
    or kind in the batch leave an instance's items as they are."""
    host("""
    def grids(*instances):
        c = new_ctx()
        items = (rel.BatchItem * len(instances))()
        for it, (n, m, hint) in zip(items, instances):
            it.fact, it.dim, it.q, it.out, it.group_capacity = fact(n), dim(m), rel.Query(1000, rel.GROUP_BY["dim_grp"]), groups(n), hint
        tune = (rel.BatchTuning * 2)(rel.BatchTuning(18, 8, 512, 512, 16384, 0), rel.BatchTuning(31, 4, 512, 0, 65536, 0))
        kernels()
        assert L.rel_batch_create_as(c, items, len(instances), tune, 2, 1, P(ctypes.c_void_p())) == 0
        return [g for name, g in kernels() if "k_batch_probe" in name]
    many, few, large = (100_000, 25_000, 20_000), (200_000, 25_000, 300), (1_000_000, 1000, 300)
    assert grids(*4 * [many]) == [4 * 25] and grids(*4 * [few]) == [4 * 49] and grids(*8 * [large]) == [8 * 31]
    assert grids(*4 * [many], *4 * [few], *8 * [large]) == [4 * 25 + 4 * 49, 8 * 31]
    """)


def test_batch_instances_of_many_dim_keys_go_by_shared_tables(host):
    """A workgroup that takes an instance whole reads all its dim keys again for each slice of its join table."""
    host("""
    def whole(k, n, m, by, hint=300):
        c = new_ctx()
        items = (rel.BatchItem * k)()
        for it in items:
            it.fact, it.dim, it.q, it.out, it.group_capacity = fact(n), dim(m), rel.Query(1000, rel.GROUP_BY[by]), groups(n), hint
        kernels()
        assert L.rel_batch_create(c, items, k, None, 0, P(ctypes.c_void_p())) == 0
        return sum(g for name, g in kernels() if "k_batch_whole" in name)
    for by in ("dim_grp", "prio_flag", "fk"):
        assert whole(1, 1000, 8_000_000, by) == 0 and whole(1, 1000, 1_000_000, by) == 0 and whole(4, 30_000, 1_000_000, by) == 0
        assert whole(256, 30_000, 3000, by) == 256 and whole(256, 300_000, 75_000, by) == 256 and whole(1, 1_000_000, 1000, by) == 0
    assert whole(300, 1000, 1 << 20, "fk") == 0  # more keys than group numbers
    """)


def test_batch_is_split_between_the_ways_only_for_a_clear_gain(host):
    """Instances of different sizes: a few of them apart cost the shared tables' kernels, one after another."""
    host("""
    def whole(k, hi):
        c = new_ctx()
        items = (rel.BatchItem * k)()
        for i, it in enumerate(items):
            n = int(1000 * (hi / 1000) ** (i / (k - 1)))
            it.fact, it.dim, it.q, it.out, it.group_capacity = fact(n), dim(n // 4), rel.Query(1000, rel.GROUP_BY["dim_grp"]), groups(n), 2 ** (7 * i % 17)
        tune = (rel.BatchTuning * 3)(rel.BatchTuning(12, 4, 512, 128, 4096, 1024), rel.BatchTuning(15, 1, 512, 512, 16384, 0),
                                     rel.BatchTuning(31, 8, 512, 512, 16384, 0))
        kernels()
        assert L.rel_batch_create(c, items, k, tune, 3, P(ctypes.c_void_p())) == 0
        return sum(g for name, g in kernels() if "k_batch_whole" in name)
    assert [whole(k, hi) for k, hi in ((54, 36_000), (144, 66_000), (234, 62_000))] == [54, 144, 234]
    assert 0 < whole(200, 400_000) < 200  # (the largest would keep the others waiting)
    """)


def test_tunings_are_measured_where_they_apply(host):
    """autotune.gpu_measure's batches launch the kernels that read the tuning, with the candidate's workgroup size."""
    host("""
    import types
    from paper_2608_13696_amd import autotune
    c = new_ctx()
    ctx = types.SimpleNamespace(h=c, check=lambda st: (_ for _ in ()).throw(AssertionError(st)) if st else None)
    class Tensor:
        is_cuda, device = True, None
        def __init__(self, n): self.n = n
        def numel(self): return self.n
        def data_ptr(self): return column()
    rel._alloc_groups = lambda cap, device: types.SimpleNamespace(c=groups(cap))
    class Events:
        def __init__(self, **kw): pass
        def record(self): pass
        def elapsed_time(self, other): return 1.0
    import torch
    torch.cuda.synchronize, torch.cuda.Event = (lambda: None), Events
    n, m = 3000, 700
    inst = ({k: Tensor(n) for k in ("fk", "price_cents", "qty", "day", "flag")}, {k: Tensor(m) for k in ("pk", "prio", "grp")}, 1000, "dim_grp", 90)
    for cand in (autotune.Candidate(4, 256, 512, 4096), autotune.Candidate(1, 128, 128, 4096, 1024)):
        kernels()
        autotune.gpu_measure(ctx, [inst] * 300)(cand)
        names = kernels()
        assert not launched(names, "k_batch_whole")
        assert launched(names, f"k_batch_probeILi{cand.block}ELi{cand.items_per_thread}E")
    """)


def test_workgroups_that_update_a_group_table_in_device_memory(host):
    """No more at once than its atomics are worth."""
    host("""
    c = new_ctx()
    for n in (1000, 30_000_000):
        kernels()
        assert query(c, n, 130_000, "dim_grp") == 0
        grids = [g for name, g in kernels() if "k_fusedILi2ELi1E" in name]
        assert grids == [1 if n == 1000 else 4 * 256]
    """)
