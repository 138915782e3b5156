"""What librel's host side keeps, reuses and gives back, without a GPU."""
import os

import pytest

from tests import hoststub

pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(hoststub.ROOT, "paper_2608_13696_amd", "librel.so")),
                                reason="librel.so not built")


@pytest.fixture
def host(tmp_path_factory):
    return lambda body: hoststub.run(tmp_path_factory, body)


@pytest.mark.parametrize("by", ["fk", "prio_flag"])
def test_recorded_fill_counts_for_the_recorded_call_only(host, by):
    host(f"""
    c = new_ctx()
    fill = "k_fill_u64" if {by!r} == "fk" else "k_init_groups"
    small, large = (5000, 20) if {by!r} == "fk" else (10, 20), (5000, 100) if {by!r} == "fk" else (31, 100)
    assert query(c, *small, {by!r}) == 0 and launched(kernels(), fill)  # a first use
    assert query(c, *small, {by!r}) == 0 and not launched(kernels(), fill)
    stub.stub_capture(1)
    assert query(c, *large, {by!r}) == 0 and launched(kernels(), fill)
    stub.stub_capture(0)
    assert query(c, *large, {by!r}) == 0 and launched(kernels(), fill)  # nothing has run yet
    assert query(c, *large, {by!r}) == 0 and not launched(kernels(), fill)
    """)


def test_table_memory_is_kept_for_a_stream_while_the_context_is_on_it(host):
    host("""
    c = new_ctx(0x1000)
    st, t = table(c, 100_000); assert st == 0
    slots = stub.stub_used()
    L.rel_join_table_destroy(t)
    assert stub.stub_used() == slots and stub.stub_frees() == 0
    st, t = table(c, 100_000)  # takes it again
    assert stub.stub_used() == slots
    L.rel_ctx_set_stream(c, ctypes.c_void_p(0x2000))
    stub.stub_kill(0x1000)  # the borrowed stream's owner destroys it
    L.rel_join_table_destroy(t)
    assert stub.stub_dead_uses() == 0
    stub.stub_revive(0x1000)  # a new stream at the old one's address: nothing orders it after the old one's work
    L.rel_ctx_set_stream(c, ctypes.c_void_p(0x1000))
    st, t2 = table(c, 100_000)
    assert stub.stub_used() > slots or stub.stub_frees() == 1
    L.rel_join_table_destroy(t2)
    L.rel_ctx_destroy(c)
    assert stub.stub_used() == 0
    """)


def test_table_memory_of_recorded_work_is_not_kept(host):
    host("""
    c = new_ctx()
    st, t = table(c, 100_000)
    stub.stub_capture(1)
    assert L.rel_join_probe(c, t, column(), None, 1000, column(), column(), 1000, column()) == 0
    stub.stub_capture(0)
    L.rel_join_table_destroy(t)
    assert stub.stub_frees() == 1
    st, t = table(c, 100_000)
    L.rel_join_table_destroy(t)
    assert stub.stub_frees() == 1
    stub.stub_capture(1)  # kept memory is not for a recorded build either, and a recorded build's is not kept
    st, t = table(c, 100_000)
    L.rel_join_table_destroy(t)
    stub.stub_capture(0)
    assert stub.stub_frees() == 2
    """)


@pytest.mark.parametrize("call", ["query(c, 1_000_000, 500_000, 'fk')", "table(c, 300_000)[0]", "batch(c, [(1000, 100_000, 'fk')])"])
def test_kept_table_memory_is_given_back_when_there_is_none_left(host, call):
    host(f"""
    def batch(c, sizes):
        items = (rel.BatchItem * len(sizes))()
        for it, (n, m, by) in zip(items, sizes):
            it.fact, it.dim, it.q, it.out = fact(n), dim(m), rel.Query(1000, rel.GROUP_BY[by]), groups(n)
        return L.rel_batch_create(c, items, len(sizes), None, 0, P(ctypes.c_void_p()))
    c = new_ctx()
    st, t = table(c, 4_000_000)
    assert st == 0
    L.rel_join_table_destroy(t)
    stub.stub_limit(stub.stub_used() + 1_000_000)
    assert {call} == 0
    assert stub.stub_frees() >= 1
    """)


def test_batch_without_memory_for_the_groups_of_large_instances(host):
    """The working memory beside the tables is one that a batch can do without."""
    host("""
    k, n, m = 256, 100_000, 20_000
    def batch(c):
        items = (rel.BatchItem * k)()
        for it in items:
            it.fact, it.dim, it.q, it.out = fact(n), dim(m), rel.Query(1000, rel.GROUP_BY["dim_grp"]), groups(n)
        h = ctypes.c_void_p()
        before = stub.stub_used()
        st = L.rel_batch_create(c, items, k, None, 0, P(h))
        used = stub.stub_used() - before
        if st == 0:
            L.rel_batch_destroy(h)
        return st, used
    c = new_ctx()
    st, all_of_it = batch(c)
    extra = k * n * 16
    assert st == 0 and all_of_it > extra
    stub.stub_limit(stub.stub_used() + all_of_it - extra)
    st, tables = batch(c)
    assert st == 0 and tables < all_of_it - extra
    stub.stub_limit(stub.stub_used() + tables - 1)
    assert batch(c)[0] == rel.OOM
    """)


@pytest.mark.parametrize("hint", [0, 1_000_000])
def test_groupby_without_memory_to_partition_its_rows(host, hint):
    host(f"""
    n = 20_000_000
    c = new_ctx()
    assert groupby(c, n, {hint}) == 0 and launched(kernels(), "k_gb_scatter")
    L.rel_ctx_destroy(c)
    c = new_ctx()
    stub.stub_limit(stub.stub_used() + 32 * (2 << 25 if not {hint} else 2 << 20) + n * 15)  # the group table, and too little more
    assert groupby(c, n, {hint}) == 0
    names = kernels()
    assert not launched(names, "k_gb_scatter") and launched(names, "k_groupby_global" if {hint} else "k_groupby_lds")
    assert L.rel_last_error(c) == b""
    """)


def test_planned_join_without_memory_for_its_partials(host):
    """The partials' memory is taken last, so that every limit from what the call needs at the least upwards will do."""
    host("""
    n, m, expected = 8_000_000, 6_000_000, 3_000_000
    def call(limit):
        c = new_ctx()
        stub.stub_limit(limit if limit else BIG)
        plan = rel.Plan(expected, rel.PLACE["global"], rel.PLACE["partitioned"], 0, 0)
        st, names, used = query(c, n, m, "dim_grp", plan), kernels(), stub.stub_used()
        assert st != 0 or L.rel_last_error(c) == b""
        stub.stub_limit(BIG)
        L.rel_ctx_destroy(c)
        return st, launched(names, "k_part_join_eagerILb1E"), used
    st, partials, most = call(0)
    assert st == 0 and partials
    least = 2 * (n * 17 + 1024) + m * 16 + 32 * (2 << 22)  # columns and the group table
    seen = set()
    for limit in [*range(least, most, (most - least) // 40), most]:
        st, partials, used = call(limit)
        assert st == 0 or not seen, limit  # refused for want of bookkeeping memory at the lowest limits only
        if st == 0:
            seen.add(partials)
    assert seen == {False, True}
    """)
