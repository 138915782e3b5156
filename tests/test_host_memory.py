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
