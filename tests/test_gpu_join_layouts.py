"""GPU parity of stand-alone join tables around the choice between the dense
array and the hash table, and of gathers around the sizes that are read by
slices; table memory that passes from one table to the next."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2608_13696_amd import rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = rel.Context(0)
    yield c
    c.close()


D = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731


def _check(table, fk, sel, pk, payload):
    fi, pl, c = table.probe(D(fk), D(sel))
    efi, epl = oracle.join_probe(fk, sel, pk, payload)
    fi, pl = fi.cpu().numpy(), pl.cpu().numpy()
    o = np.argsort(fi)
    assert c == efi.shape[0]
    assert np.array_equal(fi[o], efi) and np.array_equal(pl[o], epl)


# a table may be dense from 65536 keys on, and is when they span at most twice their number
@pytest.mark.parametrize("m", [65_535, 65_536, 100_003])
@pytest.mark.parametrize("span,base", [(1.0, 0), (2.0, -(2 ** 31)), (2.0, None), (2.0001, -50_000), (40.0, 7)])
@pytest.mark.parametrize("with_payload", [False, True])
def test_key_ranges(ctx, m, span, base, with_payload):
    rng = np.random.default_rng(m)
    width = int(m * span) + (span > 2)
    base = 2 ** 31 - width if base is None else base  # (None: the range ends at the largest int32)
    off = np.concatenate([[0, width - 1], 1 + rng.permutation(width - 2)[:m - 2]])
    pk = (rng.permutation(off) + base).astype(np.int32)
    payload = rng.integers(-(2 ** 31), 2 ** 31, size=m, dtype=np.int64).astype(np.int32) if with_payload else None
    if with_payload:
        payload[:4] = [0, -1, -(2 ** 31), 2 ** 31 - 1]
    n = 300_007
    fk = np.clip(rng.integers(base - 1000, base + width + 1000, size=n), -(2 ** 31), 2 ** 31 - 1).astype(np.int32)
    fk[:3] = [-(2 ** 31), 2 ** 31 - 1, -1]
    sel = np.flatnonzero(rng.random(n) < 0.45).astype(np.int32)
    t = ctx.join_build(D(pk), D(payload))
    assert ctx.sync() == 0
    _check(t, fk, sel, pk, payload)
    _check(t, fk, None, pk, payload)
    t.close()


@pytest.mark.parametrize("with_payload", [False, True])
@pytest.mark.parametrize("span", [1, 50])
def test_repeated_keys_are_reported_by_the_build(ctx, span, with_payload):
    m = 70_000
    pk = (np.random.default_rng(2).permutation(m) * span).astype(np.int32)
    pk[-1] = pk[17]
    t = ctx.join_build(D(pk), D(np.arange(m, dtype=np.int32)) if with_payload else None)
    assert ctx.sync() == rel.DEV_DUPKEY
    t.close()


def test_keys_at_an_odd_address_and_high_load(ctx):
    m = 80_001
    pk = np.random.default_rng(3).permutation(m).astype(np.int32)
    fk = np.arange(-5, m + 5, dtype=np.int32)
    payload = pk[::-1].copy()
    buf = torch.empty(m + 1, dtype=torch.int32, device="cuda:0")
    buf[1:] = D(pk)
    for keys in (buf[1:], D(pk)):
        t = ctx.join_build(keys, D(payload), max_load=0.9)
        assert ctx.sync() == 0
        _check(t, fk, None, pk, payload)
        t.close()


def test_memory_of_closed_tables_is_reused_safely():
    ctx = rel.Context(0)
    rng = np.random.default_rng(4)
    m = 90_000
    other = torch.cuda.Stream()
    for k in range(6):
        pk = (rng.permutation(m) * (1 if k % 2 else 30)).astype(np.int32)  # dense and hash layouts in turn
        fk = pk[rng.integers(0, m, size=200_001)]
        t = ctx.join_build(D(pk))
        _check(t, fk, None, pk, None)
        if k == 3:  # probed on a second stream as well
            torch.cuda.synchronize()
            with torch.cuda.stream(other):
                ctx.set_stream(other)
                _check(t, fk, None, pk, None)
                torch.cuda.synchronize()
            ctx.set_stream(torch.cuda.current_stream())
        t.close()
    t = ctx.join_build(D(pk))
    raw = ctypes.c_void_p(t.h.value)
    t.h = None
    ctx.close()  # a table may outlive its context as far as being destroyed
    assert rel.lib().rel_join_table_destroy(raw) == rel.OK


@pytest.mark.parametrize("dt", [torch.int8, torch.int16, torch.int32, torch.int64])
@pytest.mark.parametrize("mb", [4.0, 4.000001, 11.3, 41.0, 64.0, 64.000001])  # slices are 4 MB, at most 16 of them
def test_gather_by_slices(ctx, dt, mb):
    es = torch.empty(0, dtype=dt).element_size()
    rows = int(mb * (1 << 20)) // es + (mb != int(mb) and es > 1)
    n = (2 << 20) + 3
    g = torch.Generator(device="cuda:0").manual_seed(rows)
    src = torch.randint(-100, 100, (rows,), generator=g, device="cuda:0", dtype=torch.int32).to(dt)
    idx = torch.randint(0, rows, (n,), generator=g, device="cuda:0", dtype=torch.int32)
    idx[:4] = torch.tensor([0, rows - 1, rows // 2, 0], dtype=torch.int32)
    for count in (n, n - 2, 3, 0):
        cnt = torch.tensor([count], device="cuda:0")
        out, = ctx.join_gather(None, idx, cnt, [(src, "dim")])
        assert torch.equal(out[:count], src[idx[:count].long()])
    assert ctx.sync() == 0
    idx[5], idx[n - 1] = rows, -1  # out of range: zero, and the status bit
    out, = ctx.join_gather(None, idx, torch.tensor([n], device="cuda:0"), [(src, "dim")])
    assert int(out[5]) == 0 and int(out[n - 1]) == 0 and ctx.sync() == rel.DEV_BADARG
    ok = torch.ones(n, dtype=torch.bool, device="cuda:0")
    ok[5] = ok[n - 1] = False
    assert torch.equal(out[:n][ok], src[idx[ok].long()])
