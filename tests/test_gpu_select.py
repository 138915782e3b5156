"""GPU parity of the two-pass selection where its splits change: the edges of
a wave's 2048-row step and of a tile, the share of rows at which the second
pass changes its way of writing, the size above which tiles grow, and
predicate literals at the ends of their column's type."""
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


@pytest.mark.parametrize("n", [1, 3, 255, 257, 2047, 2048, 2049, 8193, 16383, 16384, 16385, 49_153,
                               4096 * 16384, 4096 * 16384 + 1, 4096 * 32768 + 2049])
def test_sizes_around_steps_and_tiles(ctx, n):
    col = np.random.default_rng(n).integers(0, 100, size=n, dtype=np.int32)
    d = torch.from_numpy(col).cuda()
    for op, lit in (("lt", 60), ("ge", 97), ("ne", 200)):
        idx, c = ctx.filter_compact(d, op, lit)
        exp = oracle.filter_compact(col, op, lit)
        assert c == exp.shape[0] and np.array_equal(idx.cpu().numpy(), exp), (op, lit)


@pytest.mark.parametrize("selected", [0, 1, 4095, 4096, 4097, 16384])  # of a step's 16384 rows
def test_steps_around_the_sparse_limit(ctx, selected):
    rng = np.random.default_rng(selected)
    col = np.zeros((3, 16384), np.int32)
    for step in range(3):
        col[step, rng.permutation(16384)[:selected if step == 1 else 5000]] = 1
    col = col.reshape(-1)[:-7]
    idx, c = ctx.filter_compact(torch.from_numpy(col).cuda(), "eq", 1)
    assert np.array_equal(idx.cpu().numpy(), oracle.filter_compact(col, "eq", 1)) and c == int(col.sum())


def _float_values(dt):
    f = np.finfo(dt)
    v = [0.0, -0.0, f.smallest_subnormal, -f.smallest_subnormal, f.tiny, -f.tiny, 0.1, -0.1, 1.0, f.max, -f.max, np.inf, -np.inf, np.nan]
    return np.array(v, dt)


@pytest.mark.parametrize("mode", ["compiled", "interpreted"])
@pytest.mark.parametrize("dt", [np.float32, np.float64, np.int8, np.int16, np.int32, np.int64])
def test_literals_at_the_ends_of_the_type(ctx, mode, dt):
    """Every operator against literals that the column's type holds, rounds or cannot hold."""
    n = 2048 + 300  # one whole step of a wave and rows tested one by one
    if np.dtype(dt).kind == "f":
        pool = _float_values(dt)
        lits = [float(x) for x in _float_values(np.float64)] + [float(np.float32(0.1)), 1e39, 1e-46, 16777217.0]
    else:
        i = np.iinfo(dt)
        pool = np.array([i.min, i.min + 1, -1, 0, 1, 63, 64, i.max - 1, i.max], dt)
        big = np.iinfo(np.int64)
        lits = sorted({int(i.min), int(i.max), -1, 0, 64, max(int(i.min) - 1, int(big.min)), min(int(i.max) + 1, int(big.max)),
                       int(big.min), int(big.max)})
    col = pool[np.random.default_rng(5).integers(0, pool.size, size=n)]
    d = torch.from_numpy(col).cuda()
    terms = [dict(column=0, op=op, values=[v]) for op in ("lt", "le", "gt", "ge", "eq", "ne") for v in lits]
    terms += [dict(column=0, op="between", values=[a, b]) for a, b in ((lits[0], lits[-1]), (lits[-1], lits[0]), (lits[1], lits[1]))]
    terms += [dict(column=0, op="in", values=lits[:16]), dict(column=0, op="in", values=[lits[0], lits[0]]),
              dict(column=0, op="in", values=[-1, 0, 62]), dict(column=0, op="in", values=[-1, 0, 63])]
    if mode == "compiled":  # one kernel each: a third of them
        terms = terms[::3]
    for t in terms:
        p = rel.Predicate(ctx, [t], [d.dtype], mode)
        idx, _ = p.filter([d])
        p.close()
        assert np.array_equal(idx.cpu().numpy(), oracle.pred_filter([col], [t])), (t["op"], t["values"])
