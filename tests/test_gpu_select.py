"""GPU parity of the two-pass selection where its splits change: the edges of
a wave's 2048-row step and of a tile, the share of rows at which the second
pass changes its way of writing, and the size above which tiles grow."""
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
