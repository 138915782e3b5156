"""GPU parity of the sketch kernels where they change course: row counts around a
workgroup's and a load's share, keys of both signs around the hash's carry, keys
whose register row lies past the hash's high word, few distinct keys, and samples
with repeats, zeros and fewer entries than threads."""
import numpy as np
import pytest
import torch

import datagen
import oracle
from paper_2608_13696_amd import rel
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu

# keys whose hash has 26 zero bits below the register number
DEEP = [6598086, 194818587, 246457805, 415665071, 452933367, 621728452]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = rel.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,m,k", [(1, 1, 1), (3, 4, 2), (4095, 4096, 63), (4097, 4099, 64), (8191, 8193, 65), (16_385, 5, 255),
                                   (600_001, 70_003, 256), (2_200_007, 2_100_003, 256)])
@pytest.mark.parametrize("keys", ["spread", "few", "deep"])
def test_sketch_edges(ctx, n, m, k, keys):
    r = np.random.default_rng(n + k)
    T = datagen.make_tables(n, m, 3 + n, day_lt=1000, group_by="dim_grp", grp_card=max(1, min(m, 50)))
    if keys == "spread":
        T.fk = r.integers(-(2**31), 2**31, n).astype(np.int32)
        T.grp = r.integers(-(2**31), 2**31, m).astype(np.int32)
    elif keys == "few":
        T.fk = r.integers(-1, 3, n).astype(np.int32)
        T.grp = np.zeros(m, np.int32)
    else:
        T.fk[r.integers(0, n, min(n, 7))] = r.choice(DEEP, min(n, 7))
        T.grp = np.full(m, DEEP[2], np.int32)
    fs, ds = datagen.sample_index(k, n, 5, 1), datagen.sample_index(k, m, 5, 2)
    fact, dim = to_dev(T)
    feat, hll = rel.sketch(ctx, fact, dim, T.day_lt, T.group_by, torch.from_numpy(fs).cuda(), torch.from_numpy(ds).cuda())
    hf, hg = oracle.hll_registers(T.fk), oracle.hll_registers(T.grp)
    hll = hll.cpu().numpy()
    assert np.array_equal(hll[:64], hf) and np.array_equal(hll[64:], hg)
    ref = oracle.sketch_features(T.fk, T.day, T.pk, T.grp, T.day_lt, T.group_by, fs, ds, hf, hg)
    got = feat.cpu().numpy().astype(np.float64)
    assert np.allclose(got, ref.astype(np.float32).astype(np.float64), rtol=1e-6, atol=1e-6), \
        np.flatnonzero(~np.isclose(got, ref, rtol=1e-6, atol=1e-6))
