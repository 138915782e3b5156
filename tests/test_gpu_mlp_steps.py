"""The planner network's kernels where a workgroup's 16-sample steps end, and
above the size at which workgroups take several steps, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import datagen
from oracle import mlp as omlp
from paper_2608_13696_amd import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 257, 4096, 4097, 8209])
def test_forward_and_backward_at_step_edges(B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = rel.Context(0)
    rng = np.random.default_rng(B)
    th = omlp.he_uniform(datagen.unit(omlp.N_PARAMS, 3, 7)).astype(np.float32)
    x, t = rng.normal(size=(B, 40)).astype(np.float32), rng.normal(size=(B, 2)).astype(np.float32)
    P, X, T = (torch.from_numpy(a).cuda() for a in (th, x, t))
    y = rel.mlp_forward(ctx, P, X).cpu().numpy()
    g, loss = rel.mlp_backward(ctx, P, X, T)
    yr, _ = omlp.forward(th.astype(np.float64), x.astype(np.float64))
    lr, gr = omlp.backward(th.astype(np.float64), x.astype(np.float64), t.astype(np.float64))
    # FP32 sums of at most 64 terms per layer, of at most 8209 samples in partial sums of at most
    # 64: a random walk of roundings of 2^-24 over them stays under 1e-5 of the result's norm
    off = lambda a, b: np.linalg.norm(a - b) / np.linalg.norm(b)  # noqa: E731
    assert off(y, yr) < 1e-5
    assert off(g.cpu().numpy(), gr) < 1e-5
    assert abs(float(loss) - lr) < 1e-5 * lr
    ctx.close()
