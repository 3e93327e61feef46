"""The surrogate's gradient at row counts whose groups of 32 do not divide evenly
over the splits of the weight products, below the batch the scratch is made for:
every weight and bias block against the float64 oracle."""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp

from gpu_common import requires_gpu
from test_gpu_mlp import _mlp, _oracle_inputs

pytestmark = [pytest.mark.gpu, requires_gpu]


# groups of 32 rows / splits: 4/1, 12/3, 20/5, 36/9, 132/32, 548/32
@pytest.mark.parametrize("rows", [128, 384, 640, 1152, 4224, 17536])
def test_gradient_blocks_match_oracle(rows):
    m = _mlp(batch=20480, seed=5)
    rng = np.random.default_rng(rows)
    v = rng.uniform(-1, 1, size=(rows, 5)).astype(np.float32)
    t = rng.normal(scale=2.0, size=rows).astype(np.float32)
    msk = (rng.random(rows) < 0.7).astype(np.float32)
    full = rng.uniform(-1, 1, size=(20480, 5)).astype(np.float32)
    dev = "cuda"
    m.grad(torch.tensor(full, device=dev), torch.ones(20480, device=dev), torch.ones(20480, device=dev))  # fills it
    g, loss = m.grad(torch.tensor(v, device=dev), torch.tensor(t, device=dev), torch.tensor(msk, device=dev))
    g = g.cpu().double().numpy()
    _, theta_q, ffn, feats = _oracle_inputs(m, v)
    yo, cache = omlp.forward(theta_q, v, ffn, feats=feats)
    go = omlp.backward(theta_q, cache, yo, t.astype(np.float64), msk.astype(np.float64))
    lo = omlp.loss(yo, t, msk)
    assert abs(float(loss) - lo) <= 2e-2 * lo
    k = 0
    for W, b in omlp.layer_shapes():
        for shape in (W, b):
            n = int(np.prod(shape))
            blk, ref = g[k:k + n], go[k:k + n]
            # bf16 operands of every product: the bound of the gradient's parity test
            assert np.max(np.abs(blk - ref)) <= 2e-2 * np.max(np.abs(ref)) + 1e-12, (k, shape)
            k += n
