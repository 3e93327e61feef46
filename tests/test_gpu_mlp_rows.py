"""The surrogate's gradient kernel (64 rows from input to weights' operands) at
the sizes it is launched for: every multiple of 1024 rows that fills its grid
unevenly, with masked rows, against the weighted sum over smaller batches."""
import numpy as np
import pytest
import torch

from gpu_common import ctx, lib, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


def _rows(n, seed):
    g = np.random.default_rng(seed)
    v = np.concatenate([g.uniform(-200, 200, (n, 2)), g.uniform(10, 60, (n, 1)), g.uniform(-200, 200, (n, 2))], 1)
    t = g.normal(-90.0, 15.0, n)
    mask = (g.random(n) < 0.9).astype(np.float32)
    return [torch.tensor(x.astype(np.float32), device=ctx().torch_device) for x in (v, t, mask)]


def _mlp(rows):
    lib()
    from paper_2303_11103_amd import surrogate
    c, h = np.array([0.0, 0.0, 35.0, 0.0, 0.0]), np.array([200.0, 200.0, 25.0, 200.0, 200.0])
    return surrogate.MLP(ctx(), batch=rows, ff_scale=1.0, ff_scale_cell=4.0, seed=3, center=c, half=h,
                         prior=(3.5e9, 1.5), ff_rows_tx=8, ff_rows_rel=40, ff_scale_rel=32.0)


@pytest.mark.parametrize("rows", [2048, 3072, 17 * 1024, 33 * 1024, 64 * 1024])
def test_gradient_is_the_mean_over_parts(rows):
    v, t, mask = _rows(rows, rows)
    g, loss = _mlp(rows).grad(v, t, mask)
    small = _mlp(1024)
    gs, ls, n = torch.zeros_like(g, dtype=torch.float64), 0.0, float(mask.sum())
    for b in range(0, rows, 1024):
        c = slice(b, b + 1024)
        gp, lp = small.grad(v[c].contiguous(), t[c].contiguous(), mask[c].contiguous())
        share = float(mask[c].sum()) / n
        gs += share * gp.double()
        ls += share * float(lp)
    assert torch.isfinite(g).all()
    # the row sums and products of both sides round in bf16 the same way up to
    # the factor 2 / (rows in use) of the output error, which bf16 rounds to
    # 2^-9 relative per operand: independent over rows, the sums agree far closer
    rel = float((g.double() - gs).norm() / gs.norm())
    print("rows %d rel %.2e loss %.6f %.6f" % (rows, rel, float(loss), ls), flush=True)
    assert rel < 2.0 ** -8
    assert abs(float(loss) - ls) < 1e-5 * ls


def test_masked_rows_do_not_count():
    v, t, mask = _rows(2048, 1)
    mask[1024:] = 0.0
    g, loss = _mlp(2048).grad(v, t, mask)
    gp, lp = _mlp(1024).grad(v[:1024].contiguous(), t[:1024].contiguous(), mask[:1024].contiguous())
    assert float((g - gp).norm()) <= 1e-5 * float(gp.norm())
    assert abs(float(loss) - float(lp)) <= 1e-6 * float(lp)
    g, loss = _mlp(2048).grad(v, t, torch.zeros_like(mask))
    assert float(g.abs().max()) == 0.0 and float(loss) == 0.0
