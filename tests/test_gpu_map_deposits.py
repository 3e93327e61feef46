"""Coverage maps that merge a wave's deposits per cell, and launches sized to
few rays: hit counts and gains against maps of the same rays summed from parts
of the lattice small enough not to merge, on both sides of the rule."""
import numpy as np
import pytest
import torch

import scenegen as sg
from gpu_common import ctx, lib, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


# (scene, rays, depth, cell): rays around a block of 512 and below a wave; the
# cell under the transmitter gets far fewer, about as many, and far more rays
# than the rule asks for, up to a grid of one cell (all lanes of a wave)
@pytest.mark.parametrize("name, rays, depth, cell, n", [
    ("toy", 1, 1, 1.0, 200), ("toy", 511, 5, 1.0, 200), ("toy", 513, 0, 5.0, 40), ("toy", 29_000, 1, 1.0, 200),
    ("toy", 300_001, 2, 1.0, 201), ("toy", 200_000, 3, 400.0, 1), ("urban", 100_003, 3, 2.0, 200),
    ("urban", 2_000_000, 3, 4.0, 101)])
@pytest.mark.parametrize("scatter", [False, True])
def test_map_is_the_sum_of_its_parts(name, rays, depth, cell, n, scatter):
    m = lib()
    w = sg.toy_workload() if name == "toy" else sg.diff_workload(num_rays=1000)
    s = m.Scene.from_scenegen(ctx(), w.scene)
    if scatter:
        s.set_scattering([0.4] * len(w.scene.material_names), 5)
    tx = w.tx[0]
    g = sg.Grid(tx.pos[0] - n * cell / 2, tx.pos[1] - n * cell / 2, cell, n, n, 1.5)
    p = m.TraceParams(w.scene.freq_hz, depth, rays)
    whole = m.coverage_map(ctx(), s, p, tx, g)
    # a part's rays under the transmitter stay below the rule's 32 (14 triangles) or 160
    h = tx.pos[2] - 1.5
    under = rays * cell * cell / (4 * np.pi * h * h)
    parts = int(np.clip(np.ceil(under / (20.0 if name == "toy" else 120.0)), 1, min(rays, 60)))
    gain = torch.zeros((n, n), dtype=torch.float64, device=ctx().torch_device)
    hits = torch.zeros((n, n), dtype=torch.int64, device=ctx().torch_device)
    bounces = 0
    for b in range(parts):
        q = m.TraceParams(w.scene.freq_hz, depth, rays, ray_begin=b, ray_stride=parts)
        o = m.coverage_map(ctx(), s, q, tx, g)
        gain += o["gain"].double()
        hits += o["hits"]
        bounces = bounces + o["ray_bounces"]
    assert torch.equal(whole["hits"].long(), hits)
    assert torch.equal(whole["ray_bounces"], bounces)
    # fp32 sums of positive terms in another order: one rounding per addition
    bound = 2.0 ** -23 * (hits.double() + 2) * gain
    assert ((whole["gain"].double() - gain).abs() <= bound).all()
