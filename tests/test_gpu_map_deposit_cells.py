"""Merged deposits of large cells, up to one cell for the whole plane (every lane
of a wave in one group), against a map of the same rays over the same square in
cells so small that nothing is merged."""
import numpy as np
import pytest
import torch

import scenegen as sg
from gpu_common import ctx, lib, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


# (scene, rays, depth, cells per side, small cells per cell and side, merging asked for
# from so many rays in the cell under the transmitter)
@pytest.mark.parametrize("name, rays, depth, n, parts, rule", [
    ("toy", 64, 0, 1, 1600, 32.0), ("toy", 1_000, 1, 1, 1600, 32.0), ("toy", 20_001, 3, 1, 1600, 32.0),
    ("toy", 20_001, 1, 2, 800, 32.0), ("urban", 200_003, 2, 4, 200, 160.0)])
@pytest.mark.parametrize("scatter", [False, True])
def test_large_cells_are_the_sum_of_small_ones(name, rays, depth, n, parts, rule, scatter):
    m = lib()
    w = sg.toy_workload() if name == "toy" else sg.diff_workload(num_rays=1000)
    s = m.Scene.from_scenegen(ctx(), w.scene)
    if scatter:
        s.set_scattering([0.4] * len(w.scene.material_names), 5)
    tx, cell, p = w.tx[0], 400.0 / n, m.TraceParams(w.scene.freq_hz, depth, rays)
    x0, y0, h = tx.pos[0] - 210.0, tx.pos[1] - 190.0, tx.pos[2] - 1.5
    under = rays / (4 * np.pi * h * h)   # rays per square metre below the transmitter
    assert under * cell * cell >= rule > under * (cell / parts) ** 2
    big = m.coverage_map(ctx(), s, p, tx, sg.Grid(x0, y0, cell, n, n, 1.5))
    small = m.coverage_map(ctx(), s, p, tx, sg.Grid(x0, y0, cell / parts, n * parts, n * parts, 1.5))
    hits = small["hits"].long().reshape(n, parts, n, parts).sum((1, 3))
    gain = small["gain"].double().reshape(n, parts, n, parts).sum((1, 3)) / parts ** 2
    assert int(hits.sum()) > 0
    assert torch.equal(big["hits"].long(), hits)
    assert torch.equal(big["ray_bounces"], small["ray_bounces"])
    # fp32 sums of positive terms: one rounding per addition on either side
    assert ((big["gain"].double() - gain).abs() <= 2.0 ** -23 * (hits.double() + 2) * gain).all()
