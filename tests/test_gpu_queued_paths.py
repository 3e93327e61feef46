"""Diffracted and scattered paths through their queues: calls of many receivers
against calls of one (queues of another size, tiles of another remainder)."""
import numpy as np
import pytest
import torch

import scenegen as sg
from gpu_common import ctx, lib, requires_gpu, scene

pytestmark = [pytest.mark.gpu, requires_gpu]


def _rx(s, n):
    pts = sg.sample_street_points(s, n, -240.0, 240.0, 1.5, seed=9)
    z = [1.5, 30.0, 70.0]
    return [sg.Device((float(q[0]), float(q[1]), z[i % 3])) for i, q in enumerate(pts)]


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130])
def test_diffracted_paths_of_many_receivers_equal_those_of_one(n):
    m = lib()
    w = sg.diff_workload(num_rays=1000)
    rx = _rx(w.scene, n)
    big = m.compute_diffraction(ctx(), scene(w.scene), w.scene.freq_hz, w.tx, rx, P=256)
    assert int(big["num_paths"].sum()) > 0
    for i in sorted({0, n // 2, n - 1}):
        one = m.compute_diffraction(ctx(), scene(w.scene), w.scene.freq_hz, w.tx, [rx[i]], P=256)
        for k in ("num_paths", "wedge", "a", "T", "tau", "aod", "aoa"):
            assert torch.equal(big[k][:, i], one[k][:, 0]), k


@pytest.mark.parametrize("n, rays, depth", [(1, 1, 1), (3, 1_000, 0), (5, 4_097, 1), (17, 20_001, 3)])
def test_scattered_paths_of_many_receivers_equal_those_of_one(n, rays, depth):
    m = lib()
    w = sg.diff_workload(num_rays=1000)
    s = m.Scene.from_scenegen(ctx(), w.scene)
    s.set_scattering([0.6, 0.35][:len(w.scene.material_names)], 11)
    p = m.TraceParams(w.scene.freq_hz, depth, rays)
    rx = _rx(w.scene, n)
    slots = max(64, rays * max(depth, 1))
    big = m.compute_scattering(ctx(), s, p, w.tx, rx, P=slots)
    for i in sorted({0, n // 2, n - 1}):
        one = m.compute_scattering(ctx(), s, p, w.tx, [rx[i]], P=slots)
        for k in ("num_paths", "depth", "ray", "faces", "a", "T", "tau", "aod", "aoa"):
            assert torch.equal(big[k][:, i], one[k][:, 0]), k
    got = big["num_paths"][0].cpu().numpy()
    dep, ray = big["depth"][0].cpu().numpy(), big["ray"][0].cpu().numpy()
    for i in range(n):   # ascending (ray, depth), nothing behind them
        key = ray[i, :got[i]] * (depth + 1) + dep[i, :got[i]]
        assert (np.diff(key) > 0).all() and (dep[i, got[i]:] < 0).all()
    if rays > 1_000:
        assert got.sum() > 0
