"""The passes of the image method for every depth its kernels are sized for, and
across the bound of one queue: paths against the oracle's image method over the
same candidates, and a call of many receivers against calls of few."""
import numpy as np
import pytest
import torch

import scenegen as sg
from gpu_common import ctx, lib, oracle_params, params, requires_gpu, scene
from oracle import geom, image, sbr

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("depth", [0, 1, 2, 3, 4, 6, 8])
def test_paths_match_the_oracle_at_every_depth(depth):
    m = lib()
    w = sg.toy_workload()
    p = params(w, max_depth=depth, num_rays=20_000, max_paths_per_rx=64)
    o = m.compute_paths(ctx(), scene(w.scene), p, w.tx, w.rx)
    g = geom.Geometry(w.scene)
    r = sbr.trace(w.scene, w.tx[0], oracle_params(p), candidates=True, geo=g)
    ref = image.paths(g, w.tx[0], w.rx, r.candidates)
    num, dep = o["num_paths"][0].cpu().numpy(), o["depth"][0].cpu().numpy()
    a, faces, tau = (o[k][0].cpu().numpy() for k in ("a", "faces", "tau"))
    total = 0
    for i, paths in enumerate(ref):
        assert num[i] == len(paths)
        got = {tuple(faces[i, j, :dep[i, j]]): (complex(*a[i, j]), tau[i, j]) for j in range(num[i])}
        for q in paths:
            ga, gt = got[tuple(q.faces)]
            assert abs(ga - q.a) <= 1e-4 * abs(q.a) and abs(gt - q.tau) <= 1e-6 * q.tau
        total += len(paths)
    assert total > 0


def test_many_receivers_equal_few():
    """More (receiver, candidate) pairs than one queue holds (2^22)."""
    m = lib()
    w = sg.diff_workload(num_rays=200_000)
    pts = sg.sample_street_points(w.scene, 12_000, -240.0, 240.0, 1.5, seed=7)
    rx = [sg.Device(tuple(map(float, q))) for q in pts]
    p = params(w, max_paths_per_rx=32)
    big = m.compute_paths(ctx(), scene(w.scene), p, w.tx, rx)
    pairs = len(rx) * (m.last_candidate_count(ctx()) + 1)
    assert pairs > 2 ** 22, pairs
    for first in (0, 5_990, 11_900):
        few = m.compute_paths(ctx(), scene(w.scene), p, w.tx, rx[first:first + 100])
        for k in ("num_paths", "depth", "faces", "a", "tau", "T"):
            assert torch.equal(big[k][:, first:first + 100], few[k]), k
