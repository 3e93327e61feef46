"""The coverage gradient for every number of materials its kernel is built for
and for ray counts around its batches of 64: the derivatives against central
differences of the kernel's own fp64 sum, the sum over interleaved parts of
the lattice against the whole, and the sum against the forward map."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import scenegen as sg
from gpu_common import ctx, lib, params, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

GRID = sg.Grid(-200.0, -200.0, 4.0, 100, 100, 1.5)


def _scene(m, nm, city=False):
    s = sg.make_city(0, 6) if city else sg.diff_workload(num_rays=1000).scene
    tri = (np.asarray(s.tri_mat) + 2 * (np.arange(len(s.tri_mat)) // 2 % 2)) % nm
    mats = [(4.0, 0.0625), (6.0, 0.03125), (3.0, 0.125), (5.0, 0.25)][:nm]   # exact in float32, steps below too
    return m.Scene(ctx(), s.V, s.F, tri.astype(np.int32), mats), np.array(mats)


def _grad(m, sc, p, tx):
    tri, t = m.trace_record(ctx(), sc, p, tx)
    return m.coverage_grad(ctx(), sc, p, tx, GRID, tri, t).cpu().numpy()


def _tx(w, yaw=0.5, pitch=0.25):
    t = w.tx[0]
    return SimpleNamespace(pos=t.pos, yaw=yaw, pitch=pitch, roll=0.125, pattern=1, pol=2)


@pytest.mark.parametrize("scatter", [False, True])
@pytest.mark.parametrize("nm, rays, city", [(1, 20_001, False), (2, 4_097, False), (3, 20_001, False),
                                            (4, 20_001, False), (2, 20_001, True)])
def test_derivatives_match_differences_of_the_sum(nm, rays, city, scatter):
    """city: more triangles than the walk of the geometry stages."""
    m = lib()
    w = sg.diff_workload(num_rays=rays)
    p = params(w)
    sc, mats = _scene(m, nm, city)
    if scatter:
        sc.set_scattering([0.5] * nm, 3)
    out = _grad(m, sc, p, _tx(w))
    assert out[0] > 0
    fwd = float(m.coverage_map(ctx(), sc, p, _tx(w), GRID)["gain"].double().sum())
    assert abs(out[0] - fwd) < 1e-4 * fwd
    got, ref, h = out[1:], [], 2.0 ** -10
    for i in range(nm):
        for c, step in ((0, h), (1, 2.0 ** -13)):
            v = []
            for sgn in (1, -1):
                x = mats.copy()
                x[i, c] += sgn * step
                with sc.materials_set_to(x):
                    v.append(_grad(m, sc, p, _tx(w))[0])
            ref.append((v[0] - v[1]) / (2 * step))
    for k in range(2):
        d = [_grad(m, sc, p, _tx(w, 0.5 + (k == 0) * e, 0.25 + (k == 1) * e))[0] for e in (h, -h)]
        ref.append((d[0] - d[1]) / (2 * h))
    ref = np.array(ref)
    # truncation of the differences: h^2/6 times third derivatives
    scale = np.repeat([np.abs(ref[0:2 * nm:2]).max(), np.abs(ref[1:2 * nm:2]).max()], nm).reshape(2, nm).T.reshape(-1)
    scale = np.concatenate([scale, [np.abs(ref[2 * nm:]).max()] * 2])
    print(got, ref, flush=True)
    assert (np.abs(got - ref) <= 1e-3 * scale).all()


@pytest.mark.parametrize("rays", [1, 63, 65, 257, 10_007, 200_003, 2 ** 24 + 1001])
def test_parts_of_the_lattice_add_up(rays):
    m = lib()
    w = sg.diff_workload(num_rays=rays)
    p = params(w)
    sc, _ = _scene(m, 2)
    whole = _grad(m, sc, p, _tx(w))
    parts = 0.0
    for b in range(min(3, rays)):
        q = params(w)
        q.ray_begin, q.ray_stride = b, 3
        parts = parts + _grad(m, sc, q, _tx(w))
    assert np.isfinite(whole).all()
    # the same fp64 terms in another order; rounding of at most 1e-16 per term of magnitude below the sum of magnitudes
    assert np.allclose(parts, whole, rtol=1e-9, atol=1e-12 * np.abs(whole).max())
