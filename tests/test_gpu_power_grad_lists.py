"""Received-power gradients of full path lists (every lane of a block busy,
slots across blocks and receivers, many materials): equal to the sum over calls
of one slot each."""
import numpy as np
import pytest
import torch

import scenegen as sg
from gpu_common import ctx, lib, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


def _sequences(rng, scene, face_of, n, depth):
    """Random face sequences without two reflections in a row off one plane."""
    v = np.asarray(scene.V, np.float64)[np.asarray(scene.F)]
    normal = np.cross(v[:, 1] - v[:, 0], v[:, 2] - v[:, 0])
    normal /= np.linalg.norm(normal, axis=1)[:, None]
    normal *= np.sign(normal[np.arange(len(normal)), np.abs(normal).argmax(1)])[:, None]
    plane = np.round(np.concatenate([normal, (normal * v[:, 0]).sum(1)[:, None]], 1), 3)
    out = np.zeros((n, depth), np.int32)
    for q in range(n):
        last = None
        for k in range(depth):
            t = rng.integers(len(plane))
            while last is not None and (plane[t] == last).all():
                t = rng.integers(len(plane))
            out[q, k], last = face_of[t], plane[t]
    return out


# slots around a block of 16 (8 lanes each), materials up to the largest table
@pytest.mark.parametrize("nrx, P, depth, nm", [(1, 1, 0, 1), (1, 15, 1, 2), (1, 17, 3, 32), (3, 11, 3, 7), (2, 33, 8, 32)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_full_lists_are_the_sum_of_their_slots(nrx, P, depth, nm, adjoint):
    m = lib()
    w = sg.diff_workload(num_rays=1000)
    rng = np.random.default_rng(100 * P + depth)
    tri = rng.integers(0, nm, len(w.scene.tri_mat)).astype(np.int32)
    mats = [(2.0 + 0.25 * i, 0.01 * (i + 1)) for i in range(nm - 1)] + [(3.0, np.inf)]   # the last one conducts
    sc = m.Scene(ctx(), w.scene.V, w.scene.F, tri, mats)
    fd = max(depth, 1)
    dep = rng.integers(0, depth + 1, (nrx, P)).astype(np.int32)
    dep[0, 0] = depth
    faces = _sequences(rng, w.scene, sc.face_ids(), nrx * P, fd).reshape(nrx, P, fd)
    up = rng.uniform(0.5, 2.0, nrx)
    adj = rng.normal(size=(nrx, P, 2))
    rx = [sg.Device((float(x), float(y), 1.5)) for x, y in rng.uniform(-200, 200, (nrx, 2))]
    tx = sg.Device(w.tx[0].pos, 0.3, 0.2, 0.1, 1, 2)
    p = m.TraceParams(w.scene.freq_hz, depth, 1000, max_paths_per_rx=P)
    dev = ctx().torch_device

    def grad(r, q):
        d, f = torch.tensor(dep[r, q], device=dev), torch.tensor(faces[r, q], device=dev)
        if adjoint:
            return m.paths_coef_grad(ctx(), sc, p, tx, rx[r], d, f, torch.tensor(adj[r, q], device=dev))
        return m.paths_power_grad(ctx(), sc, p, tx, rx[r], d, f, torch.tensor(up[r], device=dev))

    whole = grad(slice(None), slice(None)).cpu().numpy()
    one = np.array([grad(slice(r, r + 1), slice(q, q + 1)).cpu().numpy() for r in range(nrx) for q in range(P)])
    assert np.isfinite(whole).all() and np.abs(whole[2 * nm:]).max() > 0
    # the same fp64 terms in another order: one rounding per addition of the sum of magnitudes
    assert (np.abs(whole - one.sum(0)) <= (nrx * P + 2) * 2.0 ** -52 * np.abs(one).sum(0)).all()
