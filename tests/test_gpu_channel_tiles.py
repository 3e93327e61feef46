"""Channel responses and their adjoint at the edges of the kernels' tiles
(rows = time steps x receive x transmit elements, subcarriers, path slots),
against the phase formula summed in float64 with NumPy.

Tolerances: a response is rounded to float32 once (2^-24 of the sum of |a|) and
every phase carries at most 2^14 cycles in float64 (2 pi 2^14 2^-53 = 1.2e-11
rad), as does every adjoint entry per unit of the sum of |G|."""
import numpy as np
import pytest
import torch

from gpu_common import ctx, lib, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]
C0 = 299792458.0
FREQ = 3.5e9


def _unit(a):
    return np.stack([np.sin(a[..., 0]) * np.cos(a[..., 1]), np.sin(a[..., 0]) * np.sin(a[..., 1]),
                     np.cos(a[..., 0])], -1)


# (nrx, P, time steps, rx elements, tx elements, K): below and at the rule that
# takes tiles (8 rows and 1024 outputs per link), one off every tile size
@pytest.mark.parametrize("nrx,P,T,nr,nt,K", [
    (3, 1, 1, 1, 1, 1), (2, 257, 1, 1, 1, 130), (2, 64, 7, 1, 1, 147), (2, 64, 2, 2, 2, 128), (2, 65, 1, 3, 3, 127),
    (1, 100, 2, 5, 13, 129), (2, 63, 3, 1, 43, 64), (2, 9, 3, 2, 22, 33), (1, 130, 1, 1, 257, 17), (2, 5, 3, 1, 171, 16),
    (1, 17, 1, 2, 513, 1), (1, 300, 4, 4, 16, 65)])
def test_responses_and_adjoint_at_tile_edges(nrx, P, T, nr, nt, K):
    m = lib()
    rng = np.random.default_rng(P * 1000 + K)
    depth = np.where(rng.random((2, nrx, P)) < 0.6, rng.integers(0, 4, (2, nrx, P)), -1).astype(np.int32)
    depth[0, 0] = -1 if P > 1 else 0       # a link without paths
    tau = rng.uniform(0.0, 2e-6, (2, nrx, P)).astype(np.float32)
    a = rng.normal(size=(2, nrx, P, 2)).astype(np.float32)
    aod, aoa = (np.stack([rng.uniform(0, np.pi, (2, nrx, P)), rng.uniform(-np.pi, np.pi, (2, nrx, P))],
                         -1).astype(np.float32) for _ in range(2))
    te, re = rng.normal(0.0, 0.1, (nt, 3)), rng.normal(0.0, 0.1, (nr, 3))
    vt, vr = rng.normal(0.0, 5.0, (2, 3)), rng.normal(0.0, 5.0, (nrx, 3))
    G = (rng.normal(size=(2, nrx, T, nr, nt, K)) + 1j * rng.normal(size=(2, nrx, T, nr, nt, K))).astype(np.complex64)
    lam = C0 / FREQ
    kt, kr = _unit(aod.astype(np.float64)), _unit(aoa.astype(np.float64))
    fk = (np.arange(K) - K // 2) * 30e3
    fd = ((kt * vt[:, None, None]).sum(-1) + (kr * vr[None, :, None]).sum(-1)) / lam
    want = np.zeros(G.shape, np.complex128)
    adj = np.zeros((2, nrx, P), np.complex128)
    for i in range(2):
        for r in range(nrx):
            for p in np.nonzero(depth[i, r] >= 0)[0]:
                cyc = ((np.arange(T) / 14e3 * fd[i, r, p])[:, None, None, None]
                       + (re @ kr[i, r, p] / lam)[:, None, None] + (te @ kt[i, r, p] / lam)[:, None]
                       - (FREQ + fk) * float(tau[i, r, p]))
                e = np.exp(2j * np.pi * (cyc - np.floor(cyc)))
                want[i, r] += (a[i, r, p, 0] + 1j * float(a[i, r, p, 1])) * e
                adj[i, r, p] = (np.conj(G[i, r].astype(np.complex128)) * e).sum()
    dev = ctx().torch_device
    paths = {k: torch.tensor(v, device=dev) for k, v in
             dict(a=a, tau=tau, aod=aod, aoa=aoa, depth=depth).items()}
    kw = dict(num_subcarriers=K, tx_el=te, rx_el=re, v_tx=vt, v_rx=vr, num_time_steps=T, fs=14e3)
    H = m.paths_cfr(ctx(), paths, FREQ, **kw).cpu().numpy()
    g = m.paths_cfr_adjoint(ctx(), paths, torch.tensor(G, device=dev), FREQ, **kw).cpu().numpy()
    amp = np.abs(a[..., 0] + 1j * a[..., 1]) * (depth >= 0)
    tol = (amp.sum(-1) * (2.0 ** -23 + 2.4e-11))[:, :, None, None, None, None] + 1e-30
    assert np.all(np.abs(H - want) <= tol)
    gtol = 2.4e-11 * np.abs(G).reshape(2, nrx, -1).sum(-1)[:, :, None]
    assert np.all(np.abs(g[..., 0] + 1j * g[..., 1] - adj) <= gtol)
    assert np.all(g[depth < 0] == 0.0)
