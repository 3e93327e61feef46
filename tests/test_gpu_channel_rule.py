"""Channel responses on both sides of the rule that takes tiles (the outputs of
all links together), with rows and subcarriers one off a tile, against the phase
formula in float64 with NumPy.

Tolerance: a response is rounded to float32 once (2^-24 of the sum of |a|), and
every phase carries at most 2^14 cycles in float64 (2 pi 2^14 2^-53 = 1.2e-11
rad)."""
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


# (links, time steps, rx elements, tx elements, subcarriers); outputs from just
# below to just above 2^18, 3 2^17 and 5 2^17, and few subcarriers
@pytest.mark.parametrize("n,T,nr,nt,K", [
    (1, 4096, 1, 1, 1), (2, 3, 1, 171, 3), (3, 1, 4, 13653, 4), (3, 7, 3, 2081, 5), (3, 1, 1, 43691, 5),
    (80, 2, 1, 257, 16), (79, 1, 1, 513, 16), (5, 1, 3, 257, 17), (91, 1, 1, 257, 17), (24, 1, 2, 257, 32),
    (62, 1, 1, 129, 33), (61, 1, 1, 129, 33), (33, 1, 1, 129, 64), (63, 1, 1, 65, 65), (31, 1, 1, 65, 129),
    (32, 1, 1, 65, 129), (255, 1, 1, 8, 129)])
def test_responses_around_the_rule(n, T, nr, nt, K):
    m = lib()
    rng = np.random.default_rng(n * 1000 + K)
    P = 5
    depth = np.where(rng.random((1, n, P)) < 0.7, rng.integers(0, 4, (1, n, P)), -1).astype(np.int32)
    tau = rng.uniform(0.0, 2e-6, (1, n, P)).astype(np.float32)
    a = rng.normal(size=(1, n, P, 2)).astype(np.float32)
    aod, aoa = (np.stack([rng.uniform(0, np.pi, (1, n, P)), rng.uniform(-np.pi, np.pi, (1, n, P))],
                         -1).astype(np.float32) for _ in range(2))
    te, re = rng.normal(0.0, 0.1, (nt, 3)), rng.normal(0.0, 0.1, (nr, 3))
    vr = rng.normal(0.0, 5.0, (n, 3))
    dev = ctx().torch_device
    paths = {k: torch.tensor(v, device=dev) for k, v in dict(a=a, tau=tau, aod=aod, aoa=aoa, depth=depth).items()}
    H = m.paths_cfr(ctx(), paths, FREQ, num_subcarriers=K, tx_el=te, rx_el=re, v_tx=np.zeros((1, 3)), v_rx=vr,
                    num_time_steps=T, fs=14e3).cpu().numpy()
    lam = C0 / FREQ
    fk = (np.arange(K) - K // 2) * 30e3
    for r in range(n):
        ok = depth[0, r] >= 0
        kt, kr = _unit(aod[0, r, ok].astype(np.float64)), _unit(aoa[0, r, ok].astype(np.float64))
        fd = kr @ vr[r] / lam
        row = ((np.arange(T) / 14e3)[:, None, None, None] * fd + (re @ kr.T / lam)[None, :, None]
               + (te @ kt.T / lam)[None, None])
        sub = -(FREQ + fk)[None] * tau[0, r, ok].astype(np.float64)[:, None]
        c = a[0, r, ok, 0] + 1j * a[0, r, ok, 1].astype(np.float64)
        want = (np.exp(2j * np.pi * (row - np.floor(row))) * c).reshape(T * nr * nt, ok.sum()) @ np.exp(
            2j * np.pi * (sub - np.floor(sub)))
        tol = np.abs(c).sum() * (2.0 ** -23 + 2.4e-11) + 1e-30
        assert np.abs(H[0, r].reshape(want.shape) - want).max() <= tol
