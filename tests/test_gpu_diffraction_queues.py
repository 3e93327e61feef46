"""Diffracted paths where far more (receiver, wedge) pairs survive than the queues
have room for: 200 parallel ridges, all of which diffract towards every receiver
above them, against calls few enough for queues of every pair."""
import numpy as np
import pytest
import torch

import scenegen as sg
from gpu_common import ctx, lib, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


def _ridges(n):
    V, F = [], []
    for i in range(n):
        x, b = 2.0 * i - n, len(V)
        V += [(x - 0.5, -200.0, 0.0), (x, -200.0, 1.0), (x + 0.5, -200.0, 0.0),
              (x - 0.5, 200.0, 0.0), (x, 200.0, 1.0), (x + 0.5, 200.0, 0.0)]
        F += [(b, b + 1, b + 4), (b, b + 4, b + 3), (b + 1, b + 2, b + 5), (b + 1, b + 5, b + 4)]
    return np.array(V, np.float32), np.array(F, np.int32)


# pairs up to the line, where the queues hold all of them, and beyond it
@pytest.mark.parametrize("nrx, ntx", [(20_971, 1), (20_972, 1), (26_000, 2)])
def test_more_survivors_than_room(nrx, ntx):
    m = lib()
    V, F = _ridges(200)
    sc = m.Scene(ctx(), V, F, np.zeros(len(F), np.int32), [(5.0, 0.01)])
    assert sc.info()["num_wedges"] == 200
    rng = np.random.default_rng(3)
    rx = [sg.Device((float(x), float(y), float(z))) for x, y, z in
          zip(rng.uniform(-150, 150, nrx), rng.uniform(-100, 100, nrx), rng.uniform(20, 40, nrx))]
    tx = [sg.Device((7.3, 3.1, 30.0)), sg.Device((-21.7, -11.9, 55.0))][:ntx]
    big = m.compute_diffraction(ctx(), sc, 3.5e9, tx, rx, P=256)
    assert int(big["num_paths"].min()) >= 100
    for first in (0, nrx // 2, nrx - 300):
        few = m.compute_diffraction(ctx(), sc, 3.5e9, tx, rx[first:first + 300], P=256)
        for k in ("num_paths", "wedge", "a", "T", "tau", "aod", "aoa"):
            assert torch.equal(big[k][:, first:first + 300], few[k]), k
