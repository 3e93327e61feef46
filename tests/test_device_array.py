"""Lists of devices packed for the C ABI: every accepted form gives the bytes
of the structure filled field by field, and what that refuses stays refused."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import scenegen as sg
from paper_2303_11103_amd import rt


def _ns(**kw):
    return SimpleNamespace(**{**dict(pos=(1.0, 2.0, 3.0), yaw=0.1, pitch=-0.2, roll=0.3, pattern=1, pol=2), **kw})


def _no_pol():
    d = _ns()
    del d.pol
    return d


@pytest.mark.parametrize("odd", [
    None, _ns(pos=np.array([0.1, 1e-45, -0.0], np.float32)), _ns(pos=np.arange(5.0)), _ns(pos={0: 1.0, 1: 2.0, 2: 3.0}),
    _ns(yaw=np.float64(0.1), pattern=np.int64(2)), _ns(pattern=1.0, pol=True), _ns(yaw="0.5"), _ns(yaw=1e39),
    _ns(pitch=float("nan"), roll=float("inf")), _ns(pattern=2 ** 31), _no_pol()])
def test_device_array_bytes(odd):
    devs = [sg.Device((0.1 * i, -i, 1.5), 0.01 * i, pattern=i % 3, pol=i % 4) for i in range(5)]
    if odd is not None:
        devs.insert(3, odd)
    got = rt.device_array(devs)
    assert len(got) == len(devs)
    assert bytes(got) == b"".join(bytes(rt.device_struct(d)) for d in devs)


@pytest.mark.parametrize("odd, err", [(_ns(pos=(1.0, 2.0)), IndexError), (_ns(pos={1.0, 2.0, 3.0}), TypeError),
                                      (_ns(yaw=None), TypeError), (SimpleNamespace(pos=(0, 0, 0)), AttributeError)])
def test_device_array_refuses(odd, err):
    for f in (rt.device_array, lambda v: [rt.device_struct(d) for d in v]):
        with pytest.raises(err):
            f([_ns(), odd])
