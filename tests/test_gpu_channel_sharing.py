"""The adjoint's partial sums: two streams of one context do not share them, and
more tiles than they have room for go through several launches."""
import numpy as np
import pytest
import torch

from gpu_common import lib, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


def _paths(c, rng, n, P, valid):
    depth = np.where(rng.random((1, n, P)) < valid, rng.integers(0, 4, (1, n, P)), -1).astype(np.int32)
    d = dict(a=rng.normal(size=(1, n, P, 2)), tau=rng.uniform(0.0, 2e-6, (1, n, P)),
             aod=rng.uniform(0.0, np.pi, (1, n, P, 2)), aoa=rng.uniform(0.0, np.pi, (1, n, P, 2)))
    d = {k: torch.tensor(v.astype(np.float32), device=c.torch_device) for k, v in d.items()}
    return dict(d, depth=torch.tensor(depth, device=c.torch_device))


def _responses(c, rng, shape):
    g = torch.tensor(rng.normal(size=shape + (2,)).astype(np.float32), device=c.torch_device)
    return torch.view_as_complex(g)


def test_adjoints_on_two_streams_do_not_mix():
    m = lib()
    c = m.Context(0)
    rng = np.random.default_rng(5)
    kw = dict(num_subcarriers=130, num_time_steps=64, fs=14e3, tx_el=rng.normal(size=(4, 3)) * 0.1)
    paths = _paths(c, rng, 4, 64, 0.7)   # row ranges times two subcarrier tiles: partial sums
    G = [_responses(c, rng, (1, 4, 64, 1, 4, 130)) for _ in range(2)]
    want = [m.paths_cfr_adjoint(c, paths, g, 3.5e9, **kw) for g in G]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [[], []]
    for _ in range(50):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                got[k].append(m.paths_cfr_adjoint(c, paths, G[k], 3.5e9, **kw))
    torch.cuda.synchronize()
    for k in range(2):
        for g in got[k]:   # partial sums are added in a fixed order
            assert torch.equal(g, want[k])


def test_more_tiles_than_partial_sums_have_room_for():
    """Two parts of 1 KiB per tile of 64 slots, 33 tiles per link: 64 MiB end
    inside link 992."""
    m = lib()
    c = m.Context(0)
    rng = np.random.default_rng(6)
    n, P = 1010, 2100
    kw = dict(num_subcarriers=130, num_time_steps=8, fs=14e3)
    paths = _paths(c, rng, n, P, 0.02)
    G = _responses(c, rng, (1, n, 8, 1, 1, 130))
    g = m.paths_cfr_adjoint(c, paths, G, 3.5e9, **kw)
    assert bool((g[paths["depth"] < 0] == 0.0).all())
    for r in (0, 991, 992, 993, n - 1):
        one = m.paths_cfr_adjoint(c, {k: v[:, r:r + 1].contiguous() for k, v in paths.items()},
                                  G[:, r:r + 1].contiguous(), 3.5e9, **kw)
        assert float(one.abs().max()) > 0.0
        assert torch.equal(g[:, r:r + 1], one), r
