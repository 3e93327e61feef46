"""Coverage gradients recorded into graphs, and of one context on two streams:
a recorded call keeps nothing of the context's scratch (which later calls grow
and reuse), and calls on different streams do not read each other's queue."""
import numpy as np
import pytest
import torch

import scenegen as sg
from gpu_common import lib, params, requires_gpu
from test_gpu_coverage_grad_kernel import GRID, _tx

pytestmark = [pytest.mark.gpu, requires_gpu]


def _case(m, c, rays, nm, city=False, scatter=False):
    s = sg.make_city(0, 6) if city else sg.diff_workload(num_rays=1000).scene
    tri = (np.asarray(s.tri_mat) + 2 * (np.arange(len(s.tri_mat)) // 2 % 2)) % nm
    scene = m.Scene(c, s.V, s.F, tri.astype(np.int32), [(4.0, 0.0625), (6.0, 0.03125), (3.0, 0.125), (5.0, 0.25)][:nm])
    if scatter:
        scene.set_scattering([0.5] * nm, 3)
    w = sg.diff_workload(num_rays=rays)
    p, tx = params(w), _tx(w)
    return scene, p, tx, m.trace_record(c, scene, p, tx)


def _close(got, want):
    # the same fp64 terms in another order; rounding of at most 1e-16 per term of magnitude below the sum of magnitudes
    return np.allclose(got, want, rtol=1e-9, atol=1e-12 * np.abs(want).max())


# ray counts around a wave and a block, and several per lane; every number of
# materials; more triangles than the queued walk stages
@pytest.mark.parametrize("rays, nm, city, scatter", [
    (1, 1, False, False), (63, 2, False, True), (257, 3, False, False), (10_007, 4, False, True),
    (200_003, 1, False, False), (400_001, 2, True, True), (1_500_001, 2, False, False)])
def test_recorded_gradient_equals_the_eager_one_after_larger_calls(rays, nm, city, scatter):
    m = lib()
    c = m.Context(0)
    scene, p, tx, (tri, t) = _case(m, c, rays, nm, city, scatter)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):   # the context's first gradient
        out = m.coverage_grad(c, scene, p, tx, GRID, tri, t)
    want = m.coverage_grad(c, scene, p, tx, GRID, tri, t).cpu().numpy()
    scene2, p2, tx2, (tri2, t2) = _case(m, c, 2 * rays + 70_000, 2)
    large = None
    for _ in range(3):
        got2 = m.coverage_grad(c, scene2, p2, tx2, GRID, tri2, t2)   # grows and fills the queue
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert _close(out.cpu().numpy(), want)
        large = got2.cpu().numpy() if large is None else large
        assert _close(got2.cpu().numpy(), large)


def test_gradients_on_two_streams_do_not_mix():
    m = lib()
    c = m.Context(0)
    cases = [_case(m, c, rays, nm) for rays, nm in ((1_700_001, 2), (600_001, 3))]
    want = [m.coverage_grad(c, s, p, tx, GRID, *rec).cpu().numpy() for s, p, tx, rec in cases]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = [[], []]
    for _ in range(20):
        for k, (s, p, tx, rec) in enumerate(cases):
            with torch.cuda.stream(streams[k]):
                got[k].append(m.coverage_grad(c, s, p, tx, GRID, *rec))
    torch.cuda.synchronize()
    for k in range(2):
        for g in got[k]:
            assert _close(g.cpu().numpy(), want[k])
