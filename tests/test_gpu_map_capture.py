"""An incremental map captured into a graph (reset, add, read) and replayed: with its horizons
complete, and with them still being computed on another stream, for which a replay could not
wait.  Every replay gives the eager map."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _map(gm, closed, F):
    m = workloads.sphere_mesh(freq=12, radius=0.4, displace=0.03, seed=2)
    tri = m.I if closed else m.I[: 3 * len(m.I) // 4]
    scene = gm.Scene([(m.V, tri)])
    s = scene.build_samples(900.0, 1)
    f = workloads.shell_fixations(np.random.default_rng(3), [m], F, dur=(0.1, 0.5))
    fix = gm.Fixations(f.eye, f.gaze, f.dur)
    return gm.DensityMap(scene, s.pos, 4.0, occlusion="full", tri=s.tri, mesh=s.mesh), fix


@pytest.mark.parametrize("closed", [True, False])
@pytest.mark.parametrize("F", [400, 70000])  # gathered blocks, and a block that runs alone
def test_captured_reset_add_read(closed, F):
    import torch
    import paper_2601_07571_amd as gm
    assert torch.cuda.is_available()
    dm, fix = _map(gm, closed, F)
    want = dm.add(fix).read().density.clone()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        dm.reset()
        dm.add(fix).read()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            dm.reset()
            out = dm.add(fix).read()
    for _ in range(3):
        out.density.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert float(want.max()) > 0 and torch.equal(out.density, want)
        with torch.cuda.stream(stream):  # eager work on the same map between the replays
            dm.reset()
            assert torch.equal(dm.add(fix).read().density, want)
        torch.cuda.synchronize()


@pytest.mark.parametrize("closed", [True, False])
def test_captured_while_the_horizons_are_computed(closed):
    import torch
    import paper_2601_07571_amd as gm
    dm, fix = _map(gm, closed, 400)
    want = dm.add(fix).read().density.clone()   # its own horizons, and the records' buffer
    dm, fix = _map(gm, closed, 400)
    dm.add(fix.subset(0, 20)).read()            # too few fixations for horizons
    dm.reset()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        for _ in range(40):
            busy = torch.mm(busy, busy).clamp_(-1, 1)
        first = dm.add(fix).read()              # the horizons, behind the products
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(b):
        graph.capture_begin()
        dm.reset()
        out = dm.add(fix).read()
        graph.capture_end()
    torch.cuda.synchronize()
    assert float(want.max()) > 0 and torch.equal(first.density, want)
    for _ in range(3):
        out.density.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.density, want)
        dm.reset()
        assert torch.equal(dm.add(fix).read().density, want)
        torch.cuda.synchronize()
