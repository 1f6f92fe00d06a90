"""A capture cannot allocate: a call whose horizons would pay, captured after a warm-up of the same
sizes whose horizons did not, is captured without them and gives the eager call's map."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("closed", [True, False])
def test_captured_call_needs_no_new_buffers(closed):
    import torch
    import paper_2601_07571_amd as gm
    assert torch.cuda.is_available()
    gm.load_library()
    m = workloads.sphere_mesh(freq=16, radius=0.4, displace=0.03, seed=2)
    tri = m.I if closed else m.I[: 3 * len(m.I) // 4]
    scene = gm.Scene([(m.V, tri)])
    s = scene.build_samples(900.0, 1)
    f = workloads.shell_fixations(np.random.default_rng(3), [m], 160, dur=(0.1, 0.5))
    fix = gm.Fixations(f.eye, f.gaze, f.dur)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for _ in range(2):
            scene.accumulate(s.pos, fix, 0.5, occlusion="full", tri=s.tri, mesh=s.mesh)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            out = scene.accumulate(s.pos, fix, 5.0, occlusion="full", tri=s.tri, mesh=s.mesh)
    want = None
    for _ in range(3):
        out.density.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = out.density.clone()
        if want is None:
            other = gm.Scene([(m.V, tri)])
            want = other.accumulate(s.pos, fix, 5.0, occlusion="full", tri=s.tri, mesh=s.mesh).density
            torch.cuda.synchronize()
        assert float(want.max()) > 0 and torch.equal(got, want)
