"""Device memory that the horizons of an open scene's points take: 16 bytes a point for the
normals and 4 for the horizon, and no back-face lists, which a scene without a closed mesh
never writes."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def test_open_scene_holds_no_backface_lists():
    import torch
    import paper_2601_07571_amd as gm
    m = workloads.heightfield_mesh(fine=(64, 128), coarse=(32, 64))
    scene = gm.Scene([(m.V, m.I)])
    assert not scene.mesh_closed().any()
    s = scene.build_samples(2.5e5, 1)
    n, F = int(s.pos.shape[0]), 1000
    f = workloads.shell_fixations(np.random.default_rng(2), [m], F, dur=(0.1, 0.5))
    fix = gm.Fixations(f.eye, f.gaze, f.dur)
    out = scene.accumulate(s.pos, fix, 0.2, tri=s.tri, mesh=s.mesh)  # F sigma^2 = 0.01: no horizons
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    scene.accumulate(s.pos, fix, 2.0, tri=s.tri, mesh=s.mesh, out=out)  # 1.2: horizons
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    assert 18 * n <= used <= 20 * n + 4 * 2 ** 21, (used, n)  # two buffers, in pieces of 2 MB
