"""Mesh ids outside the scene: a point with such an id has no own mesh.  Full occlusion does not
ask for it, self occlusion finds no occluder; horizons and the pair check are in use (F sigma^2
= 0.24), on an open scene and on one with a closed mesh."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("closed", [False, True])
@pytest.mark.parametrize("bad", [1, 7, 1 << 20, 2147483647, -1, -2147483648])
def test_mesh_ids_outside_the_scene(closed, bad):
    import torch
    import paper_2601_07571_amd as gm
    m = workloads.sphere_mesh(freq=8, radius=0.4, displace=0.05, seed=3)
    scene = gm.Scene([(m.V, m.I if closed else m.I[: 3 * len(m.I) // 4])])
    s = scene.build_samples(300.0, 1)
    f = workloads.shell_fixations(np.random.default_rng(3), [m], 200, dur=(0.1, 0.5))
    fix = gm.Fixations(f.eye, f.gaze, f.dur)
    ids = torch.full_like(s.mesh, bad)
    want = scene.accumulate(s.pos, fix, 2.0, occlusion="full", tri=s.tri, mesh=s.mesh).density
    got = scene.accumulate(s.pos, fix, 2.0, occlusion="full", tri=s.tri, mesh=ids).density
    assert float(want.max()) > 0 and torch.equal(got, want)
    alone = scene.accumulate(s.pos, fix, 2.0, occlusion="self", tri=s.tri, mesh=ids).density
    assert torch.equal(alone, scene.accumulate(s.pos, fix, 2.0, occlusion="none").density)
    n = int(s.pos.shape[0])
    p, e = np.arange(n, dtype=np.int32), (np.arange(n) % 200).astype(np.int32)
    vis = [scene.pair_visibility(s.pos, f.eye, p, e, occlusion="full", tri=s.tri, mesh=i).cpu() for i in (s.mesh, ids)]
    assert torch.equal(*vis) and 0 < int(vis[0].sum()) < n
