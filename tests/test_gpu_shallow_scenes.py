"""Scenes whose trees are a few levels deep, or flat: their launches are cut into longer chunks,
as launches without a visibility test are, and their points get no horizons, which cost more
than the walks they shorten."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _scene(gm, name):
    if name == "relief":  # a plate with waves of 2e-4 of its size
        m = workloads.plate_mesh(0.8, 32)
        m.V[:, 2] = 8e-5 * np.sin(50 * m.V[:, 0]) * np.cos(40 * m.V[:, 1])
        return gm.Scene([(m.V, m.I)]), m, 0.64
    m = {"cube": lambda: workloads.cube_mesh(0.5), "plate": lambda: workloads.plate_mesh(0.8, 32),
         "coarse": lambda: workloads.sphere_mesh(freq=4, radius=0.3), "fine": lambda: workloads.sphere_mesh(freq=40, radius=0.3)}[name]()
    area = np.linalg.norm(np.cross(m.V[m.I[:, 1]] - m.V[m.I[:, 0]], m.V[m.I[:, 2]] - m.V[m.I[:, 0]]), axis=1).sum() / 2
    return gm.Scene([(m.V, m.I)]), m, area


def test_chunks_follow_the_depth():
    import torch
    import paper_2601_07571_amd as gm
    assert torch.cuda.is_available()
    items = {}
    for name in ("cube", "plate", "coarse", "fine"):
        scene, m, area = _scene(gm, name)
        s = scene.build_samples(60000 / area, 1)
        f = workloads.shell_fixations(np.random.default_rng(3), [m], 1000, dur=(0.1, 0.5))
        b = gm.Batch([dict(scene=scene, pos=s.pos[:50000].contiguous(), tri=s.tri[:50000].contiguous(),
                           mesh=s.mesh[:50000].contiguous(), fix=gm.Fixations(f.eye, f.gaze, f.dur), theta_deg=1.0)])
        items[name] = b.info()["work_items"]
    assert items["cube"] == items["plate"] < items["coarse"] < items["fine"], items


@pytest.mark.parametrize("name,horizons", [("cube", False), ("plate", False), ("relief", True), ("coarse", True),
                                           ("fine", True)])
def test_horizons_where_walks_are_long(name, horizons):
    """Device memory of a second call whose fixations suffice for horizons (F sigma^2 = 1.2)."""
    import torch
    import paper_2601_07571_amd as gm
    scene, m, area = _scene(gm, name)
    s = scene.build_samples(1.2e6 / area, 1)
    n = int(s.pos.shape[0])
    f = workloads.shell_fixations(np.random.default_rng(3), [m], 1000, dur=(0.1, 0.5))
    fix = gm.Fixations(f.eye, f.gaze, f.dur)
    out = scene.accumulate(s.pos, fix, 0.2, tri=s.tri, mesh=s.mesh)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    scene.accumulate(s.pos, fix, 2.0, tri=s.tri, mesh=s.mesh, out=out)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    # 4 bytes a point more than closed meshes hold anyway (an open flat one: 20), in pieces of 2 MB
    assert (used >= 4 * n) == horizons, (used, n)
