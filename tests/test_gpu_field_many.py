"""Training of many small meshes: the networks are taken in groups that share one scratch.

The scratch stays bounded whatever their number (439 MB of activations and row sums, against 1.2
MB for every network before), and a network's step does not depend on the group it is in: the
step gradient of networks at both ends and at group edges equals gm_field_gradient's over the
points drawn for it, by the same means and with the same tolerance as the tests of one step."""
import numpy as np
import pytest

import workloads
from test_gpu_field_step import _philox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_meshes,batch", [
    (300, 1024),   # 32 tiles for 12 slots a network, 6 rows: groups of many networks
    (700, 64),     # two tiles: two rows
    (300, 16384),  # 512 tiles for 12 slots: 43 rounds, groups of a few networks
])
def test_many_networks(n_meshes, batch):
    import torch
    import paper_2601_07571_amd as gm
    meshes = [workloads.sphere_mesh(level=1, radius=0.2, center=(0.5 * m, 0, 0)) for m in range(n_meshes)]
    scene = gm.Scene([(m.V, m.I) for m in meshes])
    s = scene.build_samples(300.0, 3)
    n = int(s.pos.shape[0])
    target = torch.tensor(np.random.default_rng(5).uniform(0, 1, n).astype(np.float32), device="cuda")
    f = gm.Field(scene, seed=4)
    p0 = f.get_params().reshape(n_meshes, -1)
    seed, hold, eps = 77, 0.25, np.float32(1e4)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    f.train(s.pos, s.mesh, target, steps=1, batch=batch, lr=1e-30, lr_final=float(1e3 * eps), beta1=0.0, beta2=0.0,
            eps=float(eps), holdout=hold, seed=seed)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    # besides: a few words a point, allocation in pieces of 2 MB
    assert used <= 439e6 + 64 * n + 32e6, used
    p1 = f.get_params().reshape(n_meshes, -1)
    i = np.arange(n, dtype=np.uint64)
    z = np.zeros_like(i)
    train = _philox([i, z, z, z + np.uint64(3)], seed, 0)[0] >= np.uint64(int(hold * 2 ** 32))
    mesh = s.mesh.cpu().numpy()
    f.set_params(p0)
    for m in sorted({0, 1, 15, 16, 17, 255, 256, 257, n_meshes // 2, n_meshes - 2, n_meshes - 1}):
        idx = np.nonzero(train & (mesh == m))[0]
        j = np.arange(batch, dtype=np.uint64)
        z = np.zeros_like(j)
        c = _philox([j, z, z, z + np.uint64(4)], (seed ^ 0x5bd1e995) ^ m, 0x1b873593)[0]
        pick = torch.tensor(idx[((c * np.uint64(len(idx))) >> np.uint64(32)).astype(np.int64)], device="cuda")
        g = f.gradient(s.pos[pick], target[pick], net=m)[0].astype(np.float64)
        d = p0[m].astype(np.float64) - p1[m]
        got = d * float(eps) / (1e3 * float(eps) - np.abs(d))
        tol = 1e-5 * np.linalg.norm(g) + 2.0 ** -23 * np.linalg.norm(np.abs(p0[m]) + 1e3 * np.abs(g)) / 1e3
        assert np.linalg.norm(got - g) <= tol, (m, np.linalg.norm(got - g), tol, np.linalg.norm(g))
