"""Points that do not lie on the triangle they are given: a triangle hides a point unless it is
the point's own, whichever way the map finds that out.  Points well inside a closed body, seen
through their own triangle alone, are visible; the same points without a triangle are not."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth", [0.0, 1e-6, 1e-3, 0.05, 0.12])
@pytest.mark.parametrize("F", [40, 200])  # without and with horizons (F sigma^2 = 0.05 and 0.24)
def test_points_behind_their_own_triangle(depth, F):
    import torch
    import paper_2601_07571_amd as gm
    assert torch.cuda.is_available()
    m = workloads.sphere_mesh(freq=12, radius=0.25)
    V, I = np.asarray(m.V, np.float64), np.asarray(m.I)
    pick = np.random.default_rng(2).choice(len(I), F, replace=False)
    c = V[I[pick]].mean(1)
    n = np.cross(V[I[pick, 1]] - V[I[pick, 0]], V[I[pick, 2]] - V[I[pick, 0]])
    n /= np.linalg.norm(n, axis=1, keepdims=True)
    pos = (c - depth * n).astype(np.float32)
    eye, gaze = (c + 1.5 * n).astype(np.float32), (-n).astype(np.float32)
    dur = np.full(F, 0.3, np.float32)
    meshes = [(m.V, m.I)]
    scene = gm.Scene(meshes)
    mesh = np.zeros(F, np.int32)
    for tri in (pick.astype(np.int32), np.full(F, -1, np.int32)):
        got = scene.accumulate(pos, gm.Fixations(eye, gaze, dur), 2.0, occlusion="full", tri=tri, mesh=mesh)
        torch.cuda.synchronize()
        got = got.density.cpu().numpy().astype(np.float64)
        ref = oracle.density(oracle.Scene(meshes), pos, tri, mesh, eye, gaze, dur, 2.0, mode=oracle.OCC_FULL)
        # the suite's tolerance: 1e-5 relative and the oracle's own ambiguous pairs
        assert np.all(np.abs(got - ref.rho) <= 1e-5 * ref.rho + ref.budget + 1e-30), np.abs(got - ref.rho).max()
        if tri[0] >= 0:
            assert np.all(ref.rho > 0)
        elif depth >= 1e-3:
            assert np.all(ref.rho <= ref.budget)  # an edge of two triangles may be ambiguous
