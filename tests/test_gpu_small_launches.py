"""Sizes at which a map's small kernels change form: prefix sums by one block up to 32,768
elements (8,192 a pass), outputs with the maximum taken by every block up to 16,384 points,
fixation records by one block up to 16,384 fixations.

Sums, triangle indices and densities are exact integers or their one rounding, so they are
compared bit for bit, with the oracle or with the same points in a launch on the other side.
Launches of other fixation counts may take another fixed-point scale: their densities are two
roundings to FP32 apart at most, 2^-22 relative."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gm():
    import torch
    import paper_2601_07571_amd as gm
    assert torch.cuda.is_available()
    gm.load_library()
    return gm


@pytest.mark.parametrize("T", [1, 8191, 8192, 8193, 32768, 32769])
def test_prefix_sums_of_triangle_counts(gm, T):
    rng = np.random.default_rng(T)
    c = rng.uniform(-1, 1, (T, 1, 3))
    V = (c + rng.uniform(-0.02, 0.02, (T, 3, 3))).reshape(-1, 3).astype(np.float32)
    meshes = [(V, np.arange(3 * T, dtype=np.int32).reshape(T, 3))]
    s = gm.Scene(meshes).build_lattice(6000.0)
    ref = oracle.lattice_scene(meshes, 6000.0)
    assert np.array_equal(s.tri.cpu().numpy(), ref.tri)
    assert np.array_equal(s.pos.cpu().numpy().view(np.uint32), ref.pos32.view(np.uint32))


@pytest.fixture(scope="module")
def points(gm):
    m = workloads.sphere_mesh(freq=12, radius=0.4, displace=0.03, seed=1)
    scene = gm.Scene([(m.V, m.I)])
    s = scene.build_samples(11000.0, 2)
    assert int(s.pos.shape[0]) > 16385
    f = workloads.shell_fixations(np.random.default_rng(5), [m], 200, dur=(0.1, 0.5))
    return scene, s, f


@pytest.mark.parametrize("n", [1, 2, 255, 257, 16384, 16385])
def test_outputs_of_any_number_of_points(gm, points, n):
    import torch
    scene, s, f = points
    fix = gm.Fixations(f.eye, f.gaze, f.dur)
    every = scene.accumulate(s.pos, fix, 3.0, occlusion="none", tri=s.tri, mesh=s.mesh).density
    out = scene.accumulate(s.pos[:n].contiguous(), fix, 3.0, occlusion="none", tri=s.tri[:n].contiguous(),
                           mesh=s.mesh[:n].contiguous())
    torch.cuda.synchronize()
    assert torch.equal(out.density, every[:n])
    top = float(out.density.max())
    assert float(out.max.cpu()[0]) == top
    assert float(out.density_norm.max()) == (1.0 if top > 0 else 0.0)


@pytest.mark.parametrize("F", [201, 1024, 16384, 16385])
def test_fixations_of_zero_duration_change_nothing(gm, points, F):
    import torch
    scene, s, f = points
    n = 4001
    args = dict(occlusion="none", tri=s.tri[:n].contiguous(), mesh=s.mesh[:n].contiguous())
    want = scene.accumulate(s.pos[:n].contiguous(), gm.Fixations(f.eye, f.gaze, f.dur), 3.0, **args).density
    k = np.arange(F) % 200
    order = np.random.default_rng(F).permutation(F)
    dur = np.where(np.arange(F) < 200, f.dur[k], 0.0).astype(np.float32)
    got = scene.accumulate(s.pos[:n].contiguous(), gm.Fixations(f.eye[k][order], f.gaze[k][order], dur[order]), 3.0, **args).density
    torch.cuda.synchronize()
    assert float(want.max()) > 0
    assert bool(((got - want).abs() <= 2.0 ** -22 * want).all())
