"""The rules that settle visibility pairs without a walk of the triangles, or shorten it, on
the GPU against the FP64 oracle (which knows none of them), on scenes made to break them.

Solid boxes: a segment that meets a box inside a closed mesh is occluded.  Bodies that are
closed but hold outside space (a hollow shell, a jar whose mouth is narrower than a grid
cell), a body of one box, two bodies that overlap, an eye inside a body's bounding box, the
occluder's closed flag cleared, self occlusion (another mesh's solid must not count).

Horizons: a segment steeper than everything near its point begins its walk beyond it.  Steps,
a thin fence standing on a floor, a plate floating just above it, a groove, a floor whose
triangles are far larger than the objects on it, and points without a known triangle.

The tolerance is parity_util's: 1e-5 relative plus the oracle's own ambiguous pairs, and no
visibility decision other than the oracle's outside its fragile set."""
import numpy as np
import pytest

import oracle
import parity_util
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gm():
    import torch
    import paper_2601_07571_amd as gm
    assert torch.cuda.is_available()
    gm.load_library()
    return gm


def _grid(nx, ny, f):
    """(nx x ny)-cell sheet, vertex (i, j) at f(i / nx, j / ny)."""
    V = np.array([f(i / nx, j / ny) for j in range(ny + 1) for i in range(nx + 1)], np.float32)
    F = []
    for j in range(ny):
        for i in range(nx):
            a = j * (nx + 1) + i
            F += [(a, a + 1, a + nx + 2), (a, a + nx + 2, a + nx + 1)]
    return V, np.array(F, np.int32)


def _floor(size=2.0, cells=40, z=0.0):
    return _grid(cells, cells, lambda u, v: ((u - 0.5) * size, (v - 0.5) * size, z))


def _sphere(radius, center, freq=14):
    m = workloads.sphere_mesh(freq=freq, radius=radius, center=center)
    return m.V, m.I


def _join(*meshes):
    V, F, base = [], [], 0
    for v, f in meshes:
        V.append(v)
        F.append(f + base)
        base += len(v)
    return np.concatenate(V).astype(np.float32), np.concatenate(F).astype(np.int32)


def _shell():
    """One closed mesh: an outer sphere and, wound the other way, an inner one."""
    v, f = _sphere(0.25, (0, 0, 0.4))
    w, g = _sphere(0.2, (0, 0, 0.4))
    return _join((v, f), (w, g[:, [0, 2, 1]]))


def _jar():
    """A surface of revolution, closed: outer wall, a narrow mouth, inner wall."""
    prof = [(0.0, 0.1), (0.25, 0.1), (0.25, 0.6), (0.012, 0.6), (0.012, 0.55), (0.2, 0.55), (0.2, 0.15), (0.0, 0.15)]
    n = 40
    V, rows = [], []
    for r, z in prof:
        if r == 0.0:
            rows.append([len(V)] * n)
            V.append((0, 0, z))
        else:
            rows.append(list(range(len(V), len(V) + n)))
            V += [(r * np.cos(2 * np.pi * k / n), r * np.sin(2 * np.pi * k / n), z) for k in range(n)]
    F = []
    for a, b in zip(rows[:-1], rows[1:]):
        for k in range(n):
            p, q, r, s = a[k], a[(k + 1) % n], b[(k + 1) % n], b[k]
            F += [t for t in ((p, q, r), (p, r, s)) if len(set(t)) == 3]
    V = np.array(V, np.float32); F = np.array(F, np.int32)
    v = V[F].astype(np.float64)
    if np.einsum("ij,ij->", v[:, 0], np.cross(v[:, 1], v[:, 2])) < 0:
        F = F[:, [0, 2, 1]]
    return V, F


def _cube(edge, center):
    m = workloads.cube_mesh(edge, center)
    return m.V, m.I


def _eyes(rng, F, lo, hi, target):
    eye = rng.uniform(lo, hi, (F, 3))
    tgt = np.asarray(target)[None] + rng.uniform(-0.35, 0.35, (F, 3)) * [1, 1, 0.2]
    return eye.astype(np.float32), (tgt - eye).astype(np.float32), rng.uniform(0.1, 0.5, F).astype(np.float32)


def _check(gm, meshes, k, eye, gaze, dur, theta, occlusion, clear=None, with_tri=True, most=6000):
    import torch
    scene = gm.Scene(meshes)
    if clear is not None:
        scene.set_mesh_closed(clear, False)
    s = scene.build_samples(k, 5)
    assert int(s.pos.shape[0]) <= most
    out = scene.accumulate(s.pos, gm.Fixations(eye, gaze, dur), theta, occlusion=occlusion,
                           tri=s.tri if with_tri else None, mesh=s.mesh)
    torch.cuda.synchronize()
    pos, mesh = s.pos.cpu().numpy(), s.mesh.cpu().numpy()
    tri = s.tri.cpu().numpy() if with_tri else np.full(len(pos), -1, np.int32)
    mode = {"self": oracle.OCC_SELF, "full": oracle.OCC_FULL}[occlusion]
    ref = oracle.density(oracle.Scene(meshes), pos, tri, mesh, eye, gaze, dur, theta, mode=mode)
    got = out.density.cpu().numpy().astype(np.float64)
    parity_util.check(gm, scene, meshes, pos, tri, mesh, eye, gaze, dur, theta, mode, got, ref)
    firm, fragile, pairs = parity_util.count_flips(scene, meshes, pos, tri, mesh, eye, gaze, dur, theta, mode)
    assert firm == 0 and pairs > 1000, (firm, pairs)
    return scene.density_stats()


SOLIDS = {
    "sphere": lambda: [_floor(), _sphere(0.25, (0, 0, 0.5))],
    "one_box": lambda: [_floor(), _cube(0.4, (0, 0, 0.45))],
    "shell": lambda: [_floor(), _shell()],
    "jar": lambda: [_floor(), _jar()],
    "overlap": lambda: [_floor(), _join(_sphere(0.22, (0, 0, 0.4)), _sphere(0.2, (0.15, 0, 0.5)))],
    "many": lambda: [_floor()] + [_sphere(0.08, (0.2 * a - 0.5, 0.2 * b - 0.5, 0.3), 6) for a in range(6) for b in range(6)],
}


@pytest.mark.parametrize("occlusion", ["full", "self"])
@pytest.mark.parametrize("name", sorted(SOLIDS))
def test_solid_boxes(gm, name, occlusion):
    rng = np.random.default_rng(3)
    eye, gaze, dur = _eyes(rng, 40, (-0.5, -0.5, 1.4), (0.5, 0.5, 2.0), (0, 0, 0))
    st = _check(gm, SOLIDS[name](), 500.0 if name != "many" else 300.0, eye, gaze, dur, 4.0, occlusion)
    assert 0 < st["visible"] < st["in_cone"], st


def test_eyes_inside_the_bounding_box_and_inside_the_body(gm):
    """Eyes in the corners of the sphere's box (outside the body) and in the jar's hollow."""
    rng = np.random.default_rng(4)
    eye, gaze, dur = _eyes(rng, 24, (0.2, 0.2, 0.6), (0.24, 0.24, 0.7), (0, 0, 0.2))
    _check(gm, [_floor(), _sphere(0.25, (0, 0, 0.5))], 500.0, eye, gaze, dur, 5.0, "full")
    eye, gaze, dur = _eyes(rng, 24, (-0.1, -0.1, 0.3), (0.1, 0.1, 0.45), (0, 0, 0))
    _check(gm, [_floor(), _jar()], 700.0, eye, gaze, dur, 5.0, "full")


def test_cleared_flag_takes_the_mesh_out_of_the_rule(gm):
    rng = np.random.default_rng(6)
    eye, gaze, dur = _eyes(rng, 30, (-0.5, -0.5, 1.4), (0.5, 0.5, 2.0), (0, 0, 0))
    on = _check(gm, SOLIDS["one_box"](), 500.0, eye, gaze, dur, 4.0, "full")
    off = _check(gm, SOLIDS["one_box"](), 500.0, eye, gaze, dur, 4.0, "full", clear=1)
    assert on["visible"] == off["visible"] and off["triangle_tests"] > on["triangle_tests"], (on, off)


def _wavy(u, v):
    x, y = (u - 0.5) * 1.2, (v - 0.5) * 1.2
    return x, y, 0.02 * np.sin(40 * x) * np.cos(35 * y)


NEAR = {
    "steps": lambda: [_grid(48, 48, lambda u, v: ((u - 0.5) * 1.2, (v - 0.5) * 1.2, 0.01 * np.floor(8 * u)))],
    "waves": lambda: [_grid(64, 64, _wavy)],
    "groove": lambda: [_grid(48, 48, lambda u, v: ((u - 0.5) * 1.2, (v - 0.5) * 1.2, 0.8 * abs(u - 0.5)))],
    "fence": lambda: [_floor(1.2, 40), _grid(60, 2, lambda u, v: ((u - 0.5) * 1.2, 0.0003, 0.02 * v)),
                      _grid(60, 2, lambda u, v: (0.0151, (u - 0.5) * 1.2, 0.03 * v))],
    "plate": lambda: [_floor(1.2, 40), _grid(20, 20, lambda u, v: ((u - 0.5) * 0.4, (v - 0.5) * 0.4, 0.002))],
    "big_floor": lambda: [_grid(1, 1, lambda u, v: ((u - 0.5) * 1.6, (v - 0.5) * 1.6, 0.0)), _sphere(0.1, (0, 0, 0.1)),
                          _sphere(0.05, (0.2, 0.1, 0.05))],
}


@pytest.mark.parametrize("name", sorted(NEAR))
def test_horizons(gm, name):
    """160 fixations at 5 degrees (F sigma^2 = 1.2: the horizons are in use), eyes low over the
    surface and high above it."""
    rng = np.random.default_rng(8)
    a = _eyes(rng, 100, (-1.2, -1.2, 0.1), (1.2, 1.2, 0.5), (0, 0, 0))
    b = _eyes(rng, 60, (-0.5, -0.5, 1.0), (0.5, 0.5, 1.6), (0, 0, 0))
    eye, gaze, dur = (np.concatenate(x) for x in zip(a, b))
    _check(gm, NEAR[name](), 900.0, eye, gaze, dur, 5.0, "full")


def test_points_without_a_triangle(gm):
    """No own triangle: no normal, no horizon; every pair is walked, also where the point lies
    on the surface."""
    rng = np.random.default_rng(9)
    eye, gaze, dur = _eyes(rng, 160, (-0.6, -0.6, 0.6), (0.6, 0.6, 1.4), (0, 0, 0))
    _check(gm, NEAR["waves"](), 500.0, eye, gaze, dur, 5.0, "full", with_tri=False)


def test_map_blocks_share_one_horizon(gm):
    """An incremental map computes its points' horizons at the first launch that they pay for:
    blocks before and after it, on two streams, give the one-call map bit for bit."""
    import torch
    m = workloads.sphere_mesh(freq=20, radius=0.4, displace=0.04, seed=2)
    scene = gm.Scene([(m.V, m.I)])
    s = scene.build_samples(2000.0, 1)
    f = workloads.shell_fixations(np.random.default_rng(3), [m], 500, dur=(0.1, 0.5))
    fix = gm.Fixations(f.eye, f.gaze, f.dur)
    args = dict(theta_deg=4.0, occlusion="full", tri=s.tri, mesh=s.mesh)
    one = gm.DensityMap(scene, s.pos, **args).add(fix).read()
    split = gm.DensityMap(scene, s.pos, **args)
    split.add(fix.subset(0, 40))
    split.read()                       # too few fixations for horizons
    split.add(fix.subset(40, 400))
    split.read()
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    with torch.cuda.stream(other):
        split.add(fix.subset(400, 500))
        two = split.read()
    torch.cuda.synchronize()
    assert float(one.max.cpu()[0]) > 0
    assert torch.equal(one.density, two.density) and torch.equal(one.max, two.max)
    plain = scene.accumulate(s.pos, fix, 4.0, tri=s.tri, mesh=s.mesh)
    assert torch.equal(plain.density > 0, one.density > 0)
