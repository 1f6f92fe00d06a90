"""Which closed meshes have solid boxes (those of at least 1,000 triangles, under full occlusion),
seen in the work counters, and parity with the oracle on bodies that have them and hold outside
space or share their boxes' tree with others."""
import numpy as np
import pytest

import workloads
from test_gpu_rules import _check, _eyes, _floor, _join, _sphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("freq,occlusion,boxes", [(7, "full", False), (8, "full", True), (14, "full", True),
                                                  (14, "self", False)])
def test_which_meshes_have_boxes(freq, occlusion, boxes):
    """Points on an open floor (the back-face rule has no part in their pairs) under closed
    bodies: without boxes the flags make no difference to the walk, with them an occluded
    packet's triangle tests fall away."""
    import torch
    import paper_2601_07571_amd as gm
    centers = [(0.35 * a - 0.35, 0.35 * b - 0.35, 0.4) for a in range(3) for b in range(3)]
    bodies = [_sphere(0.15, c, freq) for c in centers]
    plate = workloads.plate_mesh(size=1.4, cells=40)
    scene = gm.Scene([(plate.V, plate.I)] + bodies)
    s = scene.build_samples(8000.0, 7)
    on = s.mesh == 0
    rng = np.random.default_rng(4)
    eye, gaze, dur = _eyes(rng, 100, (-0.5, -0.5, 1.4), (0.5, 0.5, 2.0), (0, 0, 0))
    args = (s.pos[on].contiguous(), gm.Fixations(eye, gaze, dur), 4.0)
    kw = dict(occlusion=occlusion, tri=s.tri[on].contiguous(), mesh=s.mesh[on].contiguous())
    got = []
    for flag in (True, False):
        for m in range(1, len(bodies) + 1):
            scene.set_mesh_closed(m, flag)
        out = scene.accumulate(*args, **kw)
        torch.cuda.synchronize()
        got.append((out.density, scene.density_stats()))
    (d0, with_), (d1, without) = got
    assert float(d0.max()) > 0 and torch.equal(d0, d1)
    # packets differ a little from run to run (the order inside a bucket)
    same = all(abs(with_[k] - without[k]) <= 0.03 * without[k] for k in ("node_visits", "triangle_tests"))
    assert same != boxes, (with_, without)
    if boxes:
        assert with_["triangle_tests"] < 0.95 * without["triangle_tests"], (with_, without)


def _jar(n):
    """A surface of revolution, closed: outer wall, a narrow mouth, inner wall."""
    prof = [(0.0, 0.1), (0.25, 0.1), (0.25, 0.6), (0.012, 0.6), (0.012, 0.55), (0.2, 0.55), (0.2, 0.15), (0.0, 0.15)]
    V, rows = [], []
    for r, z in prof:
        k = np.arange(n) if r > 0 else np.zeros(n, int)
        rows.append(len(V) + k)
        V += [(r * np.cos(2 * np.pi * i / n), r * np.sin(2 * np.pi * i / n), z) for i in range(n if r > 0 else 1)]
    F = []
    for a, b in zip(rows[:-1], rows[1:]):
        for k in range(n):
            p, q, r, s = a[k], a[(k + 1) % n], b[(k + 1) % n], b[k]
            F += [t for t in ((p, q, r), (p, r, s)) if len(set(t)) == 3]
    V, F = np.array(V, np.float32), np.array(F, np.int32)
    v = V[F].astype(np.float64)
    return V, F if np.einsum("ij,ij->", v[:, 0], np.cross(v[:, 1], v[:, 2])) > 0 else F[:, [0, 2, 1]]


def _cube(edge, center, cells):
    """A cube of cells x cells squares a side."""
    g = np.linspace(-0.5, 0.5, cells + 1)
    V, F = [], []
    for axis in range(3):
        for sign in (-1, 1):
            base = len(V)
            for b in g:
                for a in g:
                    p = [0.0, 0.0, 0.0]
                    p[axis], p[(axis + 1) % 3], p[(axis + 2) % 3] = 0.5 * sign, a, b
                    V.append(p)
            for j in range(cells):
                for i in range(cells):
                    q = base + j * (cells + 1) + i
                    f = [(q, q + 1, q + cells + 2), (q, q + cells + 2, q + cells + 1)]
                    F += f if sign > 0 else [(a, c, b) for a, b, c in f]
    return (np.array(V) * edge + np.asarray(center)).astype(np.float32), np.array(F, np.int32)


BODIES = {
    "jar": lambda: [_floor(), _jar(200)],
    "cube": lambda: [_floor(), _cube(0.4, (0, 0, 0.45), 14)],
    "many": lambda: [_floor()] + [_sphere(0.12, (0.3 * a - 0.45, 0.3 * b - 0.45, 0.35), 10) for a in range(4) for b in range(4)],
    "mixed": lambda: [_floor(), _sphere(0.2, (-0.2, 0, 0.5), 12), _cube(0.2, (0.3, 0, 0.4), 2),
                      _join(_sphere(0.15, (0, 0.3, 0.4)), _sphere(0.12, (0.1, 0.3, 0.5)))],
}


@pytest.mark.parametrize("name", sorted(BODIES))
def test_fine_bodies_match_the_oracle(name):
    import torch
    import paper_2601_07571_amd as gm
    assert torch.cuda.is_available()
    meshes = BODIES[name]()
    assert gm.Scene(meshes).mesh_closed()[1:].all() and any(len(f) >= 1000 for _, f in meshes[1:])
    rng = np.random.default_rng(3)
    eye, gaze, dur = _eyes(rng, 40, (-0.5, -0.5, 1.4), (0.5, 0.5, 2.0), (0, 0, 0))
    st = _check(gm, meshes, 400.0, eye, gaze, dur, 4.0, "full")
    assert 0 < st["visible"] < st["in_cone"], st
    eye, gaze, dur = _eyes(rng, 24, (-0.1, -0.1, 0.3), (0.1, 0.1, 0.45), (0, 0, 0))
    _check(gm, meshes, 400.0, eye, gaze, dur, 5.0, "full")
