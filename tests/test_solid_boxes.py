"""Boxes inside closed meshes (host code, no GPU): a box is wholly inside its mesh and keeps its
distance from every triangle, and long triangles cost no more time than small ones."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_07571_amd", "csrc")


@pytest.fixture(scope="module")
def boxes_of(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ is not installed")
    d = tmp_path_factory.mktemp("boxes")
    exe = str(d / "boxes")
    cmd = ["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I",
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "solid_boxes_driver.cpp"), os.path.join(CSRC, "solid_boxes.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(V, I, most=12):
        with open(d / "mesh.bin", "wb") as f:
            f.write(np.array([len(V), len(I)], np.int64).tobytes())
            f.write(np.ascontiguousarray(V, np.float32).tobytes())
            f.write(np.ascontiguousarray(I, np.int32).tobytes())
        out = subprocess.run([exe, str(d / "mesh.bin"), str(most)], capture_output=True, text=True, timeout=120)
        assert out.returncode == 0
        rows = [[float(x) for x in line.split()] for line in out.stdout.splitlines()]
        return rows[0][0], rows[0][1], np.array(rows[1:]).reshape(-1, 6)
    return run


def _rod(n, length, radius, caps_only=False):
    """A rod along (1, 1, 1) of n segments (four triangles each), or a cone of two each."""
    d = np.ones(3) / np.sqrt(3.0)
    u = np.array([1.0, -1.0, 0.0]) / np.sqrt(2.0)
    w = np.cross(d, u)
    t = 2 * np.pi * np.arange(n) / n
    a = radius * (np.cos(t)[:, None] * u + np.sin(t)[:, None] * w)
    V = np.concatenate([a, a + length * d, [[0, 0, 0]], [length * d]])
    i = np.arange(n)
    j = (i + 1) % n
    c0, c1 = np.full(n, 2 * n), np.full(n, 2 * n + 1)
    F = [np.stack([c0, j, i], 1)]
    F += [np.stack([c1, i, j], 1)] if caps_only else [np.stack([i, j, n + j], 1), np.stack([i, n + j, n + i], 1),
                                                      np.stack([c1, n + i, n + j], 1)]
    return V.astype(np.float32), np.concatenate(F).astype(np.int32)


def _mesh(name):
    if name == "cone":
        return _rod(3000, 1.0, 0.5, caps_only=True)
    m = {"sphere": lambda: workloads.sphere_mesh(freq=12, radius=0.3, center=(1, 2, 3)),
         "rough": lambda: workloads.sphere_mesh(freq=20, radius=0.4, displace=0.08, seed=2),
         "knot": lambda: workloads.torus_knot_mesh(seg=200, ring=30), "cube": lambda: workloads.cube_mesh(0.5)}[name]()
    return m.V, m.I


def _winding(V, I, p):
    a, b, c = (V[I[:, k]].astype(np.float64) - p for k in range(3))
    la, lb, lc = (np.linalg.norm(x, axis=1) for x in (a, b, c))
    det = np.einsum("ij,ij->i", a, np.cross(b, c))
    den = la * lb * lc + (a * b).sum(1) * lc + (b * c).sum(1) * la + (c * a).sum(1) * lb
    return 2 * np.arctan2(det, den).sum() / (4 * np.pi)


@pytest.mark.parametrize("mesh", ["sphere", "rough", "knot", "cube", "cone"])
def test_boxes_keep_their_distance(boxes_of, mesh):
    V, I = _mesh(mesh)
    _, pad, boxes = boxes_of(V, I)
    if mesh != "knot":
        assert len(boxes) > 0
    lo, hi = V[I].min(1).astype(np.float64), V[I].max(1).astype(np.float64)
    for b in boxes:
        gap = np.maximum(lo - b[3:], b[:3] - hi).max(1)      # largest separation over the axes
        assert gap.min() >= 0.999 * pad, (gap.min(), pad)
        assert abs(abs(_winding(V, I, 0.5 * (b[:3] + b[3:]))) - 1.0) < 1e-3


def test_long_triangles_take_no_longer(boxes_of):
    """400,000 triangles, half of which span the whole grid: cell by cell 28 s, counted at the
    blocks' corners 0.05 s, like as many small ones."""
    V, I = _rod(100_000, 2.0, 0.02)
    seconds, _, boxes = boxes_of(V, I)
    assert len(boxes) == 0 and seconds < 5.0, seconds
