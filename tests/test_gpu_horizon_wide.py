"""Horizons are found by packets of points or, for few points, by a wave each; either way they
only bound what a segment can meet near its point, so a point's density is the same bit for bit
in a launch of any number of points with the same fixations (exact sums)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

LAST = 163840  # the most points that take a wave each


@pytest.fixture(scope="module")
def case():
    import torch
    import paper_2601_07571_amd as gm
    assert torch.cuda.is_available()
    gm.load_library()
    body = workloads.sphere_mesh(freq=24, radius=0.4, displace=0.05, seed=2)
    v = np.array([(x, y, 0.02 * np.sin(30 * x) * np.cos(25 * y) - 0.5) for y in np.linspace(-1, 1, 61)
                  for x in np.linspace(-1, 1, 61)], np.float32)
    q = np.arange(60 * 60)
    a = q + q // 60
    f = np.concatenate([np.stack([a, a + 1, a + 62], 1), np.stack([a, a + 62, a + 61], 1)]).astype(np.int32)
    scene = gm.Scene([(body.V, body.I), (v, f)])
    s = scene.build_samples((LAST + 4000) / 6.2, 1)
    assert int(s.pos.shape[0]) > LAST
    fx = workloads.shell_fixations(np.random.default_rng(3), [body], 160, dur=(0.1, 0.5))
    fix = gm.Fixations(fx.eye, fx.gaze, fx.dur)  # 160 at 5 degrees: F sigma^2 = 1.2, horizons in use
    order = torch.from_numpy(np.random.default_rng(4).permutation(int(s.pos.shape[0]))).cuda()
    pos, tri, mesh = s.pos[order].contiguous(), s.tri[order].contiguous(), s.mesh[order].contiguous()

    def run(n):
        out = scene.accumulate(pos[:n], fix, 5.0, occlusion="full", tri=tri[:n], mesh=mesh[:n])
        torch.cuda.synchronize()
        return out.density

    return run, run(int(pos.shape[0]))


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1001, LAST, LAST + 1])
def test_any_number_of_points(case, n):
    run, every = case
    got = run(n)
    assert float(every.max()) > 0
    assert bool((got == every[:n]).all())
