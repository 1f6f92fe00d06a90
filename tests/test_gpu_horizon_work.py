"""That the horizons are in use where they pay and not elsewhere, seen in the work counters: the
same fixations in one call (F sigma^2 = 1.2, horizons) and in blocks of ten (0.08, none) make
the same packets, and only the horizons change what a packet's walk visits."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("known", [True, False])
def test_horizons_shorten_the_walk(known):
    import torch
    import paper_2601_07571_amd as gm
    m = workloads.sphere_mesh(freq=30, radius=0.4, displace=0.03, seed=2)
    I = m.I[: 3 * len(m.I) // 4]                       # open: no back-face rule, no solid boxes
    scene = gm.Scene([(m.V, I)])
    s = scene.build_samples(6000.0, 1)
    f = workloads.shell_fixations(np.random.default_rng(3), [m], 160, dur=(0.1, 0.5))
    tri = s.tri if known else None                     # points without a triangle have no horizon

    def work(lo, hi):
        out = scene.accumulate(s.pos, gm.Fixations(f.eye[lo:hi], f.gaze[lo:hi], f.dur[lo:hi]), 5.0, tri=tri, mesh=s.mesh)
        torch.cuda.synchronize()
        st = scene.density_stats()
        assert float(out.max) > 0
        return np.array([st["in_cone"], st["visible"], st["node_visits"], st["triangle_tests"]], np.float64)

    one = work(0, 160)
    blocks = sum(work(lo, lo + 10) for lo in range(0, 160, 10))
    assert np.array_equal(one[:2], blocks[:2]), (one, blocks)
    if known:
        assert one[2] < 0.9 * blocks[2] and one[3] < 0.9 * blocks[3], (one, blocks)
    else:
        # packets differ a little from run to run (the order inside a bucket)
        assert np.all(np.abs(one[2:] - blocks[2:]) <= 0.03 * blocks[2:]), (one, blocks)
