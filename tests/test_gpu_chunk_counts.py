"""Time of a map against the number of chunks its fixations are cut into: no count is far slower
than its neighbour (chunks differ in work; were every tile's chunk c to run on the same part of
the chip, 32 chunks would take 1.26 times as long as 33, and 33 or 97 under other fixed orders)."""
import time

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def test_no_slow_chunk_counts(monkeypatch):
    import torch
    import paper_2601_07571_amd as gm
    m = workloads.plate_mesh(size=0.8, cells=32)
    f = workloads.shell_fixations(np.random.default_rng(3), [m], 1000, dur=(0.1, 0.5))
    fix = gm.Fixations(f.eye, f.gaze, f.dur)
    best = {}
    maps = {}
    for chunk in (33, 32, 31):  # 31, 32 and 33 chunks
        monkeypatch.setenv("GM_FIX_PER_CHUNK", str(chunk))
        scene = gm.Scene([(m.V, m.I)])
        s = scene.build_samples(300000 / 0.64, 1)
        out = scene.accumulate(s.pos, fix, 1.0, tri=s.tri, mesh=s.mesh)
        torch.cuda.synchronize()
        for _ in range(12):
            t = time.perf_counter()
            for _ in range(4):
                scene.accumulate(s.pos, fix, 1.0, tri=s.tri, mesh=s.mesh, out=out)
            torch.cuda.synchronize()
            best[chunk] = min(best.get(chunk, 1e9), time.perf_counter() - t)
        maps[chunk] = out.density.clone()
    assert torch.equal(maps[31], maps[32]) and torch.equal(maps[33], maps[32])
    assert max(best.values()) <= 1.12 * min(best.values()), best
