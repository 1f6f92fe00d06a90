"""Performance cases of the density-map framework: the calls that its users make, through the
public Python entry points, over the range of sizes they are made at.

`listed()` are the fixed cases, `draw(rng)` gives another of the same ranges; `prepare` makes
what a program holds before the call (scene handle, samples, fixations, a planned batch, network
weights), `run` is one call, `work` what it cannot do without, and `exact` the same outputs in
64-bit arithmetic without this package, where that is affordable.

Scenes are procedural and seeded: displaced spheres (closed meshes), a cube, a torus-knot tube
and a two-density terrain (an open mesh), eyes walking around them at head height or spread in
a shell, gaze at surface points that face the eye, one degree of jitter.
"""
import math

import numpy as np
import torch

import paper_2601_07571_amd as gm


# ---------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------
def listed():
    return [
        # one small object, a short recording: an interactive preview, where launches and latency count
        {"name": "tiny_map", "kind": "map", "scene": "sphere", "tris": 1352, "n": 6253, "F": 100, "theta": 1.0,
         "occ": "self"},
        # one participant's session on one scanned object at a coarse sampling rate
        {"name": "session_map", "kind": "map", "scene": "sphere", "tris": 60000, "n": 12007, "F": 2501, "theta": 1.2,
         "occ": "full"},
        # the paper-shaped map: four meshes, two million samples, one long recording, full occlusion
        {"name": "objects_map", "kind": "map", "scene": "objects", "tris": 800000, "n": 2000010, "F": 6000,
         "theta": 1.0, "occ": "full"},
        # the same without a visibility test (an overview map, or samples known to be unobstructed)
        {"name": "objects_no_occlusion", "kind": "map", "scene": "objects", "tris": 100000, "n": 2000010, "F": 6000,
         "theta": 1.0, "occ": "none"},
        # many objects in a room, several recordings pooled, ten thousand samples per square metre
        {"name": "room_map", "kind": "map", "scene": "room", "tris": 500000, "n": 400003, "F": 12000, "theta": 1.0,
         "occ": "full"},
        # a study: uneven sessions planned and tuned once, replayed as one graph
        {"name": "sessions_batch", "kind": "batch", "sessions": 16, "tris": 50000, "F": 6000, "k": 5000.0},
        # objects that move while they are looked at: each fixation with the meshes' poses at its time
        {"name": "moving_objects", "kind": "posed", "tris": 100000, "n": 300007, "F": 1500, "theta": 1.0},
        # the paper's own visibility: a z-buffer per fixation
        {"name": "zbuffer_map", "kind": "zbuffer", "tris": 200000, "n": 500009, "F": 1500, "theta": 1.0, "R": 128},
        # sampling the surfaces, as each map of a new density or seed needs first
        {"name": "surface_samples", "kind": "samples", "tris": 200000, "n": 2000010},
        # the paper's per-triangle lattice on a fine mesh (three points a triangle and more)
        {"name": "lattice_samples", "kind": "lattice", "tris": 200000, "n": 1000003},
        # one frame of a renderer that asks the neural field for every visible surface point
        {"name": "field_frame", "kind": "predict", "tris": 20000, "n": 2000010},
        # two hundred steps of training a field on a map, one network per mesh, with its held-out check
        {"name": "field_training", "kind": "train", "tris": 20000, "n": 400003, "batch": 16384, "steps": 200},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["map", "map", "map", "map", "map", "batch", "posed", "zbuffer", "samples", "lattice", "predict",
                       "train"])
    if kind == "map":
        c = {"kind": kind, "scene": rng.choice(["sphere", "objects", "room"]), "tris": _log(rng, 1300, 400000),
             "n": _log(rng, 6000, 1000000), "F": _log(rng, 100, 6000), "theta": round(rng.uniform(0.5, 1.5), 2),
             "occ": rng.choice(["full", "full", "self", "none"])}
        # no more pairs in view than the largest listed map
        while c["n"] * c["F"] * c["theta"] ** 2 > 2.0e9:
            c["n"] = max(6000, int(c["n"] * 0.7))
            c["F"] = max(100, int(c["F"] * 0.8))
        return c
    if kind == "batch":
        return {"kind": kind, "sessions": rng.randint(3, 16), "tris": _log(rng, 10000, 50000), "F": _log(rng, 600, 6000),
                "k": round(rng.uniform(1000.0, 6000.0), 1)}
    if kind == "posed":
        return {"kind": kind, "tris": _log(rng, 2000, 100000), "n": _log(rng, 20000, 300000), "F": _log(rng, 40, 1500),
                "theta": round(rng.uniform(0.5, 1.2), 2)}
    if kind == "zbuffer":
        return {"kind": kind, "tris": _log(rng, 5000, 200000), "n": _log(rng, 20000, 500000), "F": _log(rng, 100, 1500),
                "theta": round(rng.uniform(0.5, 1.5), 2), "R": rng.choice([64, 128, 128])}
    if kind in ("samples", "lattice"):
        return {"kind": kind, "tris": _log(rng, 1300, 200000), "n": _log(rng, 10000, 2000000 if kind == "samples" else 1000000)}
    if kind == "predict":
        return {"kind": kind, "tris": _log(rng, 2000, 20000), "n": _log(rng, 2000, 2000000)}
    return {"kind": "train", "tris": _log(rng, 2000, 20000), "n": _log(rng, 50000, 400000),
            "batch": rng.choice([1024, 4096, 8192, 10000, 16384]), "steps": rng.randint(50, 200)}


# ---------------------------------------------------------------------------------------------
# meshes (vertices float32, indices int32) and recordings
# ---------------------------------------------------------------------------------------------
def _noise(rng, p, base=3.0, octaves=4, waves=6):
    out = np.zeros(p.shape[0])
    for o in range(octaves):
        d = rng.normal(size=(waves, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        out += (np.sin((p @ d.T) * (base * 2.0 ** o) + rng.uniform(0, 2 * np.pi, waves))).sum(1) * 0.5 ** o / math.sqrt(waves)
    return out


def _sphere(tris, radius, center, displace, rng):
    """Octahedron with every face cut into f x f triangles, pushed to a displaced sphere: closed, outward."""
    f = max(2, int(round(math.sqrt(tris / 8.0))))
    i, j = np.meshgrid(np.arange(f + 1), np.arange(f + 1), indexing="ij")
    inside = i + j <= f
    num = -np.ones((f + 1, f + 1), np.int64)
    num[inside] = np.arange(inside.sum())
    ii, jj = i[inside], j[inside]
    up = num[:-1, :-1][(i + j)[:-1, :-1] < f], num[1:, :-1][(i + j)[:-1, :-1] < f], num[:-1, 1:][(i + j)[:-1, :-1] < f]
    two = (i + j)[:-1, :-1] < f - 1
    dn = num[1:, :-1][two], num[1:, 1:][two], num[:-1, 1:][two]
    face = np.concatenate([np.stack(up, 1), np.stack(dn, 1)])
    P, T = [], []
    for o in range(8):
        s = np.array([1 if o & 1 else -1, 1 if o & 2 else -1, 1 if o & 4 else -1])
        P.append(np.stack([ii, jj, f - ii - jj], 1) * s)
        T.append((face if s.prod() > 0 else face[:, [0, 2, 1]]) + o * len(ii))
    P, T = np.concatenate(P), np.concatenate(T)
    key = (P[:, 0] + f) * (2 * f + 1) ** 2 + (P[:, 1] + f) * (2 * f + 1) + (P[:, 2] + f)
    _, first, inv = np.unique(key, return_index=True, return_inverse=True)
    d = P[first].astype(np.float64)
    # arc spacing nearly even on every face
    d = np.sign(d) * np.sin(np.abs(d) / f * (np.pi / 2))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    r = np.full(len(d), radius)
    if displace:
        h = _noise(rng, d)
        r = radius * (1.0 + displace * h / max(1e-9, np.abs(h).max()))
    return (d * r[:, None] + np.asarray(center)).astype(np.float32), inv.reshape(-1)[T].astype(np.int32)


def _cube(edge, center):
    h = edge / 2.0
    V = np.array([[x, y, z] for x in (-h, h) for y in (-h, h) for z in (-h, h)]) + np.asarray(center)
    F = []
    for a, b, c, d in [(0, 1, 3, 2), (4, 6, 7, 5), (0, 4, 5, 1), (2, 3, 7, 6), (0, 2, 6, 4), (1, 5, 7, 3)]:
        F += [(a, b, c), (a, c, d)]
    return V.astype(np.float32), np.array(F, np.int32)


def _knot(tris, center):
    """A tube around the (2, 3) torus knot: closed, concave, hides parts of itself."""
    ring = max(6, int(round(math.sqrt(tris / 20.0))))
    seg = max(24, tris // (2 * ring))

    def curve(t):
        r = 0.3 + 0.12 * np.cos(3 * t)
        return np.stack([r * np.cos(2 * t), -0.12 * np.sin(3 * t), r * np.sin(2 * t)], -1)
    t = np.arange(seg) * (2 * np.pi / seg)
    C = curve(t)
    tg = curve(t + 1e-4) - curve(t - 1e-4)
    tg /= np.linalg.norm(tg, axis=1, keepdims=True)
    N = np.cross(tg, [0.0, 1.0, 0.0])
    N /= np.linalg.norm(N, axis=1, keepdims=True)
    B = np.cross(tg, N)
    a = np.arange(ring) * (2 * np.pi / ring)
    V = (C[:, None] + 0.04 * (np.cos(a)[None, :, None] * N[:, None] + np.sin(a)[None, :, None] * B[:, None])).reshape(-1, 3)
    i, j = np.arange(seg)[:, None], np.arange(ring)[None, :]
    p, q = i * ring + j, ((i + 1) % seg) * ring + j
    r, s = ((i + 1) % seg) * ring + (j + 1) % ring, i * ring + (j + 1) % ring
    F = np.concatenate([np.stack([p, q, r], -1).reshape(-1, 3), np.stack([p, r, s], -1).reshape(-1, 3)])
    v = V[F[:, 0]], V[F[:, 1]], V[F[:, 2]]
    if np.einsum("ij,ij->", v[0], np.cross(v[1], v[2])) < 0:
        F = F[:, [0, 2, 1]]
    return (V + np.asarray(center)).astype(np.float32), F.astype(np.int32)


def _terrain(tris, size, rng):
    """A size x size relief, y up, its left half sixteen times denser than the right (open)."""
    n = max(4, int(math.sqrt(tris * 16.0 / 17.0 / 4.0)))
    fine, coarse = (n, 2 * n), (max(1, n // 4), max(1, n // 2))
    h = size / 2.0
    state = rng.integers(0, 2 ** 31)

    def half(x0, x1, nx, nz):
        X, Z = np.meshgrid(np.linspace(x0, x1, nx + 1), np.linspace(-h, h, nz + 1), indexing="ij")
        p = np.stack([X.ravel(), np.zeros(X.size), Z.ravel()], 1)
        p[:, 1] = 0.05 * np.clip(np.abs(p[:, 0]) / (0.1 * size), 0, 1) * _noise(np.random.default_rng(state), p, 2.0)
        a = np.arange(nx)[:, None] * (nz + 1) + np.arange(nz)[None, :]
        b = a + nz + 1
        return p, np.concatenate([np.stack([a, a + 1, b + 1], -1).reshape(-1, 3), np.stack([a, b + 1, b], -1).reshape(-1, 3)])
    p0, f0 = half(-h, 0.0, *fine)
    p1, f1 = half(0.0, h, *coarse)
    return np.concatenate([p0, p1]).astype(np.float32), np.concatenate([f0, f1 + len(p0)]).astype(np.int32)


def _meshes(scene, tris, rng):
    if scene == "sphere":
        return [_sphere(tris, 0.5, (0, 0, 0), 0.04, rng)]
    if scene == "terrain":
        return [_terrain(tris, 1.6, rng)]
    if scene == "objects":
        return [_sphere(0.4 * tris, 0.5, (-0.5, 0.62, -0.45), 0.05, rng), _cube(0.5, (0.55, 0.3, -0.45)),
                _knot(int(0.25 * tris), (0.0, 0.62, 0.45)), _terrain(0.35 * tris, 2.0, rng)]
    return [_sphere(tris / 25.0, 0.6, (1.5 * (a - 2), 0.6, 1.5 * (b - 2)), 0.04, rng) for a in range(5) for b in range(5)]


def _areas(V, I):
    a = V[I[:, 0]].astype(np.float64)
    return 0.5 * np.linalg.norm(np.cross(V[I[:, 1]] - a, V[I[:, 2]] - a), axis=1)


def _area(meshes):
    return float(sum(_areas(V, I).sum() for V, I in meshes))


def _walk(rng, F, r_in, r_out, height=1.6):
    """Eyes of a head that walks around the scene in steps of about 5 cm between r_in and r_out."""
    d = rng.normal(scale=0.035, size=(F, 2)).cumsum(0)
    span = r_out - r_in
    r = r_in + np.abs((d[:, 0] + 0.5 * span) % (2 * span) - span)
    a = rng.uniform(0, 2 * np.pi) + d[:, 1] / (0.5 * (r_in + r_out))
    return np.stack([r * np.cos(a), np.full(F, height), r * np.sin(a)], 1)


def _shell(rng, F, r_in, r_out):
    d = rng.normal(size=(F, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return d * rng.uniform(r_in ** 3, r_out ** 3, F)[:, None] ** (1.0 / 3.0)


def _recording(rng, meshes, eye):
    """Gaze at surface points that face the eye, an object picked at random, 1 degree of jitter; 0.1 to 0.5 s each."""
    F = len(eye)
    which = rng.integers(0, len(meshes), F)
    target = np.zeros((F, 3))
    for m, (V, I) in enumerate(meshes):
        todo = np.nonzero(which == m)[0]
        cum = np.cumsum(_areas(V, I))
        for _ in range(12):
            t = I[np.searchsorted(cum, rng.uniform(0, cum[-1], len(todo))).clip(max=len(I) - 1)]
            a, b, c = (V[t[:, k]].astype(np.float64) for k in range(3))
            target[todo] = (a + b + c) / 3
            todo = todo[np.einsum("ij,ij->i", np.cross(b - a, c - a), eye[todo] - target[todo]) <= 0]
            if not len(todo):
                break
    d = target - eye
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    u = np.cross(d, np.where(np.abs(d[:, :1]) < 0.9, [[1.0, 0, 0]], [[0, 1.0, 0]]))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    w = np.cross(d, u)
    j = np.tan(np.radians(rng.normal(size=(F, 2))))
    return eye.astype(np.float32), (d + j[:, :1] * u + j[:, 1:] * w).astype(np.float32), rng.uniform(0.1, 0.5, F).astype(np.float32)


def _eyes(scene, rng, F):
    if scene == "sphere":
        return _shell(rng, F, 1.5, 2.5)
    if scene == "terrain":
        return _walk(rng, F, 1.0, 1.9)
    if scene == "objects":
        return _walk(rng, F, 1.8, 2.6)
    return np.concatenate([_walk(rng, F // 6 + (1 if i < F % 6 else 0), 4.2, 5.5) for i in range(6)])


def _world(case, seed):
    """Meshes, recording and sampling rate of a map case."""
    rng = np.random.default_rng([seed, 17])
    scene = case.get("scene", "objects")
    meshes = _meshes(scene, case["tris"], rng)
    return meshes, _recording(rng, meshes, _eyes(scene, rng, case["F"])), case["n"] / _area(meshes)


def _fixed_world(case, seed):
    """Meshes whose areas do not depend on the seed (sample counts then do not either): vertices on
    a 2^-20 m grid, moved by a seeded whole number of 2^-6 m, which float32 holds exactly."""
    meshes = _meshes("objects", case["tris"], np.random.default_rng([case["tris"], 19]))
    by = np.random.default_rng([seed, 19]).integers(-64, 65, 3) / 64.0
    return [((np.round(V.astype(np.float64) * 2 ** 20) / 2 ** 20 + by).astype(np.float32), I) for V, I in meshes]


def _exactly(s, n):
    """The first n samples of a sampling call (its count is a rounding per mesh of rate times area)."""
    return gm.Samples(s.tri[:n].contiguous(), s.mesh[:n].contiguous(), s.bary[:n].contiguous(), s.pos[:n].contiguous())


def _sessions(case, seed):
    """Meshes, recording, number of samples and cone angle of each session; the sizes are the case's
    own on every seed, triangles and fixations uneven by a factor of ten."""
    size = np.random.default_rng([case["sessions"], case["tris"], 23])
    rng = np.random.default_rng([seed, 23])
    out = []
    for _ in range(case["sessions"]):
        u = size.uniform(size=5)
        scene = "sphere" if u[0] < 0.6 else "terrain"
        meshes = _meshes(scene, case["tris"] * 10.0 ** -u[2], rng)
        fix = _recording(rng, meshes, _eyes(scene, rng, int(round(case["F"] * 0.08 ** u[1]))))
        n = int(case["k"] * (0.2 + 1.4 * u[3]) * (3.1 if scene == "sphere" else 2.6))
        out.append((meshes, fix, n, 0.5 + 1.5 * float(u[4])))
    return out


def _poses(rng, F, meshes):
    """Row-major 3 x 4 poses: every mesh but the last turns about the vertical through its centre and drifts."""
    t = np.cumsum(rng.uniform(0.13, 0.53, F))
    pose = np.zeros((F, len(meshes), 3, 4))
    for m, (V, _) in enumerate(meshes):
        w, c = (0.05 * (m + 1) if m + 1 < len(meshes) else 0.0), V.mean(0).astype(np.float64)
        A = np.zeros((F, 3, 3))
        A[:, 0, 0] = A[:, 2, 2] = np.cos(w * t)
        A[:, 0, 2], A[:, 2, 0], A[:, 1, 1] = np.sin(w * t), -np.sin(w * t), 1.0
        pose[:, m, :, :3] = A
        pose[:, m, :, 3] = c - A @ c
        pose[:, m, 0, 3] += 0.1 * w / 0.05 * np.sin(0.2 * t)
    return pose.reshape(F, len(meshes), 12).astype(np.float32)


def _weights(seed, M):
    """He-uniform weights of M networks in the package's parameter order, small biases."""
    rng = np.random.default_rng([seed, 31])
    nets = []
    for _ in range(M):
        p = []
        for fan, width in ((96, 64), (64, 64), (64, 64), (64, 64), (64, 1)):
            p += [rng.uniform(-1, 1, fan * width) * math.sqrt(6.0 / fan) * (0.3 if width == 1 else 1.0),
                  rng.uniform(-0.05, 0.05, width)]
        nets.append(np.concatenate(p))
    return np.stack(nets).astype(np.float32)


def _target(pos, seed):
    """A map-like target in [0, 1]: a few dozen gaze spots of 3 to 10 cm."""
    rng = np.random.default_rng([seed, 37])
    g = torch.Generator(device="cpu").manual_seed(int(rng.integers(2 ** 31)))
    at = pos[torch.randint(0, pos.shape[0], (40,), generator=g).to(pos.device)]
    s = torch.tensor(rng.uniform(0.03, 0.1, 40), dtype=torch.float32, device=pos.device)
    w = torch.tensor(rng.uniform(0.1, 1.0, 40), dtype=torch.float32, device=pos.device)
    out = torch.zeros(pos.shape[0], device=pos.device)
    for k in range(40):
        out += w[k] * torch.exp(-((pos - at[k]) ** 2).sum(1) / (2 * s[k] ** 2))
    return out / out.max()


# ---------------------------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    if kind == "batch":
        ss = []
        for meshes, fix, n, theta in _sessions(case, seed):
            scene = gm.Scene(meshes)
            s = _exactly(scene.build_samples(n / _area(meshes) * (1.0 + 1e-4) + 2.0, seed), n)
            ss.append({"scene": scene, "pos": s.pos, "tri": s.tri, "mesh": s.mesh, "fix": gm.Fixations(*fix),
                       "theta_deg": theta, "occlusion": "full"})
        st["batch"] = gm.Batch(ss, tune=True)
        return st
    if kind in ("map", "posed", "zbuffer"):
        meshes, fix, k = _world(case, seed)
        st["scene"], st["fix"] = gm.Scene(meshes), gm.Fixations(*fix)
        # a little over, then the first n: the count is then the case's on every seed
        st["samples"] = _exactly(st["scene"].build_samples(k * (1.0 + 1e-4) + 64.0, seed), case["n"])
        if kind == "posed":
            st["pose"] = torch.from_numpy(_poses(np.random.default_rng([seed, 29]), case["F"], meshes)).cuda()
            s = st["samples"]
            st["map"] = gm.DensityMap(st["scene"], s.pos, case["theta"], tri=s.tri, mesh=s.mesh, posed=True)
        return st
    meshes = _fixed_world(case, seed)
    scene = st["scene"] = gm.Scene(meshes)
    k = st["k"] = case["n"] / _area(meshes)
    st["seed"] = seed
    if kind == "samples":
        st["capacity"] = int(scene.count_samples(k).sum())  # as a program sizes its buffers
    elif kind == "lattice":
        st["capacity"] = int(scene.count_lattice(k).sum())
    else:
        s = st["samples"] = _exactly(scene.build_samples(k * (1.0 + 1e-4) + 64.0, seed), case["n"])
        st["field"] = gm.Field(scene, seed=seed)
        st["weights"] = _weights(seed, len(meshes))
        st["field"].set_params(st["weights"])
        if kind == "train":
            st["target"] = _target(s.pos, seed)
    return st


def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "batch":
        return [(o.density, o.density_norm, o.max) for o in st["batch"].run()]
    if kind == "map":
        s = st["samples"]
        o = st["scene"].accumulate(s.pos, st["fix"], case["theta"], occlusion=case["occ"], tri=s.tri, mesh=s.mesh)
        return o.density, o.density_norm, o.max
    if kind == "zbuffer":
        o = st["scene"].accumulate_zbuffer(st["samples"].pos, st["fix"], case["theta"], resolution=case["R"])
        return o.density, o.density_norm, o.max
    if kind == "posed":
        st["map"].reset()
        st["map"].add_posed(st["fix"], st["pose"])
        o = st["map"].read()
        return o.density, o.density_norm, o.max
    if kind == "samples":
        s = st["scene"].build_samples(st["k"], st["seed"], capacity=st["capacity"])
        return s.tri, s.mesh, s.bary, s.pos
    if kind == "lattice":
        s = st["scene"].build_lattice(st["k"], capacity=st["capacity"])
        return s.tri, s.mesh, s.bary, s.pos
    s = st["samples"]
    if kind == "predict":
        return st["field"].predict(s.pos, s.mesh)
    st["field"].set_params(st["weights"])
    info = st["field"].train(s.pos, s.mesh, st["target"], steps=case["steps"], batch=case["batch"], seed=7)
    return st["field"].get_params(), info["rel_l2"], info["loss"]


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------
_MLP = 2 * (96 * 64 + 3 * 64 * 64 + 64)


def _map_work(n, F, tris, theta, occ):
    """Points, fixations and triangles read once, two values a point written; about 4 % of the
    pairs lie in a 1 degree cone: 60 operations for a value, and for a visibility test one descent
    of a binary tree over the triangles (two boxes of 18 operations a level)."""
    pairs = n * F * min(1.0, 0.042 * theta ** 2)
    deep = 36.0 * math.log2(max(2.0, tris)) if occ != "none" else 0.0
    return {"bytes": 28.0 * n + 28.0 * F + (18.0 * tris if deep else 0.0), "flops": pairs * (60.0 + deep)}


def work(case):
    kind, n, tris = case["kind"], case.get("n", 0), case["tris"]
    if kind == "map":
        return _map_work(n, case["F"], tris, case["theta"], case["occ"])
    if kind == "batch":
        one = _map_work(2.6 * case["k"], 0.36 * case["F"], 0.39 * tris, 1.3, "full")
        return {k: v * case["sessions"] for k, v in one.items()}
    if kind == "posed":
        w = _map_work(n, case["F"], tris, case["theta"], "full")
        return {"bytes": w["bytes"] + 192.0 * case["F"], "flops": w["flops"]}
    if kind == "zbuffer":
        w = _map_work(n, case["F"], tris, case["theta"], "none")
        px = case["F"] * case["R"] ** 2
        return {"bytes": w["bytes"] + 4.0 * px + 18.0 * tris, "flops": w["flops"] + px * 36.0 * math.log2(tris)}
    if kind == "samples":
        return {"bytes": 28.0 * n + 26.0 * tris, "flops": 160.0 * n}
    if kind == "lattice":
        n = max(n, 3.0 * tris)
        return {"bytes": 28.0 * n + 34.0 * tris, "flops": 40.0 * n + 20.0 * tris}
    if kind == "predict":
        return {"bytes": 20.0 * n, "flops": float(_MLP) * n}
    seen = 4.0 * case["steps"] * case["batch"]  # four networks
    return {"bytes": 28.0 * n + 16.0 * seen + 4.0 * case["steps"] * 18753 * 24.0, "flops": 3.0 * _MLP * seen + float(_MLP) * n}


# ---------------------------------------------------------------------------------------------
# the same outputs in 64 bits, without the package's code
# ---------------------------------------------------------------------------------------------
def _philox(c, key):
    """Philox4x32-10 of counter columns c (four uint64 arrays below 2^32) under a 64-bit key."""
    lo = np.uint64(0xFFFFFFFF)
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & lo, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & lo]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _tri_areas(V, I):
    a = V[I[:, 0]].astype(np.float64)
    u, w = V[I[:, 1]] - a, V[I[:, 2]] - a
    c = [u[:, 1] * w[:, 2] - u[:, 2] * w[:, 1], u[:, 2] * w[:, 0] - u[:, 0] * w[:, 2], u[:, 0] * w[:, 1] - u[:, 1] * w[:, 0]]
    return 0.5 * np.sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2])


def _exact_samples(meshes, k, seed):
    """(b1, b2) and position of every sample: triangles chosen by area, the square-root warp inside."""
    bary, pos = [], []
    for m, (V, I) in enumerate(meshes):
        A = _tri_areas(V, I)
        S = 52 - math.frexp(len(A) * float(A.max()))[1]
        C = np.cumsum(np.floor(np.ldexp(A, S)).astype(np.uint64))
        n = int(math.floor(math.ldexp(float(C[-1]), -S) * k + 0.5))
        j = np.arange(n, dtype=np.uint64)
        x = _philox([j, np.zeros_like(j), np.full_like(j, m), np.zeros_like(j)], seed)
        # floor(U C / 2^64), U = x0 2^32 + x1, C < 2^52
        W, s = int(C[-1]), np.uint64(32)
        w0, w1, lo = np.uint64(W & 0xFFFFFFFF), np.uint64(W >> 32), np.uint64(0xFFFFFFFF)
        ll, lh, hl = x[1] * w0, x[1] * w1, x[0] * w0
        goal = x[0] * w1 + (lh >> s) + (hl >> s) + (((ll >> s) + (lh & lo) + (hl & lo)) >> s)
        t = I[np.searchsorted(C, goal, side="right")]
        su, v = np.sqrt(np.ldexp(x[2].astype(np.float64), -32)), np.ldexp(x[3].astype(np.float64), -32)
        b1, b2 = su * (1.0 - v), su * v
        p = (1.0 - su)[:, None] * V[t[:, 0]].astype(np.float64) + b1[:, None] * V[t[:, 1]] + b2[:, None] * V[t[:, 2]]
        bary.append(np.stack([b1, b2], 1))
        pos.append(p)
    return None, None, np.concatenate(bary), np.concatenate(pos)


def _exact_lattice(meshes, k):
    bary, pos = [], []
    for V, I in meshes:
        d = (8.0 * k) * _tri_areas(V, I) + 1.0
        r = np.where(d >= 25.0, np.floor((np.sqrt(d) - 3.0) / 2.0), 1.0).astype(np.int64)
        cnt = (r + 1) * (r + 2) // 2
        t = np.repeat(np.arange(len(I)), cnt)
        idx = np.arange(len(t)) - np.repeat(np.cumsum(cnt) - cnt, cnt)
        row = ((np.sqrt(8.0 * idx + 1.0) - 1.0) / 2.0).astype(np.int64)
        row += (row + 1) * (row + 2) // 2 <= idx
        row -= row * (row + 1) // 2 > idx
        col, rr = idx - row * (row + 1) // 2, r[t].astype(np.float64)
        w1, w2, w3 = col / rr, (rr - row) / rr, (row - col) / rr
        p = w1[:, None] * V[I[t, 0]].astype(np.float64) + w2[:, None] * V[I[t, 1]] + w3[:, None] * V[I[t, 2]]
        bary.append(np.stack([w2, w3], 1))
        pos.append(p)
    return None, None, np.concatenate(bary), np.concatenate(pos)


def _hidden(x, e, own, V0, E1, E2, N):
    """Which segments x -> e (rows, float64) some triangle but their own crosses, 1e-4 of their length away from x."""
    out = torch.zeros(len(x), dtype=torch.bool, device=x.device)
    step = max(1, 40_000_000 // len(V0))
    ids = torch.arange(len(V0), device=x.device)
    for a in range(0, len(x), step):
        o, d = x[a:a + step, None], (e - x)[a:a + step, None]
        det = -(d * N).sum(-1)
        r = o - V0
        q = torch.cross(r, d.expand_as(r), dim=-1)
        u, v, t = (E2 * q).sum(-1) / det, -(E1 * q).sum(-1) / det, (r * N).sum(-1) / det
        hit = (det != 0) & (u >= 0) & (v >= 0) & (u + v <= 1) & (t > 1e-4) & (t < 1) & (ids != own[a:a + step, None])
        out[a:a + step] = hit.any(1)
    return out


def _exact_map(case, seed):
    """Density, normalised density and maximum in 64 bits; occlusion by every triangle in turn on the small scenes."""
    meshes, (eye, gaze, dur), k = _world(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    s = _exact_samples(meshes, k * (1.0 + 1e-4) + 64.0, seed)[3][:case["n"]].astype(np.float32)  # the points as the call gets them
    X = torch.from_numpy(s).to(dev).double()
    sigma = math.tan(math.radians(case["theta"]))
    rho = torch.zeros(len(X), dtype=torch.float64, device=dev)
    walk = case["occ"] != "none"
    if walk:
        V = np.concatenate([v for v, _ in meshes])
        I = np.concatenate([i for _, i in meshes])  # one mesh (the caller sees to it)
        P = torch.from_numpy(V).to(dev).double()[torch.from_numpy(I.astype(np.int64)).to(dev)]
        V0, E1, E2 = P[:, 0], P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]
        N = torch.cross(E1, E2, dim=-1)
        own = torch.from_numpy(_own_triangles(meshes, k * (1.0 + 1e-4) + 64.0, seed)[:case["n"]]).to(dev)
    for f in range(len(eye)):
        e, g = torch.from_numpy(eye[f]).to(dev).double(), torch.from_numpy(gaze[f]).to(dev).double()
        p = X - e
        d1 = p @ g
        at = torch.nonzero(d1 > 0)[:, 0]
        # a cheap look first: (p.r)^2 (1 + 16 s^2) >= |p|^2 |r|^2, with room
        q = (p * p).sum(1)
        at = at[(d1[at] ** 2 * (1 + 16 * sigma ** 2) * (1 + 1e-6) >= q[at] * (g @ g))]
        c = torch.cross(p[at], g.expand(len(at), 3), dim=1)
        t2 = (c * c).sum(1) / d1[at] ** 2
        keep = t2 <= 16 * sigma ** 2
        at, t2 = at[keep], t2[keep]
        if walk:
            seen = ~_hidden(X[at], e.expand(len(at), 3), own[at], V0, E1, E2, N)
            at, t2 = at[seen], t2[seen]
        rho[at] += float(dur[f]) / (sigma * math.sqrt(2 * math.pi)) * torch.exp(-t2 / (2 * sigma ** 2))
    top = rho.max().reshape(1)
    return rho, (rho / top if float(top) > 0 else torch.zeros_like(rho)), top


def _own_triangles(meshes, k, seed):
    (V, I), = meshes
    A = _tri_areas(V, I)
    S = 52 - math.frexp(len(A) * float(A.max()))[1]
    C = np.cumsum(np.floor(np.ldexp(A, S)).astype(np.uint64))
    n = int(math.floor(math.ldexp(float(C[-1]), -S) * k + 0.5))
    j = np.arange(n, dtype=np.uint64)
    x = _philox([j, np.zeros_like(j), np.zeros_like(j), np.zeros_like(j)], seed)
    total = int(C[-1])
    goal = np.array([(((int(a) << 32) | int(b)) * total) >> 64 for a, b in zip(x[0], x[1])], np.uint64)
    return np.searchsorted(C, goal, side="right")


def _exact_predict(case, seed):
    meshes = _fixed_world(case, seed)
    k = case["n"] / _area(meshes) * (1.0 + 1e-4) + 64.0
    pos = _exact_samples(meshes, k, seed)[3].astype(np.float32)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    weights, out, at = _weights(seed, len(meshes)), [], 0
    for m, (V, I) in enumerate(meshes):
        n = len(_exact_count(V, I, k))
        x = torch.from_numpy(pos[at:at + n]).to(dev).double()
        at += n
        used = V[np.unique(I)].astype(np.float64)
        lo, ext = used.min(0), float((used.max(0) - used.min(0)).max())
        f = torch.tensor([32.0 ** (b / 15.0) for b in range(16)], dtype=torch.float64, device=dev)
        p, o = torch.from_numpy(weights[m]).to(dev).double(), 0
        for a in range(0, n, 1 << 18):
            z = (x[a:a + (1 << 18)] - torch.from_numpy(lo).to(dev)) / ext
            ph = 2 * math.pi * f[None, :, None] * z[:, None, :]
            h = torch.stack([torch.sin(ph), torch.cos(ph)], -1).reshape(len(z), 96)
            o = 0
            for fan, width in ((96, 64), (64, 64), (64, 64), (64, 64), (64, 1)):
                h = h @ p[o:o + fan * width].reshape(fan, width) + p[o + fan * width:o + fan * width + width]
                o += fan * width + width
                h = torch.relu(h) if width > 1 else torch.nn.functional.softplus(h)
            out.append(h[:, 0])
    return torch.cat(out)[:case["n"]]


def _exact_count(V, I, k):
    A = _tri_areas(V, I)
    S = 52 - math.frexp(len(A) * float(A.max()))[1]
    total = float(np.floor(np.ldexp(A, S)).astype(np.uint64).sum())
    return range(int(math.floor(math.ldexp(total, -S) * k + 0.5)))


def exact(case, seed):
    kind = case["kind"]
    if kind == "map":
        # every triangle against every pair in view: only where that is a few 1e10 tests
        if case["occ"] != "none" and (case["scene"] != "sphere" or
                                      case["n"] * case["F"] * 0.06 * case["theta"] ** 2 * case["tris"] > 2e9):
            return None
        return _exact_map(case, seed)
    if kind in ("samples", "lattice"):
        meshes = _fixed_world(case, seed)
        k = case["n"] / _area(meshes)
        return _exact_samples(meshes, k, seed) if kind == "samples" else _exact_lattice(meshes, k)
    if kind == "predict":
        return _exact_predict(case, seed)
    # visibility through large scenes, and training (hundreds of dependent 16-bit steps)
    return None
