"""The work that programs have this library do, as cases that can be timed.

A case is a dict of plain values.  ``kind`` names the entry points it calls:

  score       render_score, logL only: a search stage over a hypothesis grid
  grad        render_score with the adjoint: gradient refinement, calibration
  marginal    render_score_marginal: the hierarchical likelihood, 4 x 4 noise grid
  render      render_batch: point images and triangle ids of many poses
  split       score: logL of point images that are in memory
  split_grad  score_backward then render_backward: the adjoint of that path
  frame       one new camera frame: depth to points, the static objects drawn,
              the observation set, one search stage scored
  tracker     one frame of the multi-object tracker: search and Adam steps
  batch       many scenes of mixed sizes with the adjoint

The objects are blobs of 1 cm voxels (12 triangles each) 0.8 m in front of the
camera, as everywhere in this repository; images go from 64 x 48 to 320 x 240,
windows from 3 x 3 to 7 x 7, objects from 200 to 6,000 voxels, searches from 16
hypotheses to 10,000.  All inputs are FP32, the only type the library takes.
"""

import math

import numpy as np
import torch

import paper_2312_08715_amd as b3d

VOXEL = 0.01
DEPTH = 0.8
SIGMA, P_OUT, VOLUME = 0.003, 0.01, 1.0
NOISE_GRID = (0.01, 4, 4)  # largest deviation, deviations, outlier probabilities


# ---- the cases ------------------------------------------------------------


def listed():
    def case(name, kind, height, width, voxels, hyps, window, others=0, table=False, scenes=1, solid=False):
        return dict(name=name, kind=kind, height=height, width=width, voxels=voxels, hyps=hyps, window=window,
                    others=others, table=table, scenes=scenes, solid=solid)

    return [
        # the smallest search the benchmark times: one launch, latency counts
        case("small_search", "score", 48, 64, 500, 256, 3),
        # the benchmark's own step: 24,000 triangles, 5,000 hypotheses, an occluder in front
        case("paper_adjoint", "grad", 120, 160, 2000, 5000, 5, others=1),
        # the first coarse-to-fine stage of an object of the table scene
        case("table_search", "score", 240, 320, 1500, 10000, 5, others=3, table=True),
        # a big object in an odd-sized image with a wide window: it fills several bands of rows
        case("ragged_adjoint", "grad", 227, 301, 6000, 700, 7, others=1),
        # camera tracking: object and table top move as one mesh and fill the image
        case("pan_search", "score", 200, 200, 1047, 729, 5, solid=True),
        # pose search under unknown noise
        case("noise_grid", "marginal", 120, 160, 2000, 5000, 5, others=1),
        # point images for a program's own likelihood
        case("render_images", "render", 120, 160, 2000, 2000, 5),
        # logL of given point images
        case("score_images", "split", 120, 160, 2000, 5000, 5),
        # and its gradient with respect to points, noise and poses
        case("score_images_adjoint", "split_grad", 120, 160, 2000, 2000, 5),
        # what every new camera frame costs a search of one object among others
        case("new_frame", "frame", 240, 320, 1500, 500, 5, others=3, table=True),
        # a frame of three-object tracking: 12,500 hypotheses and Adam steps per object
        case("track_frame", "tracker", 120, 160, 3000, 10000, 5, others=2),
        # many robots' scenes served together
        case("scene_batch", "batch", 120, 160, 2000, 500, 5, others=1, scenes=12),
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["score", "score", "grad", "grad", "marginal", "render", "split", "split_grad", "frame",
                       "tracker", "batch"])
    height, width = spread(48, 240), spread(64, 320)
    if rng.random() < 0.5:  # sizes of real cameras, else odd ones
        height, width = max(48, height // 8 * 8), max(64, width // 8 * 8)
    voxels = spread(200, 6000)
    scenes = rng.randint(2, 16) if kind == "batch" else 1
    most = 3.0e8 / (12 * voxels + height * width) / (3 * scenes if kind in ("batch", "tracker") else 1)
    if kind in ("render", "split", "split_grad"):
        most = min(most, 4.0e7 / (height * width))
    hyps = spread(16, max(17, min(10000, int(most))))
    solid = kind == "score" and rng.random() < 0.25
    others = 0 if solid else rng.randint(0, 3)
    return dict(kind=kind, height=height, width=width, voxels=voxels, hyps=hyps, window=rng.choice([3, 5, 5, 7]),
                others=min(others, 2) if kind == "tracker" else others, table=not solid and rng.random() < 0.4,
                scenes=scenes, solid=solid)


# ---- geometry and inputs --------------------------------------------------


def _radius(voxels):
    return max(0.10, VOXEL * (6.0 * voxels / (4.0 * math.pi)) ** (1.0 / 3.0))


def _f32(a):
    """Values as the library takes them, widened again."""
    return np.asarray(a, dtype=np.float32).astype(np.float64)


_CORNERS = np.array([[(k >> 0) & 1, (k >> 1) & 1, (k >> 2) & 1] for k in range(8)], dtype=np.float64)
_FACES = np.array([[0, 4, 6], [0, 6, 2], [1, 3, 7], [1, 7, 5], [0, 1, 5], [0, 5, 4], [2, 6, 7], [2, 7, 3],
                   [0, 2, 3], [0, 3, 1], [4, 5, 7], [4, 7, 6]], dtype=np.int32)
_TABLE = (np.array([[-0.5, -0.5, 0.0], [0.5, -0.5, 0.0], [0.5, 0.5, 0.0], [-0.5, 0.5, 0.0]]),
          np.array([[0, 1, 2], [0, 2, 3]], dtype=np.int32))


def _voxel_mesh(centres):
    verts = centres[:, None, :] + (_CORNERS - 0.5) * VOXEL
    tris = _FACES[None] + 8 * np.arange(len(centres), dtype=np.int32)[:, None, None]
    return _f32(verts.reshape(-1, 3)), tris.reshape(-1, 3).astype(np.int32)


def _blob(voxels, rng):
    """A learned voxel model: distinct cells of a ball, at most half of it."""
    r = _radius(voxels)
    m = int(r / VOXEL)
    g = np.stack(np.meshgrid(*[np.arange(-m, m + 1)] * 3, indexing="ij"), -1).reshape(-1, 3)
    g = g[(g ** 2).sum(1) * VOXEL ** 2 <= r * r]
    pick = np.sort(rng.choice(len(g), size=min(voxels, len(g)), replace=False))
    return _voxel_mesh(g[pick] * VOXEL)


def _bottle_on_table(voxels):
    """A solid box of about `voxels` cells standing on a 0.5 m table top, one mesh."""
    a = max(2, int(round((voxels / 1.7) ** (1.0 / 3.0))))
    n = (a, max(1, int(0.6 * a)), max(1, int(round(1.7 * a / 0.6))))
    g = np.stack(np.meshgrid(*[np.arange(k) for k in n], indexing="ij"), -1).reshape(-1, 3)
    v, t = _voxel_mesh((g - np.array([n[0] / 2, n[1] / 2, 0]) + 0.5) * VOXEL)
    lift = np.array([0.0, 0.0, 0.5 * v[:, 2].max()])
    return _f32(np.concatenate([v, 0.5 * _TABLE[0]]) - lift), np.concatenate([t, _TABLE[1] + len(v)]).astype(np.int32)


def _rotations(n, rng, angle=None):
    """Uniform rotations (Shoemake), or turns of at most `angle` about uniform axes."""
    if angle is None:
        q = rng.normal(size=(n, 4))
        q /= np.linalg.norm(q, axis=1, keepdims=True)
    else:
        k = rng.normal(size=(n, 3))
        half = 0.5 * angle * rng.random(n)
        q = np.concatenate([np.cos(half)[:, None], k * (np.sin(half) / np.linalg.norm(k, axis=1))[:, None]], 1)
    w, x, y, z = q.T
    return np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                     2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                     2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], 1).reshape(n, 3, 3)


def _poses(R, t):
    P = np.tile(np.eye(4), (len(R), 1, 1))
    P[:, :3, :3], P[:, :3, 3] = R, t
    return _f32(P)


def _tilted(degrees):
    """A frame whose +z leans towards the camera: a table top seen from above."""
    a = math.radians(90.0 + degrees)
    return np.array([[1, 0, 0], [0, math.cos(a), -math.sin(a)], [0, math.sin(a), math.cos(a)]])


class _World:
    """Meshes, poses, camera, observation and hypotheses of one scene of a case."""

    def __init__(self, case, seed, index=0):
        rng = np.random.default_rng([seed, index])
        scale = (1.0, 0.6, 1.6)[index % 3] if case["scenes"] > 1 else 1.0
        self.H = max(24, int(case["height"] * (1.0, 1.5, 0.8)[index % 3 if case["scenes"] > 1 else 0]))
        self.W = max(32, int(case["width"] * (1.0, 1.5, 0.8)[index % 3 if case["scenes"] > 1 else 0]))
        self.f = float(np.float32(0.9375 * self.W))
        n = max(100, int(case["voxels"] * scale))
        self.N = max(1, int(case["hyps"] / scale)) if case["scenes"] > 1 else case["hyps"]
        self.window = case["window"]
        if case["solid"]:
            self.mesh = _bottle_on_table(n)
            R0 = _tilted(35.0) @ _rotations(1, rng, 0.3)[0]
            t0 = np.array([0.0, 0.0, 0.6])
        else:
            self.mesh = _blob(n, rng)
            R0, t0 = _rotations(1, rng)[0], np.array([0.0, 0.0, DEPTH])
        self.truth = _poses(R0[None], t0[None])
        r = _radius(n)
        # other objects: the first in front, hiding an edge of this one, the others beside it
        places = [(1.5 * r, 0.3 * r, DEPTH - 1.8 * r), (-1.9 * r, 0.4 * r, DEPTH), (0.3 * r, -2.0 * r, DEPTH + r)]
        self.statics = [_blob(n if case["kind"] == "tracker" else max(100, n // 2), rng) for _ in range(case["others"])]
        at = [_poses(_rotations(1, rng), np.array(p)[None]) for p in places[:case["others"]]]
        if case["table"]:
            self.statics.append((_f32(_TABLE[0]), _TABLE[1]))
            at.append(_poses(_tilted(45.0)[None], np.array([[0.0, 0.7 * r, DEPTH + 0.7 * r]])))
        self.static_poses = np.concatenate(at) if at else np.zeros((0, 4, 4))
        # the observation: 2 mm depth noise on surfaces, 3 % of pixels replaced
        z, _ = _render([(*self.mesh, self.truth)] + [(*m, p[None]) for m, p in zip(self.statics, self.static_poses)],
                       self)
        z = z[0].cpu().numpy()
        z = np.where(z > 0, z + rng.normal(0.0, 0.002, z.shape), 0.0)
        z = np.where(rng.random(z.shape) < 0.03, rng.uniform(0.3, 1.5, z.shape), z)
        self.depth = torch.as_tensor(z, dtype=torch.float32, device="cuda")
        ray = self.rays().float()
        self.obs = (self.depth[..., None] * ray).contiguous()
        # hypotheses: half around the truth as in a late stage, half anywhere as in a first one
        near = (self.N + 1) // 2
        if case["solid"]:
            R, t = _rotations(self.N, rng, 0.03) @ R0, t0 + rng.uniform(-0.006, 0.006, (self.N, 3))
        else:
            R = np.concatenate([_rotations(near, rng, 0.25) @ R0, _rotations(self.N - near, rng)])
            t = t0 + np.concatenate([rng.uniform(-0.01, 0.01, (near, 3)),
                                     rng.uniform(-1, 1, (self.N - near, 3)) * (0.04, 0.04, 0.02)])
        self.poses = _poses(R, t)

    def rays(self):
        c = (torch.arange(self.W, dtype=torch.float64, device="cuda") + 0.5 - self.W / 2.0) / self.f
        r = (torch.arange(self.H, dtype=torch.float64, device="cuda") + 0.5 - self.H / 2.0) / self.f
        return torch.stack([c[None].expand(self.H, -1), r[:, None].expand(-1, self.W),
                            torch.ones(self.H, self.W, dtype=torch.float64, device="cuda")], -1)

    def K(self):
        return b3d.intrinsics(self.f, self.f, self.W / 2.0, self.H / 2.0, self.H, self.W)

    def params(self):
        return b3d.score_params(SIGMA, P_OUT, VOLUME, self.window)

    def scene(self):
        s = b3d.Scene(b3d.Mesh(*self.mesh), self.K(), self.params())
        if len(self.statics):
            s.set_background([b3d.Mesh(*m) for m in self.statics], self.static_poses)
        s.set_observed(self.obs)
        return s

    def device_poses(self):
        return torch.as_tensor(self.poses, dtype=torch.float32, device="cuda").contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        worlds = [_World(case, seed, i) for i in range(case["scenes"])]
        return dict(kind=kind, batch=b3d.Batch([(w.scene(), w.device_poses()) for w in worlds], grad=True))
    w = _World(case, seed)
    poses = w.device_poses()
    if kind in ("score", "grad", "marginal"):
        scene = w.scene()
        if kind == "marginal":
            scene.set_noise_grid(*b3d.noise_grid_midpoints(*NOISE_GRID))
        return dict(kind=kind, scene=scene, poses=poses)
    if kind == "render":
        return dict(kind=kind, mesh=b3d.Mesh(*w.mesh), poses=poses, K=w.K())
    if kind in ("split", "split_grad"):
        rend, tri = _images(w)
        state = dict(kind=kind, obs=w.obs, rend=rend, params=w.params())
        if kind == "split_grad":
            dlogL = np.random.default_rng([seed, 1 << 20]).uniform(0.5, 1.5, w.N)
            state.update(mesh=b3d.Mesh(*w.mesh), poses=poses, K=w.K(), tri=tri,
                         dlogL=torch.as_tensor(dlogL, dtype=torch.float32, device="cuda"))
        return state
    if kind == "frame":
        return dict(kind=kind, scene=w.scene(), depth=w.depth, K=w.K(), poses=poses,
                    statics=[b3d.Mesh(*m) for m in w.statics], static_poses=w.static_poses)
    assert kind == "tracker"
    n0 = max(1, int(round((w.N / 10.0) ** (1.0 / 3.0))))
    n1 = max(1, n0 // 2)
    eye = np.eye(4)
    stages = [b3d.make_grid(eye, (0.03,) * 3, (n0,) * 3, n_rot=10, rot_max_angle=math.radians(8)),
              b3d.make_grid(eye, (0.0075,) * 3, (n1,) * 3, n_rot=20, rot_max_angle=math.radians(3))]
    m = 1 + case["others"]
    rng = np.random.default_rng([seed, 1 << 21])
    start = np.concatenate([w.truth, w.static_poses[:case["others"]]]).copy()
    start[:, :3, 3] += rng.uniform(-0.01, 0.01, (m, 3))
    tracker = b3d.Tracker([b3d.Mesh(*x) for x in [w.mesh] + w.statics[:case["others"]]], w.K(), w.params(), stages,
                          start, n_refine=2)
    tracker.frame(w.obs)  # the first frame records the graph that every later one replays
    return dict(kind=kind, tracker=tracker, obs=w.obs)


def run(state):
    kind = state["kind"]
    if kind in ("score", "grad"):
        return b3d.render_score(state["scene"], state["poses"], grad=kind == "grad")
    if kind == "marginal":
        return b3d.render_score_marginal(state["scene"], state["poses"], grid=True)
    if kind == "render":
        return b3d.render_batch(state["mesh"], state["poses"], state["K"])
    if kind == "split":
        return b3d.score(state["obs"], state["rend"], state["params"])
    if kind == "split_grad":
        dr, ds, dp = b3d.score_backward(state["obs"], state["rend"], state["params"], state["dlogL"])
        return dr, ds, dp, b3d.render_backward(state["mesh"], state["poses"], state["K"], state["tri"], dr)
    if kind == "frame":
        obs = b3d.unproject(state["depth"], state["K"])
        state["scene"].set_background(state["statics"], state["static_poses"])
        state["scene"].set_observed(obs)
        return obs, b3d.render_score(state["scene"], state["poses"])
    if kind == "tracker":
        state["tracker"].frame(state["obs"])
        return state["tracker"].poses()
    return state["batch"].run()


def work(case):
    """Counted once per pass: every vertex transformed (17) and triangle tested (12), the object's pixels filled (10),
    every pair of an observed pixel that sees it and a window pixel (12, with the adjoint 22) and the adjoint of its
    pixels (30); points, poses, meshes and results moved once."""
    bytes_, flops = 0.0, 0.0
    for i in range(case["scenes"]):
        k = i % 3 if case["scenes"] > 1 else 0
        scale = (1.0, 0.6, 1.6)[k]
        H, W = case["height"] * (1.0, 1.5, 0.8)[k], case["width"] * (1.0, 1.5, 0.8)[k]
        n, N = case["voxels"] * scale, case["hyps"] / scale
        kind = case["kind"]
        pixels = H * W if case["solid"] else min(H * W, math.pi * (_radius(n) * 0.9375 * W / DEPTH) ** 2)
        grad = kind in ("grad", "split_grad", "batch")
        pairs = pixels * case["window"] ** 2
        draw_ = 8 * n * 17 + 12 * n * 12 + 10 * pixels
        mesh = n * (8 * 12 + 12 * 12)
        if kind == "render":
            flops += N * draw_
            bytes_ += mesh + N * (64 + 16 * H * W)
        elif kind in ("split", "split_grad"):
            flops += N * pairs * (22 if grad else 12)
            bytes_ += 12 * H * W + N * (4 + 12 * H * W * (2 if grad else 1) + (4 * H * W + 64 + 24 if grad else 0))
        else:
            each = draw_ + pairs * (22 if grad else 12) + (30 * pixels if grad else 0)
            if kind == "marginal":
                each += pairs * 3 * (NOISE_GRID[1] - 1) + pixels * 6 * NOISE_GRID[1] * NOISE_GRID[2]
            if kind == "tracker":
                N = (1 + case["others"]) * (1.25 * N + 2)
            flops += N * each
            bytes_ += mesh + 12 * H * W + N * (68 + (32 if grad else 0))
            if kind == "frame":
                flops += case["others"] * (draw_ / 2) + 12 * H * W * case["window"] ** 2
                bytes_ += 16 * H * W
    return {"bytes": bytes_, "flops": flops}


# ---- the same in 64 bits, in plain torch -----------------------------------


def _chunks(T, w, N):
    step = max(1, int(1.6e7 / (3 * T + 4 * w.H * w.W)))
    return [slice(a, min(a + step, N)) for a in range(0, N, step)]


def _render(objects, w):
    """Depth [n,H,W] (0: empty) and triangle id (-1) of objects (verts, tris, poses [n,4,4]) in one image each: the
    nearest camera-facing triangle whose projection holds the pixel centre, ids counted over the objects in turn."""
    d = dict(dtype=torch.float64, device="cuda")
    n = len(objects[0][2])
    size = n * w.H * w.W
    hits, first = [], 0
    for verts, tris, poses in objects:
        v, P = torch.as_tensor(verts, **d), torch.as_tensor(poses, **d)
        t = torch.as_tensor(tris.astype(np.int64), device="cuda")
        c = v[None] @ P[:, :3, :3].transpose(1, 2).contiguous() + P[:, None, :3, 3]
        px = torch.stack([w.f * c[..., 0] / c[..., 2] + w.W / 2.0, w.f * c[..., 1] / c[..., 2] + w.H / 2.0], -1)
        c, px = c[:, t], px[:, t]  # [n, T, 3, 3], [n, T, 3, 2]
        normal = torch.linalg.cross(c[:, :, 1] - c[:, :, 0], c[:, :, 2] - c[:, :, 0])
        nc = (normal * c[:, :, 0]).sum(-1)
        lo = torch.ceil(px.amin(2) - 0.5).clamp(min=0)
        hi = torch.floor(px.amax(2) - 0.5)
        hi = torch.minimum(hi, torch.tensor([w.W - 1.0, w.H - 1.0], **d))
        keep = ((c[..., 2] > 0.01).all(2) & (nc < 0) & (hi >= lo).all(2)).nonzero(as_tuple=True)
        lo, hi, px, normal, nc = lo[keep].long(), hi[keep].long(), px[keep], normal[keep], nc[keep]
        span = hi - lo + 1
        count = span[:, 0] * span[:, 1]
        k = torch.repeat_interleave(torch.arange(len(count), device="cuda"), count)
        j = torch.arange(len(k), device="cuda") - (torch.cumsum(count, 0) - count)[k]
        row = torch.div(j, span[k, 0], rounding_mode="floor")
        x, y = lo[k, 0] + j - row * span[k, 0], lo[k, 1] + row
        u, r = x + 0.5, y + 0.5
        q = px[k]
        inside = torch.ones(len(k), dtype=torch.bool, device="cuda")
        for a, b in ((1, 2), (2, 0), (0, 1)):
            e = q[:, b] - q[:, a]
            inside &= ~(e[:, 0] * (r - q[:, a, 1]) - e[:, 1] * (u - q[:, a, 0]) > 0)
        k, x, y = k[inside], x[inside], y[inside]
        dx, dy = (x + 0.5 - w.W / 2.0) / w.f, (y + 0.5 - w.H / 2.0) / w.f
        z = nc[k] / (normal[k, 0] * dx + normal[k, 1] * dy + normal[k, 2])
        hits.append(((keep[0][k] * w.H + y) * w.W + x, z, keep[1][k] + first))
        first += len(tris)
    at, z, ids = (torch.cat(x) for x in zip(*hits))
    depth = torch.full((size,), math.inf, **d).scatter_reduce_(0, at, z, "amin")
    front = z == depth[at]
    tri = torch.full((size,), 1 << 40, dtype=torch.int64, device="cuda")
    tri.scatter_reduce_(0, at[front], ids[front], "amin")
    empty = torch.isinf(depth)
    return (torch.where(empty, 0.0, depth).view(n, w.H, w.W),
            torch.where(empty, -1, tri).view(n, w.H, w.W))


def _scene_images(w, part, behind):
    """Depth and id images of the hypotheses `part` before the static objects' depth image (or None)."""
    z, tri = _render([(*w.mesh, w.poses[part])], w)
    if behind is None:
        return z, tri
    hidden = (behind > 0) & ((z == 0) | (behind < z))
    return torch.where(hidden, behind, z), torch.where(hidden, -1, tri)


def _static_depth(w):
    return _render([(*m, p[None]) for m, p in zip(w.statics, w.static_poses)], w)[0] if w.statics else None


def _images(w):
    """FP32 point images and ids of the moving object alone."""
    rend = torch.empty((w.N, w.H, w.W, 3), dtype=torch.float32, device="cuda")
    tri = torch.empty((w.N, w.H, w.W), dtype=torch.int32, device="cuda")
    ray = w.rays()
    for s in _chunks(len(w.mesh[1]), w, w.N):
        z, t = _render([(*w.mesh, w.poses[s])], w)
        rend[s], tri[s] = z[..., None] * ray, t
    return rend, tri


def _shifts(w):
    h = w.window // 2
    return [(a, b) for a in range(-h, h + 1) for b in range(-h, h + 1)]


def _window(w, points, sigmas):
    """Sums over every valid observed pixel's window of exp(-D / 2 s^2) and of that times D, per deviation s:
    pixel rows and columns, [n, V] tensors S and T for each of `sigmas`."""
    r, c = (w.obs[..., 2] > 0).nonzero(as_tuple=True)
    o = w.obs[r, c].double()
    S = [torch.zeros(len(points), len(r), dtype=torch.float64, device="cuda") for _ in sigmas]
    T = [x.clone() for x in S]
    for a, b in _shifts(w):
        y, x = r + a, c + b
        ok = (y >= 0) & (y < w.H) & (x >= 0) & (x < w.W)
        q = points[:, y.clamp(0, w.H - 1), x.clamp(0, w.W - 1)]
        D = ((o - q) ** 2).sum(-1)
        ok = ok & (q[..., 2] > 0)
        for k, s in enumerate(sigmas):
            e = torch.where(ok, torch.exp(-D / (2 * s * s)), 0.0)
            S[k] += e
            T[k] += e * D
    return r, c, S, T


def _scores(w, points):
    """logL, its derivatives by sigma and p_out, and the weight image b / L_i."""
    s, p = float(np.float32(SIGMA)), float(np.float32(P_OUT))
    norm = (2 * math.pi * s * s) ** -1.5 / (w.H * w.W)
    r, c, (S,), (T,) = _window(w, points, [s])
    L = p / VOLUME + (1 - p) * norm * S
    ds = ((1 - p) * norm * (T / s ** 3 - 3 * S / s) / L).sum(1)
    dp = ((1 / VOLUME - norm * S) / L).sum(1)
    weight = torch.zeros(points.shape[:3], dtype=torch.float64, device="cuda")
    weight[:, r, c] = (1 - p) * norm / L
    return torch.log(L).sum(1), ds, dp, weight


def _point_gradients(w, points, weight, at):
    """d logL / d q of the rendered pixels at = (n, row, column)."""
    s = float(np.float32(SIGMA))
    n, r, c = at
    q = points[n, r, c]
    g = torch.zeros_like(q)
    obs = w.obs.double()
    for a, b in _shifts(w):
        y, x = r + a, c + b
        ok = (y >= 0) & (y < w.H) & (x >= 0) & (x < w.W)
        y, x = y.clamp(0, w.H - 1), x.clamp(0, w.W - 1)
        e = obs[y, x] - q
        k = torch.where(ok, weight[n, y, x] * torch.exp(-(e * e).sum(-1) / (2 * s * s)), 0.0)
        g += k[:, None] * e
    return g / (s * s)


def _pose_gradients(w, poses, points, tri, g, at):
    """d logL / d (dt, dw) from the point gradients g of the object's pixels, visibility held."""
    n, r, c = at
    P = torch.as_tensor(poses, dtype=torch.float64, device="cuda")
    v = torch.as_tensor(w.mesh[0], dtype=torch.float64, device="cuda")
    t = torch.as_tensor(w.mesh[1].astype(np.int64), device="cuda")[tri[n, r, c].long()]
    normal = torch.linalg.cross(v[t[:, 1]] - v[t[:, 0]], v[t[:, 2]] - v[t[:, 0]])
    normal = (P[n, :3, :3] * normal[:, None]).sum(-1)
    ray = w.rays()[r, c]
    s = (g * ray).sum(-1) / (normal * ray).sum(-1)
    turn = torch.linalg.cross(normal, P[n, :3, 3] - points[n, r, c])
    out = torch.zeros(len(P), 6, dtype=torch.float64, device="cuda")
    return out.index_add_(0, n, s[:, None] * torch.cat([normal, turn], 1))


def _exact_fused(w, grad):
    logL, G = [], []
    ray, T, behind = w.rays(), len(w.mesh[1]), _static_depth(w)
    for s in _chunks(T, w, w.N):
        z, tri = _scene_images(w, s, behind)
        points = z[..., None] * ray
        l, ds, dp, weight = _scores(w, points)
        logL.append(l)
        if grad:
            at = (tri >= 0).nonzero(as_tuple=True)
            g = _pose_gradients(w, w.poses[s], points, tri, _point_gradients(w, points, weight, at), at)
            G.append(torch.cat([g, ds[:, None], dp[:, None]], 1))
    return (torch.cat(logL), torch.cat(G)) if grad else torch.cat(logL)


def _exact_marginal(w):
    top, A, B = NOISE_GRID
    sigmas = [float(np.float32(top * (a + 0.5) / A)) for a in range(A)]
    probs = [float(np.float32((b + 0.5) / B)) for b in range(B)]
    ray, grid, behind = w.rays(), [], _static_depth(w)
    for s in _chunks(len(w.mesh[1]), w, w.N):
        z, _ = _scene_images(w, s, behind)
        _, _, S, _ = _window(w, z[..., None] * ray, sigmas)
        rows = []
        for sg, Sa in zip(sigmas, S):
            norm = (2 * math.pi * sg * sg) ** -1.5 / (w.H * w.W)
            rows.append(torch.stack([torch.log(p / VOLUME + (1 - p) * norm * Sa).sum(1) for p in probs], 1))
        grid.append(torch.stack(rows, 1))
    grid = torch.cat(grid)
    return torch.logsumexp(grid.flatten(1), 1) - math.log(A * B), grid


def exact(case, seed):
    kind = case["kind"]
    if kind == "tracker":  # a chain of searches: each stage's best hypothesis is the next one's centre
        return None
    if kind == "batch":
        both = [_exact_fused(_World(case, seed, i), True) for i in range(case["scenes"])]
        return [x for x, _ in both], [x for _, x in both]
    w = _World(case, seed)
    if kind in ("score", "grad"):
        return _exact_fused(w, kind == "grad")
    if kind == "marginal":
        return _exact_marginal(w)
    if kind == "frame":
        return (w.depth.double()[..., None] * w.rays(), _exact_fused(w, False))
    ray, parts = w.rays(), []
    if kind == "render":
        for s in _chunks(len(w.mesh[1]), w, w.N):
            parts.append(_render([(*w.mesh, w.poses[s])], w)[0][..., None] * ray)
        return torch.cat(parts), None
    rend, tri = _images(w)
    if kind == "split":
        return torch.cat([_scores(w, rend[s].double())[0] for s in _chunks(1, w, w.N)])
    dlogL = torch.as_tensor(np.random.default_rng([seed, 1 << 20]).uniform(0.5, 1.5, w.N), dtype=torch.float32,
                            device="cuda").double()
    for s in _chunks(1, w, w.N):
        points, k = rend[s].double(), dlogL[s]
        _, ds, dp, weight = _scores(w, points)
        at = (points[..., 2] > 0).nonzero(as_tuple=True)
        g = _point_gradients(w, points, weight, at) * k[at[0], None]
        dr = torch.zeros_like(points)
        dr[at] = g
        parts.append((dr, ds * k, dp * k, _pose_gradients(w, w.poses[s], points, tri[s], g, at)))
    return tuple(torch.cat(x) for x in zip(*parts))
