"""Each route that a launch can take through the kernels, at the sizes where
it changes: against the FP64 oracle, or against another route that has to give
the same.  Bars as in test_gpu_parity.py."""

import ctypes

import numpy as np
import pytest
import torch

import oracle
from workloads import Camera, box_mesh, random_poses, voxel_blob, voxel_mesh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def b3d():
    import paper_2312_08715_amd as b

    assert torch.cuda.is_available(), "GPU tests need a device"
    b.load_library()
    return b


def f32(a):
    return np.asarray(a, dtype=np.float32).astype(np.float64)


def dev(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def joined(*meshes):
    """One mesh of several (verts, tris)."""
    v, t, n = [], [], 0
    for a, b in meshes:
        v.append(a)
        t.append(b + n)
        n += len(a)
    return f32(np.concatenate(v)), np.concatenate(t).astype(np.int32)


def turned(mesh, yaw):
    c, s = np.cos(yaw), np.sin(yaw)
    return mesh[0] @ np.array([[c, s, 0.0], [-s, c, 0.0], [0.0, 0.0, 1.0]]), mesh[1]


# a voxel face of 1 cm projects to f / 100 / depth pixels: below one pixel, two,
# either side of the largest box walked in step (16), and beyond the image; the
# last depth puts voxels in front of and behind the near plane
@pytest.mark.parametrize("f,depth", [(30.0, 0.6), (120.0, 0.6), (900.0, 0.6), (980.0, 0.6), (2500.0, 0.4), (60.0, 0.03)])
@pytest.mark.parametrize("kind", ["blob", "turned", "mixed"])
def test_render_of_equal_voxels_matches_oracle(b3d, f, depth, kind):
    rng = np.random.default_rng(int(f) + len(kind))
    blob = voxel_mesh(voxel_blob(60, rng, radius=0.04))
    if kind == "turned":  # edges that are equal only up to rounding
        blob = turned(blob, 0.7)
    if kind == "mixed":  # other faces of the same orientations: a slab, and voxels of another size
        c = voxel_blob(20, rng, radius=0.03)
        blob = joined(blob, box_mesh((0.3, 0.2, 0.004), (0.0, 0.0, -0.06)),
                      (voxel_mesh(c, 0.006)[0] + [0.0, 0.08, 0.0], voxel_mesh(c)[1]))
    verts, tris = f32(blob[0]), blob[1]
    cam = Camera(f, f, 33.3, 21.7, 45, 66)
    P = f32(random_poses(rng, 24, depth, 0.02))
    K = b3d.intrinsics_of(cam)
    xyz, tri = b3d.render_batch(b3d.Mesh(verts, tris), dev(P), K)
    d, ids = oracle.render([(verts, tris, P)], cam)
    same = tri.cpu().numpy() == ids
    assert same.mean() >= 0.999, f"ids equal on {same.mean():.5f}"
    z = xyz[..., 2].cpu().numpy()
    assert np.abs(z - d)[same & (ids >= 0)].max(initial=0.0) <= 1e-5
    assert np.all(z[same & (ids < 0)] == 0.0)


def scored(b3d, scene, P, grad):
    L = b3d.render_score(scene, P, grad=grad)
    return [x.cpu().numpy() for x in (L if grad else (L,))]


# blocks of 1,024, 512 and 256 threads (up to 256, 512 and more hypotheses), an
# object within the 256-thread block's depth buffer and beyond it (drawn by a
# second launch: more pixels than 24,000, or than 56,000) and a caller's own
# tile of one band of two rows: the same values whichever way
@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("H,W,window", [(48, 64, 3), (151, 200, 5), (231, 300, 7)])
def test_block_sizes_and_second_launch_give_the_same(b3d, H, W, window, grad):
    rng = np.random.default_rng(H)
    verts, tris = voxel_mesh(voxel_blob(400, rng))
    f = 0.94 * W
    cam = Camera(f, f, W / 2 + 0.2, H / 2 - 0.3, H, W)
    K = b3d.intrinsics_of(cam)
    P = f32(random_poses(rng, 600, 0.8, 0.03))
    P[::7, 2, 3] = 2.5  # far ones fit the small block
    P[5, :3, 3] = 0.0, 0.0, 0.05  # around the camera: every row of the image, bands in any block
    P = dev(P)
    scene = b3d.Scene(b3d.Mesh(f32(verts), tris), K, b3d.score_params(0.004, 0.05, 1.0, window))
    xyz, _ = b3d.render_batch(scene.mesh, P[1:2].contiguous(), K)
    noise = torch.as_tensor(rng.normal(0.0, 0.002, (H, W, 1)), dtype=torch.float32, device="cuda")
    scene.set_observed((xyz[0] * (1.0 + noise)).contiguous())
    whole = scored(b3d, scene, P, grad)
    for n in (1, 256, 257, 512, 513):
        for a, b in zip(scored(b3d, scene, P[:n].contiguous(), grad), whole):
            np.testing.assert_array_equal(a, b[:n])
    scene.set_tile(scene.tile_limits()[0])
    for n in (40, 600):
        for a, b in zip(scored(b3d, scene, P[:n].contiguous(), grad), whole):
            np.testing.assert_array_equal(a, b[:n])


@pytest.mark.parametrize("grad", [False, True])
def test_batch_of_large_and_small_images_equals_per_scene_calls(b3d, grad):
    rng = np.random.default_rng(3)
    items = []
    for H, W, n in [(48, 64, 70), (180, 240, 90), (231, 300, 30), (60, 100, 1), (151, 200, 11)]:
        verts, tris = voxel_mesh(voxel_blob(300, rng))
        cam = Camera(0.94 * W, 0.94 * W, W / 2, H / 2, H, W)
        P = f32(random_poses(rng, n, 0.8, 0.03))
        P[::5, 2, 3] = 2.0
        scene = b3d.Scene(b3d.Mesh(f32(verts), tris), b3d.intrinsics_of(cam), b3d.score_params(0.004, 0.05, 1.0, 5))
        xyz, _ = b3d.render_batch(scene.mesh, dev(P[:1]), b3d.intrinsics_of(cam))
        scene.set_observed(xyz[0].contiguous())
        items.append((scene, dev(P[:n])))
    batch = b3d.Batch(items, grad=grad)
    out = batch.run()
    logL, g = out if grad else (out, None)
    for i, (scene, P) in enumerate(items):
        one = scored(b3d, scene, P, grad)
        np.testing.assert_array_equal(logL[i].cpu().numpy(), one[0])
        if grad:
            np.testing.assert_array_equal(g[i].cpu().numpy(), one[1])


# rows and columns either side of a wave, a block and a 16-row run of the
# tables' sums; nine static objects are two launches; triangles of a few pixels
# and of the whole image.  The pose is behind the camera, so a result is the
# background's sum over the whole image: logL and its derivatives within 1e-6
# of the L1 mass of the oracle's terms (single precision rounds a sum by 6e-8).
# The static objects' render decides pixel centres on an edge in single
# precision, so with them logL may differ by two such pixels' windows
@pytest.mark.parametrize("H,W", [(1, 63), (15, 64), (16, 65), (31, 255), (17, 256), (33, 257)])
@pytest.mark.parametrize("statics", [0, 9])
def test_background_sums_match_oracle(b3d, H, W, statics):
    rng = np.random.default_rng(H * W + statics)
    f = 0.9 * max(H, W)
    cam = Camera(f, f, W / 2 + 0.37, H / 2 - 0.21, H, W)
    K = b3d.intrinsics_of(cam)
    quad = f32([[-2, -2, 0], [2, -2, 0], [2, 2, 0], [-2, 2, 0]]), np.array([[0, 2, 1], [0, 3, 2]], np.int32)
    meshes = [quad] + [voxel_mesh(voxel_blob(12, rng, radius=0.04)) for _ in range(8)]
    meshes = [(f32(v), t) for v, t in meshes][:statics]
    poses = f32(random_poses(rng, 9, 0.8, 0.1))
    poses[0] = np.eye(4)
    poses[0, 2, 3] = 1.2
    mesh = voxel_mesh(voxel_blob(5, rng, radius=0.03))
    rays = oracle.unproject(np.ones((1, H, W)), cam)[0]
    if statics:
        d, _ = oracle.render([(v, t, p[None]) for (v, t), p in zip(meshes, poses)], cam)
        z = np.where(d[0] > 0, d[0] + rng.normal(0, 0.002, (H, W)), 0.0)
    else:
        d = np.zeros((1, H, W))
        z = rng.uniform(0.5, 1.0, (H, W))
    z[rng.random((H, W)) < 0.1] = 0.0
    obs = f32(z[..., None] * rays)
    scene = b3d.Scene(b3d.Mesh(f32(mesh[0]), mesh[1]), K, b3d.score_params(0.004, 0.05, 1.0, 3))
    if statics:
        scene.set_background([b3d.Mesh(*m) for m in meshes], poses[:statics])
    scene.set_observed(dev(obs))
    P = np.eye(4)[None].copy()
    P[0, 2, 3] = -1.0
    L, g = scored(b3d, scene, dev(P), True)
    sg, po = float(np.float32(0.004)), float(np.float32(0.05))
    pts = oracle.unproject(d, cam)
    L64, l1 = oracle.score(obs, pts, sg, po, 1.0, 3)
    _, ds, dp = oracle.score_grad(obs, pts, sg, po, 1.0, 3)
    slack = 0.0 if not statics else 9 * 12.0 * 2
    assert abs(L[0] - L64[0]) <= 1e-6 * l1[0] + slack, (L[0], L64[0])
    if not statics:
        assert abs(g[0, 6] - ds[0]) <= 1e-6 * abs(ds[0]) + 1e-4
        assert abs(g[0, 7] - dp[0]) <= 1e-6 * abs(dp[0]) + 1e-4
    assert np.all(g[0, :6] == 0.0)


# the noise grid's registers hold 16 // A grid points per deviation up to four
# deviations (LDS beyond); block sizes and the second launch as for the score
@pytest.mark.parametrize("A,B", [(1, 16), (2, 8), (3, 5), (4, 4), (4, 1), (5, 3), (8, 2)])
@pytest.mark.parametrize("H,W", [(48, 64), (151, 200)])
def test_noise_grid_block_sizes_give_the_same_and_match_single_points(b3d, H, W, A, B):
    rng = np.random.default_rng(A * 31 + B)
    verts, tris = voxel_mesh(voxel_blob(200, rng))
    cam = Camera(0.94 * W, 0.94 * W, W / 2 + 0.2, H / 2 - 0.3, H, W)
    K = b3d.intrinsics_of(cam)
    P = f32(random_poses(rng, 520, 0.8, 0.03))
    P[::7, 2, 3] = 2.5
    P = dev(P)
    scene = b3d.Scene(b3d.Mesh(f32(verts), tris), K, b3d.score_params(0.004, 0.05, 1.0, 5))
    xyz, _ = b3d.render_batch(scene.mesh, P[1:2].contiguous(), K)
    obs = xyz[0].clone()
    obs[::3, ::2] = 0.0
    scene.set_observed(obs.contiguous())
    sig, po = b3d.noise_grid_midpoints(0.012, A, B)
    scene.set_noise_grid(sig, po)
    marg, grid = b3d.render_score_marginal(scene, P, grid=True)
    for n in (1, 256, 300, 512):
        m, g = b3d.render_score_marginal(scene, P[:n].contiguous(), grid=True)
        assert torch.equal(m, marg[:n]) and torch.equal(g, grid[:n])
    assert torch.equal(b3d.render_score_marginal(scene, P), marg)
    # each grid point is the plain score at its parameters; the two kernels' terms
    # ln(a + b S) differ by single-precision roundings of each pixel's term: 1e-5 of logL's size
    for a, b in ((0, 0), (A - 1, B - 1)):
        scene.set_params(b3d.score_params(float(sig[a]), float(po[b]), 1.0, 5))
        one = b3d.render_score(scene, P)
        assert (one - grid[:, a, b]).abs().max() <= 1e-5 * one.abs().max()
    ref = torch.logsumexp(grid.double().flatten(1), 1) - np.log(A * B)
    assert (marg - ref).abs().max() <= 1e-6 * ref.abs().max() + 1e-3


# the smallest images and tiles: the block's sums need more LDS than its tile
@pytest.mark.parametrize("H,W,window", [(1, 1, 1), (2, 3, 3), (5, 4, 1)])
@pytest.mark.parametrize("N", [1, 300, 600])
def test_smallest_images_match_oracle(b3d, H, W, window, N):
    rng = np.random.default_rng(N)
    verts, tris = voxel_mesh(voxel_blob(20, rng, radius=0.04))
    verts = f32(verts)
    cam = Camera(4.0, 4.0, W / 2 + 0.03, H / 2 - 0.04, H, W)
    P = f32(random_poses(rng, N, 0.2, 0.01))
    d, ids = oracle.render([(verts, tris, P)], cam)
    obs = f32(oracle.unproject(np.where(d[:1] > 0, d[:1], 0.2), cam)[0])
    scene = b3d.Scene(b3d.Mesh(verts, tris), b3d.intrinsics_of(cam), b3d.score_params(0.02, 0.1, 1.0, window))
    scene.set_observed(dev(obs))
    L, g = scored(b3d, scene, dev(P), True)
    L64, l1 = oracle.score(obs, oracle.unproject(d, cam), float(np.float32(0.02)), float(np.float32(0.1)), 1.0, window)
    assert np.all(np.abs(L - L64) <= 1e-4 * l1)
    assert np.array_equal(scored(b3d, scene, dev(P), False)[0], L)
    scene.set_noise_grid(*b3d.noise_grid_midpoints(0.03, 4, 4))
    marg, grid = b3d.render_score_marginal(scene, dev(P), grid=True)
    ref = torch.logsumexp(grid.double().flatten(1), 1) - np.log(16)
    assert (marg - ref).abs().max() <= 1e-5 * ref.abs().max() + 1e-5
    scene.set_tile(scene.tile_limits()[0])
    assert np.array_equal(scored(b3d, scene, dev(P), True)[1], g)


# the adjoint over the rectangle of drawn pixels: word and single-float images
# (a width of 4 k or not), an empty image, one pixel, a rectangle in one band
# and in several, every compiled window and the general one
@pytest.mark.parametrize("window", [1, 3, 5, 7, 9])
@pytest.mark.parametrize("H,W", [(24, 32), (37, 41), (60, 200)])
def test_score_adjoint_over_the_drawn_rectangle_matches_oracle(b3d, H, W, window):
    rng = np.random.default_rng(H + window)
    cam = Camera(0.9 * W, 0.9 * W, W / 2, H / 2, H, W)
    rays = oracle.unproject(np.ones((1, H, W)), cam)[0]
    z = np.zeros((5, H, W))
    z[1, H // 2, W - 1] = 0.8  # one pixel, in the last column
    z[2, 3:15, 5:19] = 0.8 + rng.normal(0, 0.003, (12, 14))
    z[3] = 0.8 + rng.normal(0, 0.003, (H, W))  # the whole image
    z[4, 0, 0] = z[4, H - 1, W - 1] = 0.8  # two corners: a rectangle of empty pixels
    z[3, ::3, ::4] = 0.0
    rend = f32(z[..., None] * rays)
    zo = np.where(rng.random((H, W)) < 0.2, 0.0, 0.8 + rng.normal(0, 0.003, (H, W)))
    obs = f32(zo[..., None] * rays)
    dl = f32(rng.uniform(-1.0, 2.0, 5))
    sg, po = float(np.float32(0.005)), float(np.float32(0.1))
    dr, ds, dp = b3d.score_backward(dev(obs), dev(rend), b3d.score_params(sg, po, 1.0, window), dev(dl))
    r64, s64, p64 = oracle.score_grad(obs, rend, sg, po, 1.0, window)
    k = dl[:, None, None, None]
    scale = np.abs(r64 * k).max()
    assert np.abs(dr.cpu().numpy() - r64 * k).max() <= 1e-5 * scale
    for got, want in ((ds, s64 * dl), (dp, p64 * dl)):
        assert np.all(np.abs(got.cpu().numpy() - want) <= 1e-5 * np.abs(want).max())
    none = b3d.score_backward(dev(obs), dev(rend), b3d.score_params(sg, po, 1.0, window), dev(dl), want_rendered=False)
    assert torch.equal(none[1], ds) and torch.equal(none[2], dp)
    # odd starts of the images in memory take the single-float route: the same values
    buf = torch.zeros(rend.size + 1, dtype=torch.float32, device="cuda")
    buf[1:] = dev(rend).reshape(-1)
    odd = b3d.score_backward(dev(obs), buf[1:].view(rend.shape), b3d.score_params(sg, po, 1.0, window), dev(dl))
    assert all(torch.equal(a, b) for a, b in zip(odd, (dr, ds, dp)))


# ids read four at a time or one by one, ids of no triangle among them
@pytest.mark.parametrize("H,W", [(16, 20), (17, 21), (64, 64)])
def test_pose_adjoint_reads_ids_either_way(b3d, H, W):
    rng = np.random.default_rng(W)
    verts, tris = voxel_mesh(voxel_blob(40, rng, radius=0.04))
    verts = f32(verts)
    cam = Camera(1.5 * W, 1.5 * W, W / 2 + 0.1, H / 2, H, W)
    P = f32(random_poses(rng, 7, 0.3, 0.01))
    d, ids = oracle.render([(verts, tris, P)], cam)
    g = f32(rng.normal(size=(7, H, W, 3)))
    want = oracle.render_grad(verts, tris, P, cam, ids, d, g)
    t = torch.as_tensor(ids.astype(np.int32), device="cuda")
    t[t < 0] = torch.tensor(-7, dtype=torch.int32, device="cuda")
    t[0, 0, 0] = len(tris) + 5 if ids[0, 0, 0] < 0 else t[0, 0, 0]
    K = b3d.intrinsics_of(cam)
    out = b3d.render_backward(b3d.Mesh(verts, tris), dev(P), K, t.contiguous(), dev(g)).cpu().numpy()
    assert np.all(np.linalg.norm(out - want, axis=1) <= 1e-3 * np.linalg.norm(want, axis=1) + 1e-6)
    buf = torch.zeros(t.numel() + 1, dtype=torch.int32, device="cuda")
    buf[1:] = t.reshape(-1)
    odd = b3d.render_backward(b3d.Mesh(verts, tris), dev(P), K, buf[1:].view(t.shape), dev(g)).cpu().numpy()
    assert np.all(np.abs(odd - out) <= 1e-6 * np.abs(out).max())


# point images by blocks of each size and by the second launch, rows of whole
# 16-byte words or not, with and without ids: the same images
@pytest.mark.parametrize("H,W", [(48, 64), (151, 201), (150, 200), (231, 300)])
def test_render_block_sizes_and_second_launch_give_the_same(b3d, H, W):
    rng = np.random.default_rng(W)
    verts, tris = voxel_mesh(voxel_blob(400, rng))
    cam = Camera(0.94 * W, 0.94 * W, W / 2 + 0.2, H / 2 - 0.3, H, W)
    K, mesh = b3d.intrinsics_of(cam), b3d.Mesh(f32(verts), tris)
    P = f32(random_poses(rng, 530, 0.8, 0.03))
    P[::7, 2, 3] = 2.5
    P[5, :3, 3] = 0.0, 0.0, 0.05
    P[6, 2, 3] = -1.0  # behind the camera
    P = dev(P)
    xyz, tri = b3d.render_batch(mesh, P, K)
    assert bool((tri[6] == -1).all()) and bool((xyz[6] == 0).all()) and bool(torch.isfinite(xyz).all())
    for n in (1, 256, 257, 512):
        x, t = b3d.render_batch(mesh, P[:n].contiguous(), K)
        assert torch.equal(x, xyz[:n]) and torch.equal(t, tri[:n])
    assert torch.equal(b3d.render_batch(mesh, P, K, want_tri=False)[0], xyz)
    sel = [0, 1, 5, 7, 300]
    d, ids = oracle.render([(f32(verts), tris, P[sel].cpu().numpy().astype(np.float64))], cam)
    same = tri[sel].cpu().numpy() == ids
    assert same.mean() >= 0.999
    assert np.abs(xyz[sel][..., 2].cpu().numpy() - d)[same & (ids >= 0)].max() <= 1e-5


# the windows that are unrolled (up to 7 x 7) and looped over (from 9 x 9), of
# an object across the image border
@pytest.mark.parametrize("window", [5, 7, 9, 13])
@pytest.mark.parametrize("H,W", [(24, 32), (61, 75)])
def test_wide_windows_match_oracle(b3d, H, W, window):
    rng = np.random.default_rng(H + window)
    verts, tris = voxel_mesh(voxel_blob(60, rng, radius=0.06))
    verts = f32(verts)
    cam = Camera(W, W, W / 2 + 0.03, H / 2 - 0.04, H, W)
    P = random_poses(rng, 6, 0.5, 0.02)
    P[::2, 0, 3] += 0.22  # across the right edge
    P = f32(P)
    d, _ = oracle.render([(verts, tris, P)], cam)
    zo = np.where(d[0] > 0, d[0], 0.52) + rng.normal(0, 0.002, (H, W))
    obs = f32(oracle.unproject(np.where(rng.random((H, W)) < 0.2, 0.0, zo)[None], cam)[0])
    sg, po = float(np.float32(0.01)), float(np.float32(0.1))
    scene = b3d.Scene(b3d.Mesh(verts, tris), b3d.intrinsics_of(cam), b3d.score_params(sg, po, 1.0, window))
    scene.set_observed(dev(obs))
    L, g = scored(b3d, scene, dev(P), True)
    L64, l1 = oracle.score(obs, oracle.unproject(d, cam), sg, po, 1.0, window)
    assert np.all(np.abs(L - L64) <= 1e-4 * l1)
    assert np.array_equal(scored(b3d, scene, dev(P), False)[0], L)
    # the same through the point images of the kernels' own render
    xyz, _ = b3d.render_batch(scene.mesh, dev(P), b3d.intrinsics_of(cam))
    np.testing.assert_allclose(b3d.score(dev(obs), xyz, scene.params).cpu().numpy(), L, rtol=0, atol=1e-5 * l1.max())
    _, ds, dp = b3d.score_backward(dev(obs), xyz, scene.params, torch.ones(6, device="cuda"))
    for k, want in ((6, ds), (7, dp)):
        want = want.cpu().numpy()
        inside = np.abs(want).max()
        assert np.abs(g[:, k] - want).max() <= 1e-4 * inside
    scene.set_noise_grid(np.array([0.5, 1.0, 2.0]) * sg, [po, 0.4])
    _, grid = b3d.render_score_marginal(scene, dev(P), grid=True)
    np.testing.assert_allclose(grid[:, 1, 0].cpu().numpy(), L, rtol=0, atol=1e-5 * l1.max())


# observed points that are no points: without depth (whatever x and y hold) they
# count for nothing; at infinity, where no window reaches the object, logL and
# the pose's gradient are those of a far point, in every window that skips
# what is not drawn
@pytest.mark.parametrize("window", [7, 9])
def test_points_at_infinity_beside_the_object(b3d, window):
    H, W = 40, 56
    rng = np.random.default_rng(window)
    verts, tris = voxel_mesh(voxel_blob(60, rng, radius=0.04))
    cam = Camera(W, W, W / 2 + 0.03, H / 2 - 0.04, H, W)
    K = b3d.intrinsics_of(cam)
    P = f32(random_poses(rng, 3, 0.5, 0.0))
    scene = b3d.Scene(b3d.Mesh(f32(verts), tris), K, b3d.score_params(0.01, 0.1, 1.0, window))
    xyz, _ = b3d.render_batch(scene.mesh, dev(P), K)
    z = xyz[..., 2].cpu().numpy()
    near = np.zeros((H, W), bool)  # pixels whose window sees something drawn in any of the images
    h = window // 2
    for r, c in zip(*np.nonzero((z > 0).any(0))):
        near[max(r - h, 0) : r + h + 1, max(c - h, 0) : c + h + 1] = True
    obs = xyz[0].cpu().numpy().copy()
    far = obs.copy()
    hole = (z[0] > 0) & (rng.random((H, W)) < 0.2)
    far[hole] = 0.0
    obs[hole] = [np.nan, np.inf, 0.0]
    far[~near], obs[~near] = [0.0, 0.0, 50.0], [np.nan, np.inf, np.inf]
    assert near.any() and (~near).any()
    out = []
    for image in (far, obs):
        scene.set_observed(dev(image))
        out.append(scored(b3d, scene, dev(P), True))
    np.testing.assert_allclose(out[1][0], out[0][0], rtol=1e-5)
    np.testing.assert_allclose(out[1][1][:, :6], out[0][1][:, :6], rtol=1e-4, atol=1e-4 * np.abs(out[0][1]).max())


# the one-workgroup refinement reads, in one thread, a gradient that threads of
# several waves wrote: every step's has to be that step's.  Fewer and more poses
# than fit the chip at once, an image drawn in bands of rows, one step and
# several; against the same steps launched in turn, whose arithmetic it shares
# (bars as in test_refine_poses_equals_score_and_adam_launched_in_turn), and
# against itself
@pytest.mark.parametrize("H,W,N", [(48, 64, 1), (48, 64, 1500), (120, 160, 700), (150, 200, 60)])
def test_refinement_steps_use_their_own_gradient(b3d, H, W, N):
    rng = np.random.default_rng(N)
    verts, tris = voxel_mesh(voxel_blob(150, rng, radius=0.06))
    cam = Camera(0.94 * W, 0.94 * W, W / 2 + 0.2, H / 2 - 0.3, H, W)
    K = b3d.intrinsics_of(cam)
    P = f32(random_poses(rng, N, 0.6, 0.02))
    scene = b3d.Scene(b3d.Mesh(f32(verts), tris), K, b3d.score_params(0.01, 0.1, 1.0, 3))
    xyz, _ = b3d.render_batch(scene.mesh, dev(P[:1]), K)
    scene.set_observed(xyz[0].contiguous())
    args = (1e-3, 1e-2, 0.9, 0.999, 1e-8)
    for steps in (1, 4):
        A = [dev(P) for _ in range(3)]
        for a in A:
            b3d.refine_poses(scene, a, steps, *args)
        assert torch.equal(A[0], A[1]) and torch.equal(A[0], A[2])
        B, state = dev(P), torch.zeros((N, 12), dtype=torch.float32, device="cuda")
        for it in range(1, steps + 1):
            _, g = b3d.render_score(scene, B, grad=True)
            b3d.adam_pose_step(B, g, state, it, *args)
        assert (A[0] - B).abs().max() <= 1e-6
        assert (B[:, :3, :3] - dev(P)[:, :3, :3]).abs().amax((1, 2)).min() > 1e-3  # a rotation of every pose


# pixel centres on the edges of many faces: more of them than the exact test's
# queue holds, in blocks of each size and in a band of two rows, for a mesh
# without and with large faces (a shorter queue).  The exact test is the
# oracle's, so what is covered is the same at every pixel; a centre on a shared
# edge may go to either face of the same depth
@pytest.mark.parametrize("px,large", [(2, False), (8, False), (8, True), (12, False)])
def test_centres_on_many_edges_are_decided_exactly(b3d, px, large):
    H, W, pitch = 240, 320, 0.01
    nx, ny = min(280 // px, 100), min(200 // px, 80)
    c = np.stack(np.meshgrid(np.arange(nx) - nx / 2 + 0.5, np.arange(ny) - ny / 2 + 0.5, [0.0], indexing="ij"), -1)
    mesh = voxel_mesh(c.reshape(-1, 3) * pitch, pitch)
    if large:
        mesh = joined(mesh, box_mesh((nx * pitch * 0.9, ny * pitch * 0.5, 0.02), (0.0, 0.0, -0.015)))
    verts, tris = f32(mesh[0]), mesh[1]
    f = px / pitch
    cam = Camera(f, f, W / 2, H / 2, H, W)
    P = np.tile(np.eye(4), (3, 1, 1))  # the front faces at depth 1, their edges on the centres, between, on one axis' centres
    P[:, 2, 3] = 1.0 + pitch / 2
    P[:, 0, 3], P[:, 1, 3] = np.array([0.5, 0.0, 0.3]) / f, np.array([0.5, 0.0, 0.5]) / f
    P = f32(P)
    K, m = b3d.intrinsics_of(cam), b3d.Mesh(verts, tris)
    d, ids = oracle.render([(verts, tris, P)], cam)
    images = []
    for n in (1, 100, 200):
        xyz, tri = b3d.render_batch(m, dev(np.tile(P, (n, 1, 1))), K)
        for k in (0, n - 1):
            z = xyz[3 * k : 3 * k + 3, ..., 2].cpu().numpy()
            assert np.array_equal(z > 0, d > 0), [int(((z > 0) != (d > 0))[i].sum()) for i in range(3)]
            assert np.abs(z - d).max() <= 1e-5
        images.append(tri[:3])
    assert torch.equal(images[0], images[1]) and torch.equal(images[0], images[2])
    sg, po = float(np.float32(0.01)), float(np.float32(0.1))
    scene = b3d.Scene(m, K, b3d.score_params(sg, po, 1.0, 3))
    obs = f32(oracle.unproject(np.where(d[:1] > 0, 1.002, 0.0), cam)[0])
    scene.set_observed(dev(obs))
    L64, l1 = oracle.score(obs, oracle.unproject(d, cam), sg, po, 1.0, 3)
    for n in (1, 100, 200):
        L = scored(b3d, scene, dev(np.tile(P, (n, 1, 1))), False)[0]
        assert np.all(np.abs(L[:3] - L64) <= 1e-4 * l1) and np.array_equal(L, np.tile(L[:3], n))
    scene.set_tile(scene.tile_limits()[0])
    L = scored(b3d, scene, dev(np.tile(P, (200, 1, 1))), False)[0]
    assert np.all(np.abs(L[:3] - L64) <= 1e-4 * l1) and np.array_equal(L, np.tile(L[:3], 200))


# more triangles than the queue holds at one pixel: a fan around a vertex that
# projects onto its centre
@pytest.mark.parametrize("N", [1, 600])
def test_more_triangles_at_one_centre_than_the_queue_holds(b3d, N):
    n, H, W = 2500, 24, 32
    a = np.arange(n) * (2 * np.pi / n)
    verts = f32(np.concatenate([[[0.0, 0.0, 0.0]], np.stack([np.cos(a), np.sin(a), 0.0 * a], -1) * 0.25]))
    k = np.arange(n)
    tris = np.stack([0 * k, 1 + (k + 1) % n, 1 + k], -1).astype(np.int32)  # seen from -z
    cam = Camera(32.0, 32.0, W / 2 + 0.5, H / 2 + 0.5, H, W)
    P = np.eye(4)[None].copy()
    P[0, 2, 3] = 1.0
    d, ids = oracle.render([(verts, tris, P)], cam)
    assert ids[0, H // 2, W // 2] == 0 and (ids >= 0).sum() > 100
    xyz, tri = b3d.render_batch(b3d.Mesh(verts, tris), dev(np.tile(P, (N, 1, 1))), b3d.intrinsics_of(cam))
    z = xyz[..., 2].cpu().numpy()
    assert np.array_equal(z > 0, np.broadcast_to(d > 0, z.shape)) and np.abs(z - d).max() <= 1e-5
    assert bool((tri[:, H // 2, W // 2] == 0).all()) and bool((tri == tri[:1]).all())


# the split adjoint with observed pixels that hold no measurement (whatever x and
# y are) and points at infinity where no window sees anything drawn: the same
# gradients as with zeros and far points there, with and without a workspace
@pytest.mark.parametrize("workspace", [True, False])
@pytest.mark.parametrize("window", [1, 3, 5, 7, 9])
def test_score_adjoint_with_points_that_are_none(b3d, window, workspace):
    H, W, h = 33, 48, window // 2
    rng = np.random.default_rng(window)
    cam = Camera(W, W, W / 2, H / 2, H, W)
    rays = oracle.unproject(np.ones((1, H, W)), cam)[0]
    z = np.zeros((2, H, W))
    z[0, 9:22, 12:30] = 0.8 + rng.normal(0, 0.003, (13, 18))
    z[1, 12:20, 10:33] = 0.8 + rng.normal(0, 0.003, (8, 23))
    z[:, ::3, ::4] = 0.0
    rend = f32(z[..., None] * rays)
    near = np.zeros((H, W), bool)
    for r, c in zip(*np.nonzero((z > 0).any(0))):
        near[max(r - h, 0) : r + h + 1, max(c - h, 0) : c + h + 1] = True
    plain = f32((0.8 + rng.normal(0, 0.003, (H, W)))[..., None] * rays)
    odd = plain.copy()
    hole = rng.random((H, W)) < 0.2
    plain[hole], odd[hole] = 0.0, [np.nan, np.inf, 0.0]
    beside = ~near & ~hole
    plain[beside], odd[beside] = [0.0, 0.0, 50.0], [np.nan, np.inf, np.inf]
    assert hole[near].any() and beside.any()
    p, dl = b3d.score_params(0.005, 0.1, 1.0, window), dev([1.0, -0.7])
    a, b = (b3d.score_backward(dev(o), dev(rend), p, dl, workspace=workspace) for o in (plain, odd))
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    _, s64, _ = oracle.score_grad(plain, rend, float(np.float32(0.005)), float(np.float32(0.1)), 1.0, window)
    want = s64 * dl.cpu().numpy()
    assert np.all(np.abs(b[1].cpu().numpy() - want) <= 1e-5 * np.abs(want).max())


# observed pixels that see nothing drawn are only counted, by rows: more rows
# than a workgroup has threads, rows without any, and none at all
@pytest.mark.parametrize("H,W", [(1, 7), (700, 9), (513, 4)])
def test_score_adjoint_counts_what_sees_nothing(b3d, H, W):
    rng = np.random.default_rng(H)
    cam = Camera(50.0, 50.0, W / 2, H / 2, H, W)
    rays = oracle.unproject(np.ones((1, H, W)), cam)[0]
    z = np.zeros((3, H, W))
    z[1, H // 3 : H // 3 + 3] = 0.8
    z[2, H - 1, 0] = 0.8
    rend = f32(z[..., None] * rays)
    zo = np.where(rng.random((H, W)) < 0.3, 0.0, 0.8 + rng.normal(0, 0.003, (H, W)))
    zo[H // 2 : H // 2 + 5] = 0.0
    sg, po = float(np.float32(0.005)), float(np.float32(0.1))
    for obs in (f32(zo[..., None] * rays), np.zeros((H, W, 3))):
        dr, ds, dp = b3d.score_backward(dev(obs), dev(rend), b3d.score_params(sg, po, 1.0, 3))
        r64, s64, p64 = oracle.score_grad(obs, rend, sg, po, 1.0, 3)
        assert np.abs(dr.cpu().numpy() - r64).max() <= 1e-5 * np.abs(r64).max()
        for got, want in ((ds, s64), (dp, p64)):
            assert np.all(np.abs(got.cpu().numpy() - want) <= 1e-5 * np.abs(want).max())


# the split adjoint's workgroup and LDS by image size and number of hypotheses:
# either side of 1,024 pixels, of 512 hypotheses, and of the halo that half of
# the LDS is worth: the same gradients as the general kernel and the oracle
@pytest.mark.parametrize("window", [1, 3, 7])
@pytest.mark.parametrize("H,W", [(24, 32), (25, 31), (32, 32), (33, 32), (48, 64), (60, 90)])
def test_score_adjoint_by_workgroups_of_either_size(b3d, H, W, window):
    rng = np.random.default_rng(H * W + window)
    cam = Camera(0.9 * W, 0.9 * W, W / 2, H / 2, H, W)
    rays = oracle.unproject(np.ones((1, H, W)), cam)[0]
    z = 0.8 + rng.normal(0, 0.003, (4, H, W))
    z[1, : H // 3] = z[2, :, W // 2 :] = 0.0
    z[3] = 0.0
    z[3, H // 2 : H // 2 + 9, 3:14] = 0.8
    rend = f32(z[..., None] * rays)
    zo = np.where(rng.random((H, W)) < 0.2, 0.0, 0.8 + rng.normal(0, 0.003, (H, W)))
    obs = f32(zo[..., None] * rays)
    sg, po = float(np.float32(0.005)), float(np.float32(0.1))
    p = b3d.score_params(sg, po, 1.0, window)
    want = oracle.score_grad(obs, rend, sg, po, 1.0, window)
    general = b3d.score_backward(dev(obs), dev(rend), p, workspace=False)
    for n in (1, 128, 129):
        got = b3d.score_backward(dev(obs), dev(np.tile(rend, (n, 1, 1, 1))), p)
        for k, (g, w, o) in enumerate(zip(got, general, want)):
            assert bool((g.view(n, *w.shape) == g[:4]).all())
            bar = 1e-5 * np.abs(o).max()
            assert np.abs(g[:4].cpu().numpy() - o).max() <= bar and (g[:4] - w).abs().max() <= 2 * bar, k


# larger images go by 512 threads alone up to 1,024 poses, with a second launch
# beyond: the same images as few poses at a time
@pytest.mark.parametrize("H,W", [(150, 161), (150, 200), (240, 320)])
def test_render_second_launch_beyond_two_rounds_gives_the_same(b3d, H, W):
    rng = np.random.default_rng(H + W)
    verts, tris = voxel_mesh(voxel_blob(400, rng))
    cam = Camera(0.94 * W, 0.94 * W, W / 2 + 0.2, H / 2 - 0.3, H, W)
    K, mesh = b3d.intrinsics_of(cam), b3d.Mesh(f32(verts), tris)
    P = f32(random_poses(rng, 1025, 0.8, 0.03))
    P[::7, 2, 3] = 2.5
    P[1, :3, 3] = 0.0, 0.0, 0.05
    P = dev(P)
    xyz, tri = b3d.render_batch(mesh, P, K)
    for k, n in ((0, 1024), (0, 100), (1000, 25)):
        x, t = b3d.render_batch(mesh, P[k : k + n].contiguous(), K)
        assert torch.equal(x, xyz[k : k + n]) and torch.equal(t, tri[k : k + n])
    sel = [0, 1, 2, 1024]
    d, ids = oracle.render([(f32(verts), tris, P[sel].cpu().numpy().astype(np.float64))], cam)
    same = tri[sel].cpu().numpy() == ids
    assert same.mean() >= 0.999
    assert np.abs(xyz[sel][..., 2].cpu().numpy() - d)[same & (ids >= 0)].max() <= 1e-5


# a thin, tall object in the first or the last column of an image of several
# megapixels: its band covers more pixels than an index in single precision holds
@pytest.mark.parametrize("H,W", [(1200, 4095), (3400, 1921), (3400, 1920)])
def test_thin_objects_at_the_edges_of_large_images(b3d, H, W):
    f = 2000.0
    verts, tris = box_mesh((3.0 / f, (H - 41.0) / f, 0.002))
    verts = f32(verts)
    cam = Camera(f, f, W / 2, H / 2, H, W)
    P = np.tile(np.eye(4), (2, 1, 1))
    P[:, 2, 3] = 1.0
    P[:, 0, 3] = (0.8 - W / 2) / f, (W / 2 - 0.8) / f
    P = f32(P)
    d, ids = oracle.render([(verts, tris, P)], cam)
    assert (d[0, :, 0] > 0).sum() > H - 60 and (d[1, :, -1] > 0).sum() > H - 60
    xyz, tri = b3d.render_batch(b3d.Mesh(verts, tris), dev(P), b3d.intrinsics_of(cam))
    z = xyz[..., 2].cpu().numpy()
    assert np.array_equal(z > 0, d > 0), int(((z > 0) != (d > 0)).sum())
    assert np.abs(z - d).max() <= 1e-5 and np.array_equal(tri.cpu().numpy() >= 0, ids >= 0)


# faces that share their edges only up to the rounding of the largest coordinate
# (here 60 m away): what that moves a corner by on the screen is part of the margin
# of the exact test, so coverage is the oracle's at every pixel
@pytest.mark.parametrize("N", [1, 600])
def test_nearly_equal_faces_of_a_large_mesh_are_decided_exactly(b3d, N):
    H, W, f = 120, 160, 1200.0
    k = np.arange(10)
    c = np.stack(np.meshgrid(k, k, [0.0], indexing="ij"), -1).reshape(-1, 3) * 0.01
    small, large = voxel_mesh(c, 0.01), voxel_mesh(c, 0.01)
    large = large[0] * (1.0 + 1e-3) + [0.0, 0.11, 0.0], large[1]  # 1e-5 m an edge
    mesh = turned(joined(small, large, box_mesh((0.01, 0.01, 0.01), (60.0, 0.0, 0.0))), 0.3)
    verts, tris = f32(mesh[0]), mesh[1]
    cam = Camera(f, f, 20.0, 30.0, H, W)
    P = np.tile(np.eye(4), (4, 1, 1))
    P[:, 2, 3] = 1.0
    P[:, 0, 3], P[:, 1, 3] = [0.003, -0.02, 0.011, 0.03], [0.004, -0.1, 0.0, -0.13]
    P = f32(P)
    d, ids = oracle.render([(verts, tris, P)], cam)
    assert (ids >= 0).mean() > 0.3
    xyz, tri = b3d.render_batch(b3d.Mesh(verts, tris), dev(np.tile(P, (N, 1, 1))), b3d.intrinsics_of(cam))
    for n in (0, N - 1):
        z, i = xyz[4 * n : 4 * n + 4, ..., 2].cpu().numpy(), tri[4 * n : 4 * n + 4].cpu().numpy()
        assert np.array_equal(z > 0, d > 0), int(((z > 0) != (d > 0)).sum())
        assert np.abs(z - d).max() <= 1e-5
        assert (i == ids).mean() >= 0.9999, int((i != ids).sum())


def kernels_of(call):
    """Kernels that a call launches on the current stream, from a captured graph."""
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64.so" in line)
    hip = ctypes.CDLL(path)
    st, graph, n = torch.cuda.Stream(), ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(st.cuda_stream), 0) == 0
        try:
            call()
        finally:
            rc = hip.hipStreamEndCapture(ctypes.c_void_p(st.cuda_stream), ctypes.byref(graph))
    assert rc == 0 and hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


# a tuned tile, the same tile from the cache and the same tile set: the scene's
# launches are the same; a sample too small to take the tile leaves the default
@pytest.mark.parametrize("grad", [False, True])
def test_a_cached_tile_takes_the_route_of_a_tuned_one(b3d, tmp_path, grad):
    rng = np.random.default_rng(5)
    H, W = 180, 240
    verts, tris = voxel_mesh(voxel_blob(300, rng))
    cam = Camera(0.94 * W, 0.94 * W, W / 2, H / 2, H, W)
    K, mesh = b3d.intrinsics_of(cam), b3d.Mesh(f32(verts), tris)
    P = dev(f32(random_poses(rng, 700, 0.7, 0.03)))
    xyz, _ = b3d.render_batch(mesh, P[:1].contiguous(), K)
    obs, cache, p = xyz[0].contiguous(), str(tmp_path / "tiles.json"), b3d.score_params(0.004, 0.05, 1.0, 5)
    L, g = torch.empty(700, device="cuda"), torch.empty((700, 8), device="cuda")

    def fresh():
        scene = b3d.Scene(mesh, K, p)
        scene.set_observed(obs)
        return scene

    def call(scene):
        b3d._call("b3d_render_score", scene._h, P.data_ptr(), 700, L.data_ptr(), g.data_ptr() if grad else None,
                  b3d._stream())

    default = fresh()
    want = kernels_of(lambda: call(default))
    assert want == 2
    results = []
    for how in ("tuned", "cached", "set", "tuned after set"):
        scene = fresh()
        if how == "set":
            scene.set_tile(tile)
        elif how == "tuned after set":
            scene.set_tile(scene.tile_limits()[0])
            scene.autotune(P, grad=grad)
        else:
            tile = scene.autotune(P, grad=grad, cache=cache)
        if how != "tuned after set":
            assert scene.tile_limits()[2] == tile
        assert kernels_of(lambda: call(scene)) == want, how
        call(scene)
        results.append((L.clone(), g.clone() if grad else None))
    for x, y in results[1:]:
        assert torch.equal(x, results[0][0]) and (not grad or torch.equal(y, results[0][1]))
    scene = fresh()
    size = scene.tile_limits()[2]
    for n in (1, 256, 512):
        scene.set_tile(scene.tile_limits()[0])
        assert scene.autotune(P[:n].contiguous(), grad=grad) == size == scene.tile_limits()[2]


# bands of rows in 256-thread workgroups (images below 24,000 pixels, tiles of two
# rows) give what one band gives, with the adjoint and for noise grids in registers and in LDS
@pytest.mark.parametrize("window", [3, 5, 7, 9])
def test_bands_of_small_tiles_give_the_same(b3d, window):
    rng = np.random.default_rng(window)
    H, W = 90, 120
    verts, tris = voxel_mesh(voxel_blob(300, rng, radius=0.08))
    cam = Camera(0.94 * W, 0.94 * W, W / 2 + 0.2, H / 2 - 0.3, H, W)
    K = b3d.intrinsics_of(cam)
    P = dev(f32(random_poses(rng, 600, 0.6, 0.03)))
    scene = b3d.Scene(b3d.Mesh(f32(verts), tris), K, b3d.score_params(0.004, 0.05, 1.0, window))
    xyz, _ = b3d.render_batch(scene.mesh, P[1:2].contiguous(), K)
    scene.set_observed(xyz[0].contiguous())
    few = P[:200].contiguous()  # one large workgroup each, in one band
    want = [scored(b3d, scene, few, grad) for grad in (False, True)]
    grids = []
    for A, B in ((3, 5), (5, 3)):
        scene.set_noise_grid(*b3d.noise_grid_midpoints(0.012, A, B))
        grids.append(b3d.render_score_marginal(scene, few, grid=True))
    scene.set_tile(scene.tile_limits()[0])
    for grad in (False, True):
        for a, b in zip(scored(b3d, scene, P, grad), want[grad]):
            np.testing.assert_array_equal(a[:200], b)
    for (A, B), ref in zip(((3, 5), (5, 3)), grids):
        scene.set_noise_grid(*b3d.noise_grid_midpoints(0.012, A, B))
        for a, b in zip(b3d.render_score_marginal(scene, P, grid=True), ref):
            assert torch.equal(a[:200], b)
