"""Each route that a launch can take through the kernels, at the sizes where
it changes: against the FP64 oracle, or against another route that has to give
the same.  Bars as in test_gpu_parity.py."""

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
