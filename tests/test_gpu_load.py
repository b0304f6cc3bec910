"""Cloud loading at its limits: bounding boxes of cells around the 1024 points
one wave takes (larger cells are taken in slices of the sorted points), seen
through the exact cull decision, against the oracle."""

import numpy as np
import pytest

from oracle import grid as G
from synth.camera import Camera
from tests.gpu_util import render_gpu

pytestmark = pytest.mark.gpu


def _look(rng, W=64, H=48):
    """A narrow camera at a random place, with z_near and z_far that cut through the cells."""
    a, b = rng.uniform(0, 2 * np.pi), rng.uniform(-0.5, 0.5)
    fwd = np.array([np.cos(a) * np.cos(b), np.sin(a) * np.cos(b), np.sin(b)])
    right = np.cross(fwd, [0, 0, 1.0])
    right /= np.linalg.norm(right)
    R = np.stack([right, np.cross(fwd, right), fwd])
    K = np.array([[90.0, 0, W / 2], [0, 90.0, H / 2], [0, 0, 1]])
    P = K @ np.concatenate([R, -(R @ rng.uniform(-4, 4, 3))[:, None]], 1)
    return Camera(P.astype(np.float32).ravel(), W, H)


@pytest.mark.parametrize("counts", [[1, 1023, 1024, 1025], [5000, 2, 1025, 2048, 1], [1024] * 6, [1, 9000, 1],
                                    [700, 700, 1500, 700, 2049, 4097, 3]])
def test_bounds_of_large_cells(lnr, ctx, counts):
    print("cells", counts, flush=True)
    rng = np.random.default_rng(sum(counts))
    xyz = [np.array([[-4.0, -4.0, -4.0], [4.0, 4.0, 4.0]])]
    for i, n in enumerate(counts):  # a cluster well inside its 1 m cell, on both signs, some at -0.0
        c = np.array([i % 4 * 2 - 3.5, i // 4 * 2 - 2.5, (i % 3) - 1.0 + 0.5])
        p = c + rng.uniform(-0.2, 0.2, (n, 3)) * rng.uniform(0.2, 1, 3)
        p[rng.random(n) < 0.1, i % 3] = c[i % 3] if i % 2 else -0.0
        xyz.append(p)
    xyz = np.concatenate(xyz).astype(np.float32)
    xyz = xyz[rng.permutation(len(xyz))]
    rgb = rng.integers(0, 256, (len(xyz), 3)).astype(np.uint8)
    g = G.partition(xyz, rgb, 1.0)
    cloud = lnr.lnr_cloud_load(ctx, xyz, rgb, 1.0)
    seen = 0
    for _ in range(48):
        cam = _look(rng)
        render_gpu(lnr, ctx, cloud, cam)
        flags = np.asarray(lnr.lnr_render_stats(ctx, g.n_cells)[2])
        want = G.cull(g, cam.P, cam.width, cam.height, cam.z_near, cam.z_far)
        assert np.array_equal(flags.astype(bool), np.asarray(want).astype(bool))
        seen += int(np.asarray(want).sum())
    assert seen > 0
