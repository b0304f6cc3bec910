"""The binning pass's on-chip z-buffer at its limits: clouds of one cell whose
points cover a chosen pixel rectangle, against the oracle bit for bit.  8 x 8
pixel blocks are its unit: up to 64 of them meet there for work items of 4096
points, up to 128 for those of 8192 (cells that fill them), and every point is
binned by itself beyond.  The offsets make rectangles straddle blocks and 32 x
32 tiles; the soft z-buffer bins every point in either case."""

import numpy as np
import pytest

from oracle import grid as G
from oracle import render as R
from synth.camera import Camera
from tests.gpu_util import assert_images_equal, image_to_host, render_gpu

pytestmark = pytest.mark.gpu


def _cloud(rng, n, x0, y0, bw, bh, W, H):
    """n points on pixels of [x0, x0 + bw) x [y0, y0 + bh), both ends hit, at three depths."""
    u = rng.integers(0, bw, n)
    v = rng.integers(0, bh, n)
    u[:2], v[:2] = (0, bw - 1), (0, bh - 1)
    z = rng.choice(np.array([2.0, 2.5, 4.0]), n)
    f = 64.0
    X = (x0 + u + rng.uniform(0.1, 0.9, n) - W / 2) / f * z
    Y = (y0 + v + rng.uniform(0.1, 0.9, n) - H / 2) / f * z
    xyz = np.stack([X, Y, z], 1).astype(np.float32)
    P = np.array([f, 0, W / 2, 0, 0, f, H / 2, 0, 0, 0, 1, 0], np.float32)
    return xyz, rng.integers(0, 256, (n, 3)).astype(np.uint8), Camera(P, W, H)


@pytest.mark.parametrize("n", [3000, 9001, 20000])
@pytest.mark.parametrize("x0,y0,bw,bh", [(0, 0, 64, 64), (8, 16, 128, 64), (3, 5, 57, 59), (8, 8, 72, 64), (8, 8, 136, 64),
                                         (31, 31, 2, 2), (28, 4, 1024, 8), (4, 30, 8, 600), (0, 0, 1, 1),
                                         (0, 0, 1100, 700)])
def test_binning_rectangles(lnr, ctx, n, x0, y0, bw, bh):
    import torch
    print("bin", n, x0, y0, bw, bh, flush=True)
    W, H = 1100, 700
    xyz, rgb, cam = _cloud(np.random.default_rng(n + bw), n, x0, y0, bw, bh, W, H)
    g = G.partition(xyz, rgb, 100.0)
    cloud = lnr.lnr_cloud_load(ctx, xyz, rgb, 100.0)
    want = R.render(g, cam)
    assert_images_equal(image_to_host(render_gpu(lnr, ctx, cloud, cam)), want, "hard")
    img = lnr.Image(H, W)
    lnr.lnr_render_soft(ctx, cloud, cam, img, 0.3)
    torch.cuda.synchronize()
    soft = R.soft_colors(g.xs, g.ys, g.zs, g.rgb, cam.P, W, H, cam.z_near, cam.z_far, want[0], 0.3)
    assert_images_equal(image_to_host(img), (want[0], want[1], soft), "soft")
    lnr.lnr_render_soft(ctx, cloud, cam, img, 0.3, flags=lnr.LNR_RENDER_ATOMIC_SPLAT)
    torch.cuda.synchronize()
    assert_images_equal(image_to_host(img), (want[0], want[1], soft), "soft, atomic splat")
