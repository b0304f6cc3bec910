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


def _views(lnr, ctx, cloud, cams):
    import torch
    imgs = [lnr.Image(c.height, c.width) for c in cams]
    lnr.lnr_render_views(ctx, cloud, cams, imgs)
    torch.cuda.synchronize()
    return imgs


def test_views_under_a_budget(lnr, ctx, room_cloud, room_cams):
    """lnr_render_views with scratch for all eight views, for some, and for none
    (then without the tiled splat): the same images, never refused for it."""
    cams = list(room_cams[:8])
    want = [image_to_host(render_gpu(lnr, ctx, room_cloud, c)) for c in cams]
    free = lnr.lnr_context_create(0)
    for img, w in zip(_views(lnr, free, room_cloud, cams), want):
        assert_images_equal(image_to_host(img), w, "no budget")
    full = lnr.lnr_allocated_bytes(free)
    one = lnr.lnr_context_create(0)
    _views(lnr, one, room_cloud, cams[:1])
    single = lnr.lnr_allocated_bytes(one)
    assert single < full
    for budget in (single, 3 * single, single // 2):
        print("budget", budget, flush=True)
        c = lnr.lnr_context_create(0, budget)
        for img, w in zip(_views(lnr, c, room_cloud, cams), want):
            assert_images_equal(image_to_host(img), w, f"budget {budget}")
        assert lnr.lnr_allocated_bytes(c) <= budget


def test_views_of_many_tiles(lnr, ctx, room_cloud, room_cams):
    """One view of more than 8192 tiles (its scan is a launch of its own) among smaller ones."""
    import dataclasses
    big = dataclasses.replace(room_cams[1], width=4096, height=2112)
    cams = [room_cams[0], big, room_cams[2]]
    for cam, img in zip(cams, _views(lnr, ctx, room_cloud, cams)):
        assert_images_equal(image_to_host(img), image_to_host(render_gpu(lnr, ctx, room_cloud, cam)),
                            f"{cam.width}x{cam.height}")


@pytest.mark.parametrize("W", [1024, 1056])
@pytest.mark.parametrize("n", [2048, 2049, 4097, 8193, 12289, 40000])
def test_units_by_records(lnr, ctx, W, n):
    """All points on two tiles, which take one unit of work per 2048 entries in
    images of up to 1024 tiles and per 4096 in larger ones, but never more
    units than segments (one per work item and tile)."""
    import torch
    print("units", W, n, flush=True)
    H = 1024
    xyz, rgb, cam = _cloud(np.random.default_rng(n), n, 500, 520, 24, 20, W, H)
    g = G.partition(xyz, rgb, 100.0)
    cloud = lnr.lnr_cloud_load(ctx, xyz, rgb, 100.0)
    want = R.render(g, cam)
    assert_images_equal(image_to_host(render_gpu(lnr, ctx, cloud, cam)), want, "hard")
    img = lnr.Image(H, W)
    lnr.lnr_render_soft(ctx, cloud, cam, img, 0.3)
    torch.cuda.synchronize()
    soft = R.soft_colors(g.xs, g.ys, g.zs, g.rgb, cam.P, W, H, cam.z_near, cam.z_far, want[0], 0.3)
    assert_images_equal(image_to_host(img), (want[0], want[1], soft), "soft")
