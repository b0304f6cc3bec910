"""The contexts' device scratch: what a call needs depends on the sizes that
its documentation names and on nothing else, and what is taken beyond that (the
multi-view launches) refuses no call, moves nothing that a captured graph
reads, and is left out where it cannot be had.  Images against single renders."""

import numpy as np
import pytest

from synth.camera import Camera
from tests.gpu_util import assert_images_equal, image_to_host, render_gpu

pytestmark = pytest.mark.gpu


def _camera(W, H, f=60.0):
    return Camera(np.array([f, 0, W / 2, 0, 0, f, H / 2, 0, 0, 0, 1, 0], np.float32), W, H)


def _grid_cloud(per_cell, side=200, depth=4.0):
    """per_cell points in each of side x side cells of 0.1 m, in front of the camera."""
    rng = np.random.default_rng(per_cell)
    i = np.repeat(np.arange(side * side), per_cell)
    c = np.stack([i % side, i // side], 1) * 0.1 - side * 0.05 + 0.05
    xy = c + rng.uniform(-0.03, 0.03, c.shape)
    xyz = np.concatenate([xy, np.full((len(xy), 1), depth)], 1).astype(np.float32)
    return xyz, rng.integers(0, 256, (len(xyz), 3)).astype(np.uint8)


def _tiles(cam):
    return -(-cam.width // 32) * -(-cam.height // 32)


def _documented(n, n_cells, items, cam):
    """Bytes of lnr_render: cull flags, work queues, counters, and the tiled
    splat's 28 per point with a unit of work per 32 of them and a few words per tile."""
    return n_cells + 128 * items + 92 + 28 * n + 8 * (n // 32) + 32 * _tiles(cam) + 12


@pytest.mark.parametrize("W,H", [(20, 17), (640, 480)])
def test_render_scratch_is_what_is_documented(lnr, ctx, W, H):
    """Sparse cells: as many segments as points are possible."""
    xyz, rgb = _grid_cloud(1)
    cloud = lnr.lnr_cloud_load(ctx, xyz, rgb, 0.1)
    cells = len(lnr.lnr_cloud_cell_start(cloud)) - 1
    items = int((np.diff(lnr.lnr_cloud_cell_start(cloud).astype(np.int64)) > 0).sum())
    c = lnr.lnr_context_create(0)
    cam = _camera(W, H)
    render_gpu(lnr, c, cloud, cam)
    assert lnr.lnr_allocated_bytes(c) <= _documented(len(xyz), cells, items, cam)


def test_render_scratch_warmed_by_the_largest_cloud(lnr, ctx):
    """A context that has rendered a cloud of more points, and holds the work
    queues of another, allocates nothing for the other at the same size."""
    big = np.zeros((200_000, 3), np.float32)
    big[:, 2] = 2.0 + np.linspace(0, 1, len(big))
    dense = lnr.lnr_cloud_load(ctx, big, np.zeros((len(big), 3), np.uint8), 100.0)
    sparse = lnr.lnr_cloud_load(ctx, *_grid_cloud(3), 0.1)
    c = lnr.lnr_context_create(0)
    cam = _camera(256, 256)
    render_gpu(lnr, c, sparse, cam, flags=lnr.LNR_RENDER_ATOMIC_SPLAT)
    render_gpu(lnr, c, dense, cam)
    warm = lnr.lnr_allocated_bytes(c)
    img = render_gpu(lnr, c, sparse, cam)
    assert lnr.lnr_allocated_bytes(c) == warm
    assert_images_equal(image_to_host(img), image_to_host(render_gpu(lnr, ctx, sparse, cam)), "sparse")


def _views(lnr, ctx, cloud, cams):
    import torch
    imgs = [lnr.Image(c.height, c.width) for c in cams]
    lnr.lnr_render_views(ctx, cloud, cams, imgs)
    torch.cuda.synchronize()
    return imgs


def _assert_views(lnr, ctx, cloud, cams, imgs, what):
    for v, (cam, img) in enumerate(zip(cams, imgs)):
        assert_images_equal(image_to_host(img), image_to_host(render_gpu(lnr, ctx, cloud, cam)), f"{what}: view {v}")


def test_views_of_a_small_cloud_after_a_large_one_under_a_budget(lnr, ctx, room_cloud, room_cams):
    """Scratch that is larger than needed stays as it is: views whose other
    needs have grown past the budget meanwhile still render."""
    rng = np.random.default_rng(3)
    xyz = rng.uniform(-1, 1, (3000, 3)).astype(np.float32) + np.float32([0, 0, 3])
    small = lnr.lnr_cloud_load(ctx, xyz, rng.integers(0, 256, (3000, 3)).astype(np.uint8), 100.0)
    free = lnr.lnr_context_create(0)
    render_gpu(lnr, free, room_cloud, room_cams[0])
    budget = lnr.lnr_allocated_bytes(free) + 200_000
    c = lnr.lnr_context_create(0, budget)
    render_gpu(lnr, c, room_cloud, room_cams[0])
    cams = [_camera(1920, 1080, 400.0 + v) for v in range(8)]
    imgs = _views(lnr, c, small, cams)
    assert lnr.lnr_allocated_bytes(c) <= budget
    _assert_views(lnr, ctx, small, cams, imgs, "small cloud")


def test_a_captured_render_outlives_larger_views(lnr, ctx, room_cloud, room_cams):
    """A graph of lnr_render stays valid while lnr_render_views takes scratch
    for more and larger views on the same context."""
    import torch
    c = lnr.lnr_context_create(0)
    want = image_to_host(render_gpu(lnr, ctx, room_cloud, room_cams[0]))
    img = lnr.Image(room_cams[0].height, room_cams[0].width)
    lnr.lnr_render(c, room_cloud, room_cams[0], img)
    torch.cuda.synchronize()
    held = lnr.lnr_allocated_bytes(c)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lnr.lnr_render(c, room_cloud, room_cams[0], img)
    for n in (2, 8):
        cams = list(room_cams[1:1 + n])
        imgs = _views(lnr, c, room_cloud, cams)
        _assert_views(lnr, ctx, room_cloud, cams, imgs, f"{n} views")
        assert lnr.lnr_allocated_bytes(c) > held
        img.key.fill_(0)
        img.rgba.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert_images_equal(image_to_host(img), want, f"replay after {n} views")


@pytest.mark.parametrize("n", [8, 1])
def test_views_take_fewer_where_scratch_cannot_be_allocated(lnr, ctx, room_cloud, room_cams, n):
    """A failed allocation refuses no multi-view call: fewer views per pass
    then, and with one view z-buffers in device memory."""
    cams = list(room_cams[:n])
    grew = []
    for fail in (1, -1):  # the second allocation (after the work items), none
        c = lnr.lnr_context_create(0)
        render_gpu(lnr, c, room_cloud, cams[0], flags=lnr.LNR_RENDER_ATOMIC_SPLAT)  # cull flags and counters
        before = lnr.lnr_allocated_bytes(c)
        lnr.lnr_debug_fail_allocation(c, fail)
        imgs = _views(lnr, c, room_cloud, cams)
        lnr.lnr_debug_fail_allocation(c, -1)
        grew.append(lnr.lnr_allocated_bytes(c) - before)
        _assert_views(lnr, ctx, room_cloud, cams, imgs, f"failure {fail}")
    assert grew[0] < grew[1]


def test_views_do_not_ask_again(lnr, ctx, room_cloud, room_cams):
    """What a first call was refused, a repeated one does not allocate either."""
    cams = list(room_cams[:8])
    c = lnr.lnr_context_create(0)
    render_gpu(lnr, c, room_cloud, cams[0], flags=lnr.LNR_RENDER_ATOMIC_SPLAT)
    lnr.lnr_debug_fail_allocation(c, 1)
    _views(lnr, c, room_cloud, cams)
    lnr.lnr_debug_fail_allocation(c, -1)
    first = lnr.lnr_allocated_bytes(c)
    imgs = _views(lnr, c, room_cloud, cams)
    assert lnr.lnr_allocated_bytes(c) == first
    _assert_views(lnr, ctx, room_cloud, cams, imgs, "again")


@pytest.mark.parametrize("warm", [1, 2, 8])
def test_captured_views(lnr, ctx, room_cloud, room_cams, warm):
    """Eight views captured on a context that has rendered `warm` small ones: no
    allocation under capture, and every replay gives the images, also after the
    context has taken scratch for larger views."""
    import dataclasses
    import torch
    c = lnr.lnr_context_create(0)
    small = [dataclasses.replace(k, width=128, height=96) for k in room_cams[:warm]]
    _views(lnr, c, room_cloud, small)
    held = lnr.lnr_allocated_bytes(c)
    cams = list(room_cams[:8])
    imgs = [lnr.Image(k.height, k.width) for k in cams]
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        lnr.lnr_render_views(c, room_cloud, cams, imgs)
    assert lnr.lnr_allocated_bytes(c) == held
    large = [dataclasses.replace(k, width=1024, height=768) for k in room_cams[8:16]]
    for n in (0, 4, 8):
        if n:
            _assert_views(lnr, ctx, room_cloud, large[:n], _views(lnr, c, room_cloud, large[:n]), f"{n} large")
        for img in imgs:
            img.key.fill_(0)
            img.rgba.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        _assert_views(lnr, ctx, room_cloud, cams, imgs, f"replay after {n}")
    del graph
    lnr.lnr_context_destroy(c)


def test_views_give_way_under_a_budget(lnr, room_cloud, room_cams):
    """A budget that holds a network, a reconstruction, a small cloud, a server
    and a session besides what a multi-view call cannot do without: none of
    them is refused after a multi-view call, which renders the same before and
    after."""
    import torch
    import synth
    cams = list(room_cams[:8])
    blob = synth.make_unet_blob((16, 32), seed=0)
    rng = np.random.default_rng(1)
    xyz, rgb = rng.uniform(-1, 1, (1000, 3)).astype(np.float32), rng.integers(0, 256, (1000, 3)).astype(np.uint8)
    out = torch.empty((3, cams[0].height, cams[0].width), dtype=torch.float32, device="cuda")

    def everything(c, views):
        net = lnr.lnr_unet_load(c, blob, lnr.LNR_FP16)
        img = lnr.Image(cams[0].height, cams[0].width)
        img.depth.zero_()
        img.rgba.zero_()
        first = _views(lnr, c, room_cloud, cams) if views else None
        lnr.lnr_reconstruct(c, net, img, out)
        cloud = lnr.lnr_cloud_load(c, xyz, rgb, 100.0)
        srv = lnr.lnr_server_create(c, cloud, net, max_batch=1, lanes=2, n_levels=3, max_width=128, max_height=96)
        lnr.lnr_server_open_session(srv, 128, 96)
        if views:
            again = _views(lnr, c, room_cloud, cams)
            for a, b in zip(first, again):
                assert_images_equal(image_to_host(a), image_to_host(b), "again")
        return lnr.lnr_allocated_bytes(c)

    items = int((np.diff(lnr.lnr_cloud_cell_start(room_cloud).astype(np.int64)) + 4095 >> 12).sum())
    cells = len(lnr.lnr_cloud_cell_start(room_cloud)) - 1
    # (loading the small cloud takes 100 KB for a moment)
    budget = everything(lnr.lnr_context_create(0), False) + cells + 256 * items + 92 + 100_000
    c = lnr.lnr_context_create(0, budget)
    assert everything(c, True) <= budget


def _serve_two(lnr, ctx, srv, cloud, net, cams):
    """Two sessions' requests in one batch against the frames computed alone."""
    import torch
    sids = [lnr.lnr_server_open_session(srv, k.width, k.height) for k in cams]
    for t, (sid, k) in enumerate(zip(sids, cams)):
        lnr.lnr_server_submit(srv, sid, k, t)
    got = {}
    for _ in range(100000):
        lnr.lnr_server_step(srv)
        for r in lnr.lnr_server_poll(srv):
            out = torch.empty((3, r["height"], r["width"]), dtype=torch.float32, device="cuda")
            lnr.copy_from_device(r["rgb"], out)
            got[r["tag"]] = out
            assert r["batch"] == 2
        if len(got) == 2:
            break
    for t, k in enumerate(cams):
        img = render_gpu(lnr, ctx, cloud, k)
        lnr.lnr_depth_filter(ctx, img, 3, 0.5)
        want = torch.empty_like(got[t])
        lnr.lnr_reconstruct(ctx, net, img, want)
        torch.cuda.synchronize()
        assert torch.equal(got[t], want), f"request {t}"


def test_server_without_the_scratch_for_several_requests(lnr, ctx, room_cloud, room_cams):
    """A server lane's scratch for several requests per launch refuses no
    server, where it cannot be allocated or does not fit the budget."""
    import dataclasses
    import synth
    cams = [dataclasses.replace(k, width=128, height=96) for k in room_cams[:2]]
    blob = synth.make_unet_blob((16, 32, 64), seed=0)
    net = lnr.lnr_unet_load(ctx, blob, lnr.LNR_FP16)

    def create(c):
        net = lnr.lnr_unet_load(c, blob, lnr.LNR_FP16)
        return lnr.lnr_server_create(c, room_cloud, net, max_batch=2, lanes=1, n_levels=3, filter_strength=0.5,
                                     max_width=128, max_height=96)

    c = lnr.lnr_context_create(0)
    keep = create(c)
    full = lnr.lnr_allocated_bytes(c)
    lnr.lnr_server_destroy(keep)
    without = None
    for n in range(64):
        c = lnr.lnr_context_create(0)
        net_c = lnr.lnr_unet_load(c, blob, lnr.LNR_FP16)
        lnr.lnr_debug_fail_allocation(c, n)
        try:
            srv = lnr.lnr_server_create(c, room_cloud, net_c, max_batch=2, lanes=1, n_levels=3, filter_strength=0.5,
                                        max_width=128, max_height=96)
        except lnr.LnrError as e:
            assert e.status == lnr.LNR_E_OUT_OF_MEMORY
            continue
        finally:
            lnr.lnr_debug_fail_allocation(c, -1)
        if lnr.lnr_allocated_bytes(c) == full:
            lnr.lnr_server_destroy(srv)
            break
        assert without in (None, lnr.lnr_allocated_bytes(c))
        without = lnr.lnr_allocated_bytes(c)
        _serve_two(lnr, ctx, srv, room_cloud, net, cams)
        lnr.lnr_server_destroy(srv)
    assert without is not None and without < full

    # a budget that holds the second view's splat scratch, but not all of the rest
    c = lnr.lnr_context_create(0, full - 50_000)
    srv = create(c)
    assert lnr.lnr_allocated_bytes(c) == without


def test_views_with_scratch_in_several_allocations(lnr, ctx):
    """Scratch of more than 1.5 GiB is three allocations."""
    rng = np.random.default_rng(12)
    xyz = rng.uniform(-4, 4, (12_000_000, 3)).astype(np.float32) + np.float32([0, 0, 6])
    rgb = rng.integers(0, 256, (len(xyz), 3)).astype(np.uint8)
    cloud = lnr.lnr_cloud_load(ctx, xyz, rgb, 0.25)
    cams = [_camera(640 + 32 * v, 480, 300.0 + 10 * v) for v in range(8)]
    c = lnr.lnr_context_create(0)
    imgs = _views(lnr, c, cloud, cams)
    assert lnr.lnr_allocated_bytes(c) > 3 << 29
    _assert_views(lnr, ctx, cloud, cams, imgs, "12M points")
    lnr.lnr_cloud_destroy(cloud)


@pytest.mark.parametrize("per_cell,n_views,W,H,tiled", [
    (1, 1, 640, 480, False), (1, 5, 640, 480, False), (1, 6, 640, 480, True), (1, 8, 160, 149, False),
    (1, 8, 160, 281, False), (1, 8, 160, 282, True), (7, 5, 320, 281, False), (7, 5, 320, 282, True),
    (0, 1, 160, 149, False), (0, 3, 160, 149, True), (0, 1, 160, 151, True)])
def test_views_by_either_splat(lnr, ctx, room_cloud, per_cell, n_views, W, H, tiled):
    """The choice between the tiled splat and the images' key buffers, at its
    limits (40000 cells of 1 or 7 points; the room's 760): the same images."""
    cloud = lnr.lnr_cloud_load(ctx, *_grid_cloud(per_cell), 0.1) if per_cell else room_cloud
    cams = [_camera(W, H, 60.0 + 9 * v) for v in range(n_views)]
    c = lnr.lnr_context_create(0)
    lnr.lnr_profile_enable(c, True)
    imgs = _views(lnr, c, cloud, cams)
    names = {name for name, _ in lnr.lnr_profile_read(c)}
    assert ("bin" in names, "splat_views" in names) == (tiled, not tiled)
    _assert_views(lnr, ctx, cloud, cams, imgs, "views")


@pytest.mark.parametrize("n", [1, 8])
def test_views_give_way_to_their_own_counters(lnr, ctx, room_cloud, room_cams, n):
    """Budgets around what the tiled splat of n views takes: where it fits but
    the last thing that the call allocates, its counters, does not fit beside
    it, the views go to the key buffers."""
    cams = list(room_cams[:n])
    full = lnr.lnr_context_create(0)
    _views(lnr, full, room_cloud, cams)
    need = lnr.lnr_allocated_bytes(full)  # with 92 bytes of counters
    for budget in (need - 93, need - 92, need - 1, need):
        c = lnr.lnr_context_create(0, budget)
        for _ in range(2):
            imgs = _views(lnr, c, room_cloud, cams)
            _assert_views(lnr, ctx, room_cloud, cams, imgs, f"budget {budget - need}")
        assert lnr.lnr_allocated_bytes(c) <= budget
        assert (lnr.lnr_allocated_bytes(c) == need) == (budget == need)
