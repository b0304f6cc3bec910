"""The U-Net's convolution tiles at their edges.

The tile of a layer follows its size, and every tile takes its sums in the
same order, so a picture must equal the matching part of a larger picture bit
for bit away from the cut (in float32 too).  The sizes straddle the tiles' 8
and 16 rows and 32 columns and make one layer run in different tiles; the
widths give 32-, 64- and 96-channel layers (one, two and three 32-channel
tiles), half-filled ones (16, 48) and a first level whose head is not fused."""

import numpy as np
import pytest

import synth
from tests.gpu_util import UNET_PRECISIONS, check_unet_error, image_from_host
from oracle import metrics as M
from oracle import unet as U

pytestmark = pytest.mark.gpu


def _rgbda(seed, H, W):
    rng = np.random.default_rng(seed)
    filled = rng.random((H, W)) < 0.6
    depth = np.where(filled, rng.uniform(0.2, 40, (H, W)), 0).astype(np.float32)
    rgba = rng.integers(0, 256, (H, W, 4)).astype(np.uint8)
    rgba[..., 3] = filled
    rgba[~filled] = 0
    return depth, rgba


def _run(lnr, ctx, net, depth, rgba):
    import torch
    img = image_from_host(lnr, depth, rgba)
    out = torch.empty((3,) + depth.shape, dtype=torch.float32, device="cuda")
    lnr.lnr_reconstruct(ctx, net, img, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("prec", UNET_PRECISIONS)
@pytest.mark.parametrize("widths", [(16, 48), (32, 64), (48, 96), (64, 32), (96, 64)])
def test_tiles_agree_with_a_larger_picture(lnr, ctx, prec, widths):
    print("tiles", prec, widths, flush=True)
    net = lnr.lnr_unet_load(ctx, synth.make_unet_blob(widths, seed=21, bias="uniform"), prec)
    depth, rgba = _rgbda(3, 768, 1088)
    big = _run(lnr, ctx, net, depth, rgba)
    # the output depends on at most 12 pixels around it (two convolutions at
    # each side of the full level, two on pairs of pixels in between)
    m = 12
    for H, W in [(18, 34), (34, 66), (136, 258), (272, 544)]:
        got = _run(lnr, ctx, net, depth[:H, :W].copy(), rgba[:H, :W].copy())
        assert np.array_equal(got[:, :H - m, :W - m].view(np.uint32),
                              big[:, :H - m, :W - m].view(np.uint32)), f"{H}x{W}"


@pytest.mark.parametrize("prec", UNET_PRECISIONS)
def test_unfused_head(lnr, ctx, prec):
    print("head", prec, flush=True)
    blob = synth.make_unet_blob((80, 96), seed=5, bias="uniform")
    depth, rgba = _rgbda(9, 26, 70)
    net = lnr.lnr_unet_load(ctx, blob, prec)
    err = M.max_abs(_run(lnr, ctx, net, depth, rgba), U.forward(U.parse_blob(blob), depth, rgba))
    check_unet_error(prec, err, "widths (80, 96) 26x70")


@pytest.mark.parametrize("prec", UNET_PRECISIONS)
@pytest.mark.parametrize("widths", [(16, 80), (16, 160)])
def test_runs_of_one_chunk_tiles(lnr, ctx, prec, widths):
    """Level 1 reads 16 channels (one step per tile) and writes three or five
    32-channel tiles, in a picture large enough for workgroups that walk several
    tiles of different channels: their biases must not mix.  Against windows
    whose level 1 takes one tile per workgroup, bit for bit."""
    print("runs", prec, widths, flush=True)
    net = lnr.lnr_unet_load(ctx, synth.make_unet_blob(widths, seed=22, bias="uniform"), prec)
    H, W, side, m = 1056, 2112, 544, 12
    depth, rgba = _rgbda(4, H, W)
    big = _run(lnr, ctx, net, depth, rgba)
    for y in range(0, H - 2 * m, side - 2 * m):
        for x in range(0, W - 2 * m, side - 2 * m):
            y1, x1 = min(y + side, H), min(x + side, W)
            got = _run(lnr, ctx, net, depth[y:y1, x:x1].copy(), rgba[y:y1, x:x1].copy())
            # away from the cuts (the picture's own borders are the window's)
            a, b = (m if y else 0), (y1 - y - (m if y1 < H else 0))
            c, d = (m if x else 0), (x1 - x - (m if x1 < W else 0))
            assert np.array_equal(got[:, a:b, c:d].view(np.uint32),
                                  big[:, y + a:y + b, x + c:x + d].view(np.uint32)), f"window at {y}, {x}"
