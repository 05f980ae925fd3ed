"""Warped crops four pixels at a time, at the edges of the quads, of the wave's
rows and of the loads that serve a resize: output sides around multiples of 4 and
of 256 columns, sources of 8 columns and fewer, steps of exactly 2 source pixels
and just over, mirrored and turned frames, boxes at the image's corners, and a
plane wider than 2^15. Counts and features against the oracle bit for bit."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu
ONE = lbpf.ONE


def check(ref, planes, boxes, **kw):
    ctx = lbpf.Context(**kw)
    dev = [lbpf.to_device_planes(g, z) for g, z in planes]
    hist, cnt = ctx.features_warped(dev, boxes, with_counts=True)
    torch.cuda.synchronize()
    f, c, _ = ref.features_warped(planes, boxes, **kw)
    assert np.array_equal(cnt.cpu().numpy().view(np.uint32), c)
    assert np.array_equal(hist.cpu().numpy().view(np.uint32), f.view(np.uint32))
    ctx.close()


def image(rng, w, h):
    g = rng.integers(0, 256, size=(h, w)).astype(np.uint8)
    z = rng.integers(700, 1000, size=(h, w)).astype(np.uint16)
    z[rng.random((h, w)) < 0.05] = 0
    return g, z


def test_resizes(ref):
    require_gpu()
    rng = np.random.default_rng(1)
    planes = [image(rng, 640, 480), image(rng, 8, 9), image(rng, 7, 30)]
    boxes = []
    for side_w, side_h in ((200, 200), (3, 5), (4, 4), (5, 3), (63, 64), (65, 33), (255, 20), (257, 40), (700, 11)):
        for im, x, y, w, h in ((0, 0, 0, 48, 60), (0, 384, 224, 256, 256), (0, 592, 3, 48, 256),
                               (0, 10, 20, 2 * side_w if 2 * side_w < 600 else 600, 100),
                               (0, 10, 20, min(2 * side_w + 1, 600), 99), (1, 0, 0, 8, 9), (2, 0, 1, 7, 28)):
            fr = lbpf.resize_frame(x, y, w, h, side_w, side_h)
            boxes.append((im, side_w, side_h, fr, fr))
    check(ref, planes, boxes)


def test_frames(ref):
    require_gpu()
    rng = np.random.default_rng(2)
    planes = [image(rng, 300, 200)]
    w, h = 90, 70
    mirror = (-ONE, 0, 0, ONE, 200 * ONE, 10 * ONE)
    turn = (0, ONE, -ONE, 0, 250 * ONE, 20 * ONE)
    slant = (ONE // 2, ONE // 7, -ONE // 9, ONE, 40 * ONE + 77, 30 * ONE + 5)
    plain = lbpf.box_frame(5, 6)
    boxes = [(0, w, h, a, b) for a in (mirror, turn, slant, plain) for b in (plain, slant, mirror)]
    check(ref, planes, boxes)


@pytest.mark.parametrize("modality", [lbpf.MOD_GREY, lbpf.MOD_DEPTH])
def test_wide_plane_and_one_channel(ref, modality):
    require_gpu()
    rng = np.random.default_rng(3)
    planes = [image(rng, 40000, 40)]
    # Frames start below column 2^15 (their origin is 16.16 in 32 bits) and end past it.
    boxes = [(0, 50, 30, fr, fr) for fr in (lbpf.resize_frame(32700, 0, 100, 40, 50, 30),
                                            lbpf.resize_frame(32700, 2, 70, 30, 50, 30),
                                            lbpf.box_frame(32720, 10))]
    check(ref, planes, boxes, modality=modality)
