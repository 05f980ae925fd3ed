"""Crops shared by several workgroups, crops wider than a panel of 256 columns,
and every configuration off the default one, against the oracle: counts and
features bit for bit, at the edges of panels, bands and parts, with depths
whose median the estimate's window misses, and through host boxes (crops in
the kernels' arguments and in device memory), a batch and a pipeline."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf, synth
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def crop(rng, w, h, kind="face"):
    if kind == "face" and min(w, h) >= 16:
        return synth.render_crop(w, h, synth.W_RAGGED, int(rng.integers(100)), int(rng.integers(1000)))
    g = rng.integers(0, 256, size=(h, w)).astype(np.uint8)
    if kind == "flat":
        return np.full((h, w), 7, np.uint8), np.full((h, w), 900, np.uint16)
    if kind == "none":
        return g, np.zeros((h, w), np.uint16)
    if kind == "near":  # the median lies within the window of 0
        return g, rng.integers(1, 200, size=(h, w)).astype(np.uint16)
    if kind == "two":  # two surfaces of about equal share, far apart
        z = np.where(rng.random((h, w)) < 0.5, 800, 3000) + rng.integers(-9, 10, size=(h, w))
        return g, z.astype(np.uint16)
    if kind == "spread":
        return g, rng.integers(0, 65536, size=(h, w)).astype(np.uint16)
    if kind == "missed":  # the sampled grid rows see another surface than the crop
        z = np.full((h, w), 1000, np.uint16)
        z[((2 * np.arange(16) + 1) * h) >> 5] = 5000
        return g, z
    return g, rng.integers(500, 900, size=(h, w)).astype(np.uint16)


def run(ctx, ref, crops, entry="direct", frame=False, **cfg):
    """Every crop its own exactly sized image (not over-readable), or inside a
    larger frame."""
    host, boxes = [], []
    for i, (g, z) in enumerate(crops):
        h, w = z.shape
        if frame:
            G, Z = np.zeros((h + 9, w + 13), np.uint8), np.zeros((h + 9, w + 13), np.uint16)
            G[4:4 + h, 5:5 + w], Z[4:4 + h, 5:5 + w] = g, z
            host.append((G, Z))
            boxes.append([i, 5, 4, w, h])
        else:
            host.append((g, z))
            boxes.append([i, 0, 0, w, h])
    boxes = np.array(boxes, np.int32)
    dev = [lbpf.to_device_planes(g, z) for g, z in host]
    out = torch.full((len(crops), ctx.dim), float("nan"), device="cuda")
    cnt = torch.full((len(crops), ctx.dim), -1, dtype=torch.int32, device="cuda")
    if entry == "batch":
        b = ctx.batch(dev, boxes)
        ctx.features_batch(b, out, cnt)
    else:
        ctx.features(dev, boxes, out=out, counts_out=cnt)
    torch.cuda.synchronize()
    f, c, _ = ref.features(host, boxes, n_threads=8, **cfg)
    assert np.array_equal(cnt.cpu().numpy().view(np.uint32), c)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), f.view(np.uint32))


@pytest.mark.parametrize("entry,frame", [("direct", False), ("direct", True), ("batch", False)])
def test_sizes(ref, entry, frame):
    require_gpu()
    ctx = lbpf.Context()
    rng = np.random.default_rng(5)
    sizes = [(1024, 1024), (1024, 3), (3, 1024), (4, 700), (255, 256), (256, 255), (257, 300),
             (258, 258), (510, 40), (511, 11), (765, 513), (300, 9), (3, 3), (200, 200)]
    run(ctx, ref, [crop(rng, w, h) for w, h in sizes], entry, frame)
    ctx.close()


@pytest.mark.parametrize("kind", ["flat", "none", "near", "two", "spread", "missed"])
def test_depths(ref, kind):
    require_gpu()
    ctx = lbpf.Context()
    rng = np.random.default_rng(6)
    # Split (one large crop decides), and one workgroup per crop.
    run(ctx, ref, [crop(rng, w, h, kind) for w, h in ((400, 330), (129, 200), (256, 256), (33, 17))])
    run(ctx, ref, [crop(rng, w, h, kind) for w, h in ((100, 80), (60, 90))])
    ctx.close()


@pytest.mark.parametrize("n", [1, 32, 33])
def test_table_in_arguments_or_memory(ref, n):
    require_gpu()
    ctx = lbpf.Context()
    rng = np.random.default_rng(n)
    run(ctx, ref, [crop(rng, 230 + i, 250 - i) for i in range(n)])
    ctx.close()


@pytest.mark.parametrize("window", [0, 90, 255, 256, 400, 40000])
@pytest.mark.parametrize("grid,mapping,modality", [
    ((8, 8), lbpf.MAP_FULL256, lbpf.MOD_BOTH),
    ((1, 1), lbpf.MAP_FULL256, lbpf.MOD_GREY),
    ((7, 3), lbpf.MAP_U59, lbpf.MOD_GREY),
    ((8, 8), lbpf.MAP_FULL256, lbpf.MOD_DEPTH),
    ((4, 4), lbpf.MAP_U59, lbpf.MOD_BOTH),
    ((6, 5), lbpf.MAP_U59, lbpf.MOD_BOTH),
])
def test_configurations(ref, grid, mapping, modality, window):
    require_gpu()
    ctx = lbpf.Context(grid=grid, mapping=mapping, window=window, modality=modality)
    rng = np.random.default_rng(window + grid[0])
    crops = [crop(rng, 200, 200), crop(rng, 300, 70), crop(rng, 3, 40), crop(rng, 66, 3),
             crop(rng, 90, 61, "two"), crop(rng, 77, 130, "near"), crop(rng, 64, 64, "spread"),
             crop(rng, 50, 50, "flat"), crop(rng, 40, 40, "none")]
    run(ctx, ref, crops, grid_x=grid[0], grid_y=grid[1], mapping=mapping, window=window,
        modality=modality)
    ctx.close()


@pytest.mark.parametrize("max_boxes", [512, 513])
def test_pipeline(ref, max_boxes):
    """Batches of 0 to many boxes through one captured graph, split (512) and on
    the persistent kernel (513)."""
    require_gpu()
    ctx = lbpf.Context()
    W, b = synth.synthetic_weights(20, ctx.dim, synth.W_TINY)
    wts = ctx.weights(torch.from_numpy(W).cuda(), torch.from_numpy(b).cuda())
    pipe = ctx.pipeline(wts, max_boxes)
    rng = np.random.default_rng(7)
    for n in (3, 60, 0, 17, 1):
        host = [crop(rng, int(rng.integers(3, 300)), int(rng.integers(3, 300))) for _ in range(n)]
        if n == 17:
            host[3] = crop(rng, 1024, 1024)
        boxes = np.array([[i, 0, 0, z.shape[1], z.shape[0]] for i, (_, z) in enumerate(host)],
                         np.int32).reshape(-1, 5)
        pipe.launch(lbpf.ImageTable([lbpf.to_device_planes(g, z) for g, z in host]), boxes)
        torch.cuda.synchronize()
        if n:
            f, _, _ = ref.features(host, boxes, n_threads=8)
            assert np.array_equal(pipe.hist[:n].cpu().numpy().view(np.uint32), f.view(np.uint32))
    pipe.close()
    wts.close()
    ctx.close()
