"""Depth windows at and beyond the widest difference of two u16 depths, up to the
largest int32 ("every pixel with depth") and down to the lowest (no mask), against
the oracle: counts and features bit for bit, in every kind of configuration."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window", [65534, 65535, 65536, 2**30, 2**31 - 1, -2**31])
@pytest.mark.parametrize("mapping", [lbpf.MAP_U59, lbpf.MAP_FULL256])
@pytest.mark.parametrize("modality", [lbpf.MOD_BOTH, lbpf.MOD_GREY, lbpf.MOD_DEPTH])
def test_wide_windows(ref, window, mapping, modality):
    require_gpu()
    ctx = lbpf.Context(mapping=mapping, window=window, modality=modality)
    rng = np.random.default_rng(11)
    host, boxes = [], []
    for i, (w, h, top) in enumerate([(90, 80, 5000), (70, 65, 65536), (300, 40, 900), (3, 9, 65536)]):
        z = rng.integers(0, top, size=(h, w)).astype(np.uint16)
        z[rng.random((h, w)) < 0.05] = 0
        host.append((rng.integers(0, 256, size=(h, w)).astype(np.uint8), z))
        boxes.append([i, 0, 0, w, h])
    boxes = np.array(boxes, np.int32)
    dev = [lbpf.to_device_planes(g, z) for g, z in host]
    f, c = ctx.features(dev, boxes, with_counts=True)
    torch.cuda.synchronize()
    want_f, want_c, _ = ref.features(host, boxes, n_threads=8, mapping=mapping, window=window,
                                     modality=modality)
    assert np.array_equal(c.cpu().numpy().view(np.uint32), want_c)
    assert np.array_equal(f.cpu().numpy().view(np.uint32), want_f.view(np.uint32))
    ctx.close()
