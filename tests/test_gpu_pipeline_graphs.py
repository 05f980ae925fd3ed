"""The captured serving step has two graphs, for small faces and for others, and takes
the one that suits each batch: batches on both sides of the rule, one after another
through the same pipeline, against the oracle (features bit for bit) and the call
without a graph (identities)."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf, synth
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_boxes,batches", [
    (16, [(4, 48, 48), (4, 97, 96), (16, 96, 96), (1, 200, 150), (0, 9, 9), (16, 3, 3)]),
    (128, [(64, 40, 33), (65, 40, 33), (7, 96, 97), (64, 96, 96), (128, 12, 12)]),
    (129, [(16, 64, 64), (17, 64, 64), (1, 300, 20), (16, 96, 96)]),
    (513, [(5, 120, 120), (5, 20, 20)]),
])
def test_batches_of_both_kinds(ref, max_boxes, batches):
    require_gpu()
    ctx = lbpf.Context()
    W, b = synth.synthetic_weights(20, ctx.dim, synth.W_TINY)
    wts = ctx.weights(torch.from_numpy(W).cuda(), torch.from_numpy(b).cuda())
    pipe = ctx.pipeline(wts, max_boxes)
    rng = np.random.default_rng(max_boxes)
    for n, w, h in batches + batches[::-1]:
        host = [(rng.integers(0, 256, size=(h, w)).astype(np.uint8),
                 rng.integers(600, 900, size=(h, w)).astype(np.uint16)) for _ in range(n)]
        boxes = np.array([[i, 0, 0, w, h] for i in range(n)], np.int32).reshape(-1, 5)
        pipe.launch(lbpf.ImageTable([lbpf.to_device_planes(g, z) for g, z in host]), boxes)
        torch.cuda.synchronize()
        if n:
            f, _, _ = ref.features(host, boxes, n_threads=8)
            assert np.array_equal(pipe.hist[:n].cpu().numpy().view(np.uint32), f.view(np.uint32))
            _, A = ctx.score(pipe.hist[:n].contiguous(), wts)
            assert torch.equal(pipe.argmax[:n], A)
            assert np.array_equal(pipe.argmax_host[:n].numpy(), A.cpu().numpy())
    pipe.close()
    wts.close()
    ctx.close()
