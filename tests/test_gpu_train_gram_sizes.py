"""The Gram solver at the edges of its variants: one, two and four solver waves,
one copy of the margins or two, row pieces a lane, a last block of the order or a
last group of columns that is not full, and the Gram matrix's mirrored tiles.

Against the FP64 oracle trainer with the bar of the other Gram tests: weights and
biases within 1e-4 of the largest weight, the same epoch count."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

SEED = 150401883


@pytest.mark.parametrize("N", [65, 256, 257, 1023, 1024, 1025, 2048, 2049, 4095, 4097, 5120, 5121,
                               7796, 7797])
def test_sizes(ref, N):
    require_gpu()
    c = lbpf.Context(grid=(2, 8))
    rng = np.random.default_rng(N)
    lab = (np.arange(N) % 4).astype(np.int32)
    centres = rng.gamma(0.3, size=(4, c.dim))
    X = centres[lab] + rng.gamma(0.3, size=(N, c.dim))
    X = (X / X.sum(axis=1, keepdims=True)).astype(np.float32)
    K, epochs = 3, 3
    W_ref, b_ref, ep_ref = ref.train_ovr_f64(X, lab, K, max_epochs=epochs, seed=SEED, n_threads=8)
    out = c.train(torch.from_numpy(X).cuda(), torch.from_numpy(lab).cuda(), K, max_epochs=epochs,
                  seed=SEED)
    torch.cuda.synchronize()
    W, b = out["W"].cpu().numpy().astype(np.float64), out["b"].cpu().numpy().astype(np.float64)
    c.close()
    scale = np.abs(W_ref).max()
    assert scale > 0
    assert np.abs(W - W_ref).max() <= 1e-4 * scale
    assert np.abs(b - b_ref).max() <= 1e-4 * max(scale, np.abs(b_ref).max())
    assert int(out["epochs"].max()) == ep_ref
