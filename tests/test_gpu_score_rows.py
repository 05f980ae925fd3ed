"""The FP32 few-rows kernel (W read once, D shared by the waves of a workgroup
and over workgroups) at the edges of its 16- and 32-row blocks, of its 32-column
steps and of the rule that chooses it: scores within 1e-5 of the dot product's
condition scale of the FP64 product, identities the first maximum of the
call's own scores, and the same without scores."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf
from tests.gpu_util import require_gpu, score_tolerance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,modality,N,K", [
    ((8, 8), lbpf.MOD_BOTH, 1, 1),
    ((8, 8), lbpf.MOD_BOTH, 16, 33),
    ((8, 8), lbpf.MOD_BOTH, 17, 1024),
    ((8, 8), lbpf.MOD_BOTH, 33, 2049),
    ((8, 8), lbpf.MOD_BOTH, 65, 31),
    ((8, 8), lbpf.MOD_BOTH, 513, 512),   # 9 x 16 blocks
    ((4, 4), lbpf.MOD_GREY, 21, 70),     # D = 944: the last 32-column step is half full
    ((2, 2), lbpf.MOD_GREY, 64, 40),     # D = 236: fewer steps than waves
    ((2, 1), lbpf.MOD_BOTH, 5, 7),       # D = 236, one split
])
def test_few_rows(grid, modality, N, K):
    require_gpu()
    ctx = lbpf.Context(grid=grid, modality=modality)
    rng = np.random.default_rng(N * 10007 + K)
    X = rng.random((N, ctx.dim), dtype=np.float32)
    W = rng.standard_normal((K, ctx.dim), dtype=np.float32)
    b = rng.standard_normal(K).astype(np.float32)
    Xd, wts = torch.from_numpy(X).cuda(), ctx.weights(torch.from_numpy(W).cuda(), torch.from_numpy(b).cuda())
    S, A = ctx.score(Xd, wts)
    _, A2 = ctx.score(Xd, wts, want_scores=False)
    torch.cuda.synchronize()
    S64 = X.astype(np.float64) @ W.astype(np.float64).T + b
    S, A = S.cpu().numpy(), A.cpu().numpy()
    assert (np.abs(S - S64) <= score_tolerance(X, W, b)).all()
    assert np.array_equal(A, np.argmax(S, axis=1))
    assert np.array_equal(A2.cpu().numpy(), A)
    wts.close()
    ctx.close()
