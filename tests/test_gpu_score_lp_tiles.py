"""Reduced-precision scoring on every tile shape and at the edges of the rule
that chooses it: 32 x 32 tiles (at most two per CU, or up to 32 rows), 64 x 64
tiles (at most four per CU), the 256 x 128 and 256 x 256 tiles beyond. Scores
against the exact product of the quantised operands within the FP32
accumulation bound, identities the first maximum of the call's own scores."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf
from tests.gpu_util import require_gpu
from tests.lp_ref import lp_tolerance, quantised_reference

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 1), (31, 33), (32, 2050),    # 32 x 32
    (512, 1024), (513, 1025),        # 512 tiles of 32; 64 x 64
    (33, 8200),                      # 64 x 64, one row of tiles
    (300, 8200), (2100, 1030), (512, 8192),  # 64 x 64
    (480, 9000),                     # 256 x 128
    (600, 8200),                     # 256 x 256
]


@pytest.mark.parametrize("prec", ["bf16", "fp16", "fp8", "f16x3"])
@pytest.mark.parametrize("N,K", SHAPES)
def test_tiles(prec, N, K):
    require_gpu()
    # D = 944: 15 or 30 steps of 64 bytes, fewer than the waves' whole turns.
    ctx = lbpf.Context(grid=(4, 4), modality=lbpf.MOD_GREY)
    rng = np.random.default_rng(N * 10007 + K)
    X = rng.random((N, ctx.dim), dtype=np.float32)
    W = rng.standard_normal((K, ctx.dim), dtype=np.float32)
    b = rng.standard_normal(K).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    wts = ctx.weights(torch.from_numpy(W).cuda(), torch.from_numpy(b).cuda(), precision=prec)
    S, A = ctx.score(Xd, wts)
    _, A2 = ctx.score(Xd, wts, want_scores=False)
    torch.cuda.synchronize()
    S, A = S.cpu().numpy(), A.cpu().numpy()
    ref, scale = quantised_reference(X, W, b, prec)
    assert (np.abs(S - ref) <= lp_tolerance(prec, ctx.dim) * scale).all()
    assert np.array_equal(A, np.argmax(S, axis=1))
    assert np.array_equal(A2.cpu().numpy(), A)
    wts.close()
    ctx.close()
