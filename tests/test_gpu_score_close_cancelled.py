"""The identity of rows whose scores nearly cancel: weights that are close copies of one
another, of mean zero and without bias, so that the scores are small against the sums
they come from and their order is decided by rounding alone. The identity is the one
that FP32 sums in the fixed order give (see test_gpu_score_close), for every kernel
that makes scores; where D is not a multiple of 32 in four quarters of ceil(D / 128)
32 columns, each sixteen as 0 4 8 12 1 5 9 13 .. . Exact: the sums are emulated to the
last bit."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf
from tests.gpu_util import require_gpu, stacked_planes

pytestmark = pytest.mark.gpu


def fixed_order(X, W, b, ranges):
    """ranges: 1, 2, 4, or 0 for quarters. An FMA is a product and a sum in 64 bits,
    rounded once."""
    D = X.shape[1]
    if ranges:
        length, step, inner = D // ranges, 8, [0, 4, 1, 5, 2, 6, 3, 7]
    else:
        length, step, inner = (D + 127) // 128 * 32, 16, [4 * k + c for c in range(4) for k in range(4)]
    total = None
    for lo in range(0, length * (ranges or 4), length):
        acc = torch.zeros(len(X), len(W), device="cuda")
        for d0 in range(min(lo, D), min(lo + length, D), step):
            for d in (d0 + c for c in inner):
                if d < D:
                    acc = (X[:, d, None].double() * W[None, :, d].double() + acc.double()).float()
        total = acc if total is None else total + acc
    return total + b


def near_copies(seed, N, K, D, copies=None):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    X = torch.rand(N, D, generator=g, device="cuda")
    base = torch.randn(1, D, generator=g, device="cuda")
    W = base + 1e-7 * torch.randn(K, D, generator=g, device="cuda")
    if copies is not None:  # the others: nothing like them
        other = torch.ones(K, dtype=torch.bool, device="cuda")
        other[copies] = False
        W[other] = torch.randn(int(other.sum()), D, generator=g, device="cuda") * 1e-3
        X *= torch.sign(base)  # scores of the copies above the others'
        X -= 0.9995 * (X @ base.T) / (base @ base.T) * base
    return X.contiguous(), W, torch.zeros(K, device="cuda")


@pytest.mark.parametrize("N,K,ranges", [(5, 32, 4), (24, 32, 4), (4096, 16, 4), (1000, 700, 4),
                                        (2048, 1024, 2), (5120, 1024, 1)])
def test_copies_only(N, K, ranges):
    """Few rows, few identities, split and whole products."""
    require_gpu()
    c = lbpf.Context()
    X, W, b = near_copies(N + K, N, K, c.dim)
    wts = c.weights(W, b)
    S, A = c.score(X, wts)
    _, A2 = c.score(X, wts, want_scores=False)
    rows = slice(0, N, max(1, N // 400))
    want = fixed_order(X[rows], W, b, ranges)
    torch.cuda.synchronize()
    assert torch.equal(A[rows].long(), want.argmax(1))
    assert torch.equal(A2[rows], A[rows])
    assert torch.equal(S[rows].gather(1, A[rows].long()[:, None]), want.max(1, keepdim=True).values)
    wts.close()
    c.close()


@pytest.mark.parametrize("grid,modality,N,K", [((6, 6), lbpf.MOD_BOTH, 20, 300), ((6, 6), lbpf.MOD_BOTH, 300, 60),
                                               ((2, 2), lbpf.MOD_GREY, 33, 40), ((6, 6), lbpf.MOD_BOTH, 2048, 600)])
def test_quarters(grid, modality, N, K):
    """D not a multiple of 32: few rows (D = 4248 and 236), and the kernel whose order
    that is."""
    require_gpu()
    c = lbpf.Context(grid=grid, modality=modality)
    X, W, b = near_copies(N + K, N, K, c.dim)
    wts = c.weights(W, b)
    _, A = c.score(X, wts)
    rows = slice(0, N, max(1, N // 400))
    want = fixed_order(X[rows], W, b, 0)
    torch.cuda.synchronize()
    assert torch.equal(A[rows].long(), want.argmax(1))
    wts.close()
    c.close()


@pytest.mark.parametrize("N,K,ranges", [(4, 6000, 4), (300, 6000, 2), (1100, 6000, 1)])
def test_many_copies_among_others(N, K, ranges):
    """Close ones on both sides of identity 4096, more of them than a wave has lanes."""
    require_gpu()
    c = lbpf.Context()
    copies = torch.randperm(K, generator=torch.Generator().manual_seed(3))[:150].sort().values.cuda()
    X, W, b = near_copies(N, N, K, c.dim, copies)
    wts = c.weights(W, b)
    _, A = c.score(X, wts)
    rows = slice(0, N, max(1, N // 100))
    want = fixed_order(X[rows], W[copies], b[copies], ranges)
    S64 = X[rows].double() @ W.double().T
    torch.cuda.synchronize()
    near = torch.isin(S64.argmax(1), copies)  # the others' best may be a row's
    assert near.sum() >= len(S64) // 4
    assert torch.equal(A[rows].long()[near], copies[want.argmax(1)][near])
    wts.close()
    c.close()


@pytest.mark.parametrize("max_boxes", [24, 600])
def test_pipeline(max_boxes):
    """The captured serving step: one range, few rows and whole tiles."""
    require_gpu()
    c = lbpf.Context()
    n, K = 24, 640
    rng = np.random.default_rng(4)
    planes, boxes = stacked_planes(rng.integers(0, 256, size=(n, 64, 64)).astype(np.uint8),
                                   rng.integers(700, 900, size=(n, 64, 64)).astype(np.uint16))
    _, W, b = near_copies(9, 1, K, c.dim)
    wts = c.weights(W, b)
    pipe = c.pipeline(wts, max_boxes)
    pipe.launch(lbpf.ImageTable(planes), boxes)
    torch.cuda.synchronize()
    want = fixed_order(pipe.hist[:n], W, b, 1)
    assert torch.equal(pipe.argmax[:n].long(), want.argmax(1))
    pipe.close()
    wts.close()
    c.close()


@pytest.mark.parametrize("N,K,ranges", [(5, 1024, 4), (2048, 1024, 2), (5120, 1024, 1)])
def test_noalloc(N, K, ranges):
    """Without the weights' norms: scores that are not small against their sums."""
    require_gpu()
    c = lbpf.Context()
    X, W, b = near_copies(N, N, K, c.dim)
    W += 0.05
    _, A = lbpf.score_noalloc(X, W, b)
    rows = slice(0, N, max(1, N // 400))
    want = fixed_order(X[rows], W, b, ranges)
    torch.cuda.synchronize()
    assert torch.equal(A[rows].long(), want.argmax(1))
    c.close()
