"""The identity of a row whose best scores are close: it is the one that FP32 sums in
one fixed order give (an FMA per column; each eight columns as 0 4 1 5 2 6 3 7; the
sums of 1, 2 or 4 ranges of D added in order, then the bias), whichever kernel made
the scores. Exact: the sums are emulated on the host to the last bit."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def fixed_order(X, W, b, ranges):
    X, W = X.astype(np.longdouble), W.astype(np.longdouble)
    length = X.shape[1] // ranges
    total = None
    for r in range(ranges):
        acc = np.zeros((len(X), len(W)), np.float32)
        for d in range(r * length, (r + 1) * length, 8):
            for c in (0, 4, 1, 5, 2, 6, 3, 7):
                acc = (np.multiply.outer(X[:, d + c], W[:, d + c]) + acc).astype(np.float32)
        total = acc if total is None else total + acc
    return total + b


@pytest.mark.parametrize("N,K,ranges", [(5, 1024, 4), (70, 2100, 4), (300, 1100, 4), (2048, 1024, 2),
                                        (5120, 1024, 1)])
def test_near_duplicates(N, K, ranges):
    """Twenty identities that differ by a few last places, over few-rows, split and
    whole products; argmax alone and with scores."""
    require_gpu()
    c = lbpf.Context()
    rng = np.random.default_rng(N)
    X = (rng.random((N, c.dim), dtype=np.float32) / c.dim).astype(np.float32)
    W = rng.standard_normal((K, c.dim), dtype=np.float32)
    b = (0.01 * rng.standard_normal(K)).astype(np.float32)
    group = rng.permutation(K)[:20]
    W[group] = (W[group[0]] + 0.1) * (1 + 3e-7 * rng.standard_normal((20, 1))).astype(np.float32)
    b[group] = 2.0
    wts = c.weights(torch.from_numpy(W).cuda(), torch.from_numpy(b).cuda())
    S, A = c.score(torch.from_numpy(X).cuda(), wts)
    _, A2 = c.score(torch.from_numpy(X).cuda(), wts, want_scores=False)
    torch.cuda.synchronize()
    S, A, A2 = S.cpu().numpy(), A.cpu().numpy(), A2.cpu().numpy()
    rows = rng.permutation(N)[:4]
    group = np.sort(group)
    want = fixed_order(X[rows], W[group], b[group], ranges)
    assert np.array_equal(S[np.ix_(rows, group)], want)
    assert np.array_equal(A[rows], group[want.argmax(1)])
    assert np.array_equal(A, S.argmax(1))
    assert np.array_equal(A2[rows], A[rows])
    wts.close()
    c.close()


def test_many_alike():
    """More equal scores than a wave holds: rows of zeros against one bias."""
    require_gpu()
    c = lbpf.Context()
    X = torch.zeros(300, c.dim, device="cuda")
    W = torch.randn(1100, c.dim, device="cuda")
    b = torch.full((1100,), 0.25, device="cuda")
    b[3] = 0.125
    b[0] = 0.125
    wts = c.weights(W, b)
    S, A = c.score(X, wts)
    torch.cuda.synchronize()
    assert torch.equal(S, b.expand_as(S)) and (A == 1).all()
    wts.close()
    c.close()
