"""FP32 scoring on the BF16 matrix cores (three exact parts per value, six
products): error against the FP64 product, values that are no number, and the
edges of tiles, stages and splits.

Tolerance. Every value is split exactly; the dropped products are below 2^-25 of
|x w|. A flush sums 8 stages of 32 columns, 96 MFMAs of 16 products each, with
truncation: 96 x 2^-23 of the flush's sum of |x w| at most; the running sum adds
one rounding of 2^-24 per flush, and partials and the bias a few more. So
|S - S64| <= (96 * 2^-23 + (D / 256 + 20) * 2^-24) * (sum |x w| + |b|): 1.5e-5 at
D = 7552, above the FP32 bar of 1e-5 of the condition scale, which is used."""
import numpy as np
import pytest
import torch

from paper_1504_01883_amd import lbpf
from tests.gpu_util import require_gpu, score_tolerance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    c = lbpf.Context()
    yield c
    c.close()


def scores(ctx, X, W, b, **kw):
    wts = ctx.weights(torch.from_numpy(W).cuda(), torch.from_numpy(b).cuda())
    S, A = ctx.score(torch.from_numpy(X).cuda(), wts, **kw)
    torch.cuda.synchronize()
    wts.close()
    return None if S is None else S.cpu().numpy(), A.cpu().numpy()


@pytest.mark.parametrize("N,K", [(257, 2049), (1000, 700), (513, 1025), (2305, 640)])
@pytest.mark.parametrize("spread", [0, 3])
def test_scores(ctx, N, K, spread):
    """Tiles with remainders on both sides, split 2 to 16 ways over ranges of
    unequal length; spread > 0: values over many decades."""
    rng = np.random.default_rng(N + K)
    X = rng.random((N, ctx.dim), dtype=np.float32)
    W = rng.standard_normal((K, ctx.dim), dtype=np.float32)
    if spread:
        X *= np.exp(spread * rng.standard_normal(X.shape, dtype=np.float32))
        W *= np.exp(spread * rng.standard_normal(W.shape, dtype=np.float32))
    b = rng.standard_normal(K).astype(np.float32)
    S, A = scores(ctx, X, W, b)
    S64 = X.astype(np.float64) @ W.astype(np.float64).T + b
    assert (np.abs(S - S64) <= score_tolerance(X, W, b)).all()
    assert np.array_equal(A, np.argmax(S, axis=1))
    _, A2 = scores(ctx, X, W, b, want_scores=False)
    clear = np.sort(S64, axis=1)
    clear = clear[:, -1] - clear[:, -2] > 2 * score_tolerance(X, W, b).max(axis=1)
    assert np.array_equal(A2[clear], A[clear])


@pytest.mark.parametrize("grid", [(1, 16), (2, 16), (8, 8)])
def test_error_against_fp32_matrix_cores(grid):
    """Half the FP32 matrix cores' root mean square error at most (their kernel
    still serves training and device row counts; torch's FP32 product stands for
    it here: 2^-24 sqrt(D) of the result's spread, whichever library runs)."""
    require_gpu()
    c = lbpf.Context(grid=grid)
    if c.dim % 32:
        pytest.skip("the FP32 path")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    X = torch.rand(1024, c.dim, generator=g, device="cuda")
    W = torch.randn(1024, c.dim, generator=g, device="cuda")
    b = torch.zeros(1024, device="cuda")
    wts = c.weights(W, b)
    S, _ = c.score(X, wts)
    ref = X.double() @ W.double().T
    torch.cuda.synchronize()
    spread = 2.0 ** -24 * c.dim ** 0.5 * ref.std()
    assert (S.double() - ref).square().mean().sqrt() <= spread
    wts.close()
    c.close()


def test_not_numbers(ctx):
    """Infinities, NaNs, the largest and lowest finite values and sums that
    overflow give what FP32 arithmetic gives."""
    rng = np.random.default_rng(8)
    N, K, D = 600, 1100, ctx.dim
    X = rng.random((N, D), dtype=np.float32)
    W = rng.standard_normal((K, D), dtype=np.float32)
    b = np.zeros(K, np.float32)
    top = np.finfo(np.float32).max
    W[:, 5] = np.abs(W[:, 5]) + 0.5
    W[7, 5] = 0.0
    X[3, 5] = np.inf             # +inf, NaN where the weight is 0
    X[4, 5], X[4, 6] = np.inf, -np.inf
    X[5, 9] = np.nan
    W[11, 20] = -np.inf
    X[:, 20] = 0.25
    X[8, 20] = 0.0               # 0 * -inf
    W[13, 30] = -top             # a mask: finite products
    W[14, 30] = top
    X[:, 30] = 2.0 ** -20
    X[9, 30] = 0.0
    X[10, 40] = top
    W[:, 40] = 2.0 ** -30
    X[12, 50:52] = top           # overflows
    W[:, 50:52] = 2.0
    S, _ = scores(ctx, X, W, b)
    with np.errstate(all="ignore"):
        S64 = X.astype(np.float64) @ W.astype(np.float64).T
        want = np.where(np.abs(S64) > top, np.sign(S64) * np.inf, S64)
        cond = np.abs(X).astype(np.float64) @ np.abs(W).astype(np.float64).T
    assert np.array_equal(np.isnan(S), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(S[inf], want[inf].astype(np.float32))
    fin = np.isfinite(want)
    assert (np.abs(S[fin] - want[fin]) <= 1e-5 * cond[fin]).all()
    assert np.isfinite(S[20:, 13]).all() and np.isfinite(S[9, 13:15]).all()


@pytest.mark.parametrize("ex,ew", [(-100, 90), (-112, 100), (-125, 100), (-140, 120), (-60, -60)])
def test_small_values(ctx, ex, ew):
    """Values and products near FP32's smallest, beside a column of larger ones
    that meet zeros: the FP32 bar, and FP32's own last place for each product."""
    rng = np.random.default_rng(9)
    N, K, D = 300, 1100, ctx.dim
    X = np.ldexp(rng.random((N, D), dtype=np.float32), ex)
    W = np.ldexp(rng.standard_normal((K, D), dtype=np.float32), ew)
    X[::2, 7] = 1.0
    W[:, 7] = 0.0
    S, _ = scores(ctx, X, W, np.zeros(K, np.float32))
    X, W = X.astype(np.float64), W.astype(np.float64)
    tol = 1e-5 * (np.abs(X) @ np.abs(W).T) + D * 2.0 ** -149
    assert (np.abs(S - X @ W.T) <= tol).all()
