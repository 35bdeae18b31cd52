"""The fp32 products from bf16 parts: against 64 bits at the edges of tiles and slabs, and with special values.

Bound: the leading products of a group of 16 k-values round the running sum once, the other five sums are 2^-8 of it
and less, and splits of a long k meet in at most 64 further additions; a value's three parts drop below 2^-25 of a
product.  Each result is therefore within (K/16 + 64) 2^-24 of the sum of |a b|.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09887_amd import binding
    binding.lib()
    return binding


def within(got, a, b, what):
    got = got.double().cpu().numpy()
    want, size = a @ b, np.abs(a) @ np.abs(b)
    bound = (a.shape[1] / 16 + 64) * 2.0 ** -24 * size + 1e-37
    off = np.abs(got - want) / bound
    assert np.all(off <= 1.0), f"{what}: {off.max():.2f} of the bound"


def data(n, fi, fo, seed):
    r = np.random.default_rng(seed)
    f = lambda *s: r.standard_normal(s).astype(np.float32)
    return f(n, fi), f(fi, fo) * np.float32(0.1), f(fo) * np.float32(0.1), f(n, fo) * np.float32(1e-6)


SHAPES = [(1, 4, 5), (15, 16, 47), (129, 20, 64), (128, 33, 96), (257, 47, 100), (1000, 64, 130), (4100, 130, 48),
          (20000, 128, 128), (70001, 100, 256), (50000, 90, 41)]


@pytest.mark.parametrize("n,fi,fo", SHAPES)
def test_dense_products(B, n, fi, fo):
    X, W, b, g = data(n, fi, fo, n + fi)
    x, w, bias, d = (torch.as_tensor(t).cuda() for t in (X, W, b, g))
    Y = B.tma_dense_fwd(x, w, None, B.TMA_ACT_NONE)
    X, W, g = X.astype(np.float64), W.astype(np.float64), g.astype(np.float64)
    within(Y, X, W, "forward")
    out = B.tma_dense_bwd(x, Y, d, w, B.TMA_ACT_NONE)
    dW, db, dX = out[:3]
    within(dW, X.T, g, "weight gradient")
    within(db.reshape(1, -1), np.ones((1, n)), g, "bias gradient")
    within(dX, g, W.T, "input gradient")


@pytest.mark.parametrize("n,fi,fo", [(300, 64, 47), (1000, 33, 130)])
def test_special_values(B, n, fi, fo):
    X, W, _, g = data(n, fi, fo, 9)
    X[3, 5], X[140, 0], X[141, fi - 1], X[142, 7] = np.inf, -np.inf, np.nan, 3.3e38
    x, w = torch.as_tensor(X).cuda(), torch.as_tensor(W).cuda()
    Y = B.tma_dense_fwd(x, w, None, B.TMA_ACT_NONE).cpu().numpy()
    assert np.array_equal(Y[3], np.where(W[5] > 0, np.inf, -np.inf).astype(np.float32))
    assert np.array_equal(Y[140], np.where(W[0] > 0, -np.inf, np.inf).astype(np.float32))
    assert np.all(np.isnan(Y[141]))
    usual = np.ones(n, dtype=bool)
    usual[[3, 140, 141]] = False
    within(torch.as_tensor(Y[usual]), X[usual].astype(np.float64), W.astype(np.float64), "rows without Inf or NaN")
    # (the weight gradient sums over the rows: a column of X with a special value, and no other, shows it)
    d = torch.as_tensor(g).cuda()
    dW = B.tma_dense_bwd(x, None, d, w, B.TMA_ACT_NONE)[0].cpu().numpy()
    assert np.array_equal(dW[5], np.where(g[3] > 0, np.inf, -np.inf).astype(np.float32))
    assert np.all(np.isnan(dW[fi - 1]))
    rest = np.ones(fi, dtype=bool)
    rest[[0, 5, fi - 1]] = False
    within(torch.as_tensor(dW[rest]), X[:, rest].astype(np.float64).T, g.astype(np.float64), "columns without Inf or NaN")


def test_overflow_and_small_values(B):
    X, W, _, _ = data(200, 48, 64, 4)
    X[10] = 2e38
    W[:, 3] = 1.0
    X[20:40] *= np.float32(2.0 ** -100)
    x, w = torch.as_tensor(X).cuda(), torch.as_tensor(W).cuda()
    Y = B.tma_dense_fwd(x, w, None, B.TMA_ACT_NONE).cpu().numpy()
    assert Y[10, 3] == np.inf
    usual = np.ones(200, dtype=bool)
    usual[10] = False
    X, W = X.astype(np.float64), W.astype(np.float64)
    err = np.abs(Y[usual].astype(np.float64) - X[usual] @ W)
    assert np.all(err <= 67 * 2.0 ** -24 * (np.abs(X[usual]) @ np.abs(W)))
