"""The fp32 products, forward and backward: against 64 bits at the edges of tiles and slabs, and with special values.

Bound of the backward products (from bf16 parts): the leading products of a group of 16 k-values round the running sum
once, the other five sums are 2^-8 of it and less, and splits of a long k meet in at most 64 further additions; what the
parts of a value leave out of a product is below 2^-24 of it, one of the 64.  Each result is therefore within
(K/16 + 64) 2^-24 of the sum of |a b|, and within K roundings at the end of the range (2^-149 each).  A forward product
rounds once per k-value, K 2^-24 of the sum at most: less than that bound up to K = 68, and above it by roundings that would
all have to fall the same way (its bits are pinned in test_gpu_forward_order.py).
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
    bound = (a.shape[1] / 16 + 64) * 2.0 ** -24 * size + a.shape[1] * 2.0 ** -149
    off = np.abs(got - want) / bound
    assert np.all(off <= 1.0), f"{what}: {off.max():.2f} of the bound"


def data(n, fi, fo, seed):
    r = np.random.default_rng(seed)
    f = lambda *s: r.standard_normal(s).astype(np.float32)
    return f(n, fi), f(fi, fo) * np.float32(0.1), f(fo) * np.float32(0.1), f(n, fo) * np.float32(1e-6)


SHAPES = [(1, 1, 2), (1, 3, 1), (2, 1, 4), (3, 5, 6), (1, 7, 3), (40, 2, 66), (1, 4, 5), (15, 16, 47), (129, 20, 64), (128, 33, 96), (257, 47, 100), (1000, 64, 130), (4100, 130, 48),
          (20000, 128, 128), (70001, 100, 256), (50000, 90, 41)]
# backward products of 65,536 rows and more are the ones from bf16 parts: every tile, its edges and its rest of k
MANY_ROWS = [(65536, 64, 64), (65537, 20, 66), (65600, 96, 100), (66000, 33, 96), (65599, 128, 41), (70000, 130, 130), (65550, 250, 24), (65543, 5, 300)]


@pytest.mark.parametrize("n,fi,fo", SHAPES + MANY_ROWS)
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


@pytest.mark.parametrize("pitch,offset", [(0, 0), (1, 0), (3, 1), (2, 2)])
@pytest.mark.parametrize("n,fi,fo", [(130, 90, 150), (1000, 33, 41), (257, 64, 7), (77, 5, 300), (65601, 90, 150), (65537, 33, 41)])
def test_rows_at_any_address(B, n, fi, fo, pitch, offset):
    """The same products with rows that are neither aligned nor a multiple of four apart, in arrays that end with them."""
    X, W, _, g = data(n, fi, fo, n + pitch)

    def placed(t):
        flat = torch.full(((t.shape[0] - 1) * (t.shape[1] + pitch) + t.shape[1] + offset,), float("nan"), device="cuda")
        view = flat.as_strided(t.shape, (t.shape[1] + pitch, 1), offset)
        view.copy_(torch.as_tensor(t))
        return view

    x, d, w = placed(X), placed(g), torch.as_tensor(W).cuda()
    Y = B.tma_dense_fwd(x, w, None, B.TMA_ACT_NONE)
    X, W, g = X.astype(np.float64), W.astype(np.float64), g.astype(np.float64)
    within(Y, X, W, "forward")
    dW, db, dX = B.tma_dense_bwd(x, None, d, w, B.TMA_ACT_NONE)[:3]
    within(dW, X.T, g, "weight gradient")
    within(db.reshape(1, -1), np.ones((1, n)), g, "bias gradient")
    within(dX, g, W.T, "input gradient")


@pytest.mark.parametrize("n,fi,fo,pitch", [(700, 90, 150, 0), (701, 33, 41, 3), (300, 150, 41, 0), (50, 6, 130, 1), (2, 3, 5, 0)])
def test_sage_layer_at_any_width(B, n, fi, fo, pitch):
    """[H | M] with halves that are no multiples of four, in both orders of the layer's two steps."""
    r = np.random.default_rng(n)
    X, Ws, b, g = data(n, fi, fo, n)
    Wn = data(n, fi, fo, n + 1)[1]
    A = np.triu(r.random((n, n)) < 4.0 / n, 1)
    A = A | A.T
    deg = A.sum(1)
    rowptr, colidx = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32), np.nonzero(A)[1].astype(np.int32)
    inv = np.where(deg > 0, 1.0 / np.maximum(deg, 1), 0.0)
    x = torch.zeros((n, fi + pitch), device="cuda")[:, :fi]
    x.copy_(torch.as_tensor(X))
    c = lambda t: torch.as_tensor(t).cuda()
    graph = c(rowptr), c(colidx) if colidx.size else torch.zeros(1, dtype=torch.int32, device="cuda"), c(inv.astype(np.float32))
    M, out = B.tma_sage_layer_fwd(*graph, x, c(Ws), c(Wn), c(b), B.TMA_ACT_NONE)
    X, Ws, Wn, b, g64 = (t.astype(np.float64) for t in (X, Ws, Wn, b, g))
    mean = inv[:, None] * (A @ X)
    tol = 2e-6      # sums of a few fp32 roundings per term, far below the terms' own sizes
    close = lambda got, want: np.linalg.norm(got.double().cpu().numpy() - want) <= tol * np.linalg.norm(want) + 1e-30
    assert close(out, X @ Ws + mean @ Wn + b)
    dWs, dWn, db, dH = B.tma_sage_layer_bwd(*graph, x, M, out, c(g), c(Ws.astype(np.float32)), c(Wn.astype(np.float32)),
                                            B.TMA_ACT_NONE)[:4]
    assert close(dWs, X.T @ g64) and close(dWn, mean.T @ g64) and close(db, g64.sum(0))
    assert close(dH, g64 @ Ws.T + A.T @ (inv[:, None] * (g64 @ Wn.T)))


def ring(n):
    """Every node with the two beside it: rowptr, colidx, inv_deg on the GPU, and the mean over a row's neighbours."""
    v = np.arange(n)
    colidx = np.sort(np.stack([(v - 1) % n, (v + 1) % n], 1), 1).astype(np.int32).reshape(-1)
    graph = [torch.as_tensor(t).cuda() for t in (np.arange(0, 2 * n + 1, 2, dtype=np.int32), colidx, np.full(n, 0.5, np.float32))]
    return graph, lambda X: 0.5 * (np.roll(X, 1, 0) + np.roll(X, -1, 0))


# widths that are 3 mod 4 in padded rows, at the row counts of the 64 x 64 and of the 128 x 64 tiles; NaN behind the last row
@pytest.mark.parametrize("n,fi,fo", [(300, 63, 20), (40000, 63, 20), (40000, 51, 7), (70000, 63, 20)])
def test_transform_first_weight_gradient_at_the_end_of_the_rows(B, n, fi, fo):
    graph, mean = ring(n)
    X, Ws, _, g = data(n, fi, fo, n)
    Wn = data(n, fi, fo, n + 1)[1]
    ld = (fi + 3) // 4 * 4
    x = torch.full((n + 1, ld), float("nan"), device="cuda")
    x[:n] = 0.0
    x = x[:n, :fi]
    x.copy_(torch.as_tensor(X))
    c = lambda t: torch.as_tensor(t).cuda()
    M, out = B.tma_sage_layer_fwd(*graph, x, c(Ws), c(Wn), c(np.zeros(fo, np.float32)), B.TMA_ACT_NONE)
    dWs, dWn, db = B.tma_sage_layer_bwd(*graph, x, M, out, c(g), c(Ws), c(Wn), B.TMA_ACT_NONE)[:3]
    X, g = X.astype(np.float64), g.astype(np.float64)
    within(dWs, X.T, g, "self weights")
    within(db.reshape(1, -1), np.ones((1, n)), g, "bias")
    # (the gathered gradient itself is rounded once per element: one more 2^-24 per term than within() has, and it has 64 to spare)
    within(dWn, X.T, mean(g), "neighbour weights")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,fi,fo", [(700, 150, 41), (301, 99, 24), (60, 30, 7), (129, 65, 16), (65700, 150, 41), (65537, 99, 24)])
def test_row_padding_leaves_no_trace(B, n, fi, fo, dtype):
    """The transform-first layer on rows padded to a multiple of 16 bytes: whatever the padding holds, the same bits."""
    graph, _ = ring(n)
    X, Ws, b, g = data(n, fi, fo, n)
    Wn = data(n, fi, fo, n + 1)[1]
    c = lambda t: torch.as_tensor(t).cuda()

    def padded(t, fill):
        p = B._padded(*t.shape, dtype, "cuda")
        p._base.fill_(fill)
        return p.copy_(torch.as_tensor(t))

    got = []
    for fill in (0.0, float("nan")):
        x = padded(X, fill)
        M, out = B.tma_sage_layer_fwd(*graph, x, c(Ws), c(Wn), c(b), B.TMA_ACT_RELU)
        if fill == 0.0:
            first = out.clone()      # (the backward pass of both from the same output)
        for act in (B.TMA_ACT_RELU, B.TMA_ACT_NONE):
            got.append([out, *B.tma_sage_layer_bwd(*graph, x, M, padded(first, fill), padded(g, fill), c(Ws), c(Wn), act)[:4]])
    assert not B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_F32 if dtype == torch.float32 else B.TMA_BF16)
    for clean, dirty in zip(got[0] + got[1], got[2] + got[3]):
        assert torch.isfinite(clean.float()).all() and torch.equal(clean, dirty)


@pytest.mark.parametrize("n,fi,fo", [(300, 64, 47), (1000, 33, 130), (65600, 64, 47), (65600, 33, 130)])
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


# Both ends of the fp32 range: operands down to the smallest normal numbers and below, products up to its end
@pytest.mark.parametrize("xe,we,ge", [(0, 0, -126), (20, 12, -140), (-70, -60, -50), (-120, 10, 100), (-126, 0, 0), (60, -126, -20), (100, -140, 0),
                                      (110, 100, -115), (-133, 0, 110)])
@pytest.mark.parametrize("n", [300, 65600])
def test_backward_products_over_the_whole_range(B, n, xe, we, ge):
    X, W, _, g = data(n, 40, 72, 4)
    X, W, g = (np.ldexp(t, e).astype(np.float32) for t, e in ((X, xe), (W * 8, we), (g * 2 ** 20, ge)))
    X[::7], W[::5], g[:, ::3] = np.ldexp(X[::7], -3), np.ldexp(W[::5], 3), np.ldexp(g[:, ::3], -2)
    x, w, d = (torch.as_tensor(t).cuda() for t in (X, W, g))
    dW, db, dX = B.tma_dense_bwd(x, None, d, w, B.TMA_ACT_NONE)[:3]
    X, W, g = (t.astype(np.float64) for t in (X, W, g))
    within(dW, X.T, g, "weight gradient")
    within(dX, g, W.T, "input gradient")
