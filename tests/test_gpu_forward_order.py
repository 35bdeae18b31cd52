"""The order of a forward sum, bit for bit (fp32).

What a layer puts out is compared with zero, in its own ReLU or in a decision further on; a unit within a rounding of zero
falls on the other side when its sum is taken in another order, and in a batch of some thousand rows one such unit is worth
1e-4 to 5e-4 of the weights' gradient.  So the order belongs to the result:
  products     c <- fma(a[k], b[k], c), k = 0, 4, 1, 5, 2, 6, 3, 7 of every eight k-values, one accumulator;
  aggregation  neighbours in the order of the list; a weighted one is rounded before it is added where rows are whole
               16-byte pieces, and inside the addition where they are not.
Backward products of fewer than 65,536 rows keep the order too: Adam turns the last bits of a small gradient into weights that
decide otherwise in the next step.
An fma is taken here as the sum in 64 bits rounded to 32 (exact but for a second rounding, once in 2^29).
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


def dev(a):
    return torch.as_tensor(a).cuda()


def normal(seed, *shape):
    return np.random.default_rng(seed).standard_normal(shape).astype(np.float32)


def fma(a, b, c):
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


def product_in_order(a, b):
    c = np.zeros((a.shape[0], b.shape[1]), np.float32)
    for g in range(0, a.shape[1], 8):
        for k in (0, 4, 1, 5, 2, 6, 3, 7):
            if g + k < a.shape[1]:
                c = fma(a[:, g + k, None], b[None, g + k], c)
    return c


def graph(n, degrees, seed):
    """Rows of the given lengths (repeated over the n rows), neighbours spread over all rows, in ascending order."""
    first = np.random.default_rng(seed).integers(0, n, n)
    lists = []
    for v in range(n):
        d = degrees[v % len(degrees)]
        lists.append(np.sort((first[v] + np.arange(d) * max(1, n // (d + 1))) % n).astype(np.int32))
    rowptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)
    return rowptr, np.concatenate(lists)


# the tiles' edges, both sides of the tile rule (384 tiles of 128 x 128), 96 columns, widths of every remainder of four
@pytest.mark.parametrize("n,fi,fo", [(1, 3, 2), (2, 1, 4), (127, 8, 64), (130, 17, 65), (333, 150, 70), (257, 90, 150), (1000, 63, 41),
                                     (49153, 20, 96), (49300, 24, 100), (49153, 31, 47)])
def test_dense_product(B, n, fi, fo):
    X, W, b = normal(1, n, fi), normal(2, fi, fo), normal(3, fo)
    Y = B.tma_dense_fwd(dev(X), dev(W), dev(b), B.TMA_ACT_NONE)
    assert np.array_equal(Y.cpu().numpy(), product_in_order(X, W) + b)


# the aggregate-first form (2 F_out > F_in) and the transform-first one; halves of every remainder of four
@pytest.mark.parametrize("n,fi,fo", [(300, 64, 64), (301, 90, 150), (515, 33, 20), (200, 30, 41), (77, 5, 6), (24700, 20, 132), (300, 128, 47),
                                     (301, 150, 41), (400, 66, 7)])
def test_sage_layer(B, n, fi, fo):
    X, Ws, Wn, b = normal(1, n, fi), normal(2, fi, fo), normal(3, fi, fo), normal(4, fo)
    rowptr, colidx = graph(n, [0, 1, 3, 9], n)
    deg = np.diff(rowptr)
    inv = np.where(deg > 0, 1.0 / np.maximum(deg, 1), 0.0).astype(np.float32)
    g = dev(rowptr), dev(colidx), dev(inv)
    M, out = B.tma_sage_layer_fwd(*g, dev(X), dev(Ws), dev(Wn), dev(b), B.TMA_ACT_NONE)
    if B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_F32):
        M = M.cpu().numpy()
        assert np.array_equal(M, mean_in_order(rowptr, colidx, inv, X))
        want = product_in_order(np.concatenate([X, M], 1), np.concatenate([Ws, Wn], 0)) + b
    else:
        Ys, Yn = product_in_order(X, Ws), product_in_order(X, Wn)
        total = sum_in_order(rowptr, colidx, Yn, lambda s, x, _: s + x)
        want = total * inv[:, None] + Ys + b
    assert np.array_equal(out.cpu().numpy(), want)


def sum_in_order(rowptr, colidx, X, step):
    out, deg = np.zeros_like(X), np.diff(rowptr)
    for j in range(int(deg.max())):
        v = np.nonzero(deg > j)[0]
        u = colidx[rowptr[v] + j]
        out[v] = step(out[v], X[u], u)
    return out


def mean_in_order(rowptr, colidx, inv, X):
    return sum_in_order(rowptr, colidx, X, lambda s, x, _: s + x) * inv[:, None]


# rows that are no multiples of 16 bytes: up to 256 entries in the list's order, however long their neighbours are
@pytest.mark.parametrize("f,pitch", [(90, 0), (41, 0), (128, 2), (5, 3), (255, 0)])
def test_mean_of_rows_at_any_address(B, f, pitch):
    n = 700
    rowptr, colidx = graph(n, [2, 0, 25, 256, 5, 1, 24], f)
    X, deg = normal(f, n, f), np.diff(rowptr)
    inv = np.where(deg > 0, 1.0 / np.maximum(deg, 1), 0.0).astype(np.float32)
    x = torch.zeros((n, f + pitch), device="cuda")[:, :f]
    x.copy_(dev(X))
    M = B.tma_mean_aggregate(dev(rowptr), dev(colidx), dev(inv), x, out=torch.empty((n, f), device="cuda"))
    assert np.array_equal(M.cpu().numpy(), mean_in_order(rowptr, colidx, inv, X))


@pytest.mark.parametrize("f", [64, 100, 90, 33])
def test_gcn_weights(B, f):
    n = 600
    rowptr, colidx = graph(n, [0, 1, 3, 9, 24], f)
    X = normal(f, n, f)
    s = B.tma_gcn_norm(dev(rowptr))
    M, _ = B.tma_gcn_layer_fwd(dev(rowptr), dev(colidx), s, dev(X), dev(normal(1, f, f + 7)), dev(normal(2, f + 7)), B.TMA_ACT_NONE)
    s = s.cpu().numpy()
    if f % 4 == 0:
        total = sum_in_order(rowptr, colidx, X, lambda t, x, u: t + s[u, None] * x)
    else:
        total = sum_in_order(rowptr, colidx, X, lambda t, x, u: fma(s[u, None], x, t))
    want = fma(s[:, None], X, total) * s[:, None]
    assert np.array_equal(M.cpu().numpy().reshape(-1)[:n * f].reshape(n, f), want)


@pytest.mark.parametrize("n,fi,fo", [(1, 5, 3), (127, 64, 40), (300, 33, 41), (500, 130, 70), (4097, 24, 17), (40000, 200, 20), (65535, 16, 12)])
def test_input_gradient_of_few_rows(B, n, fi, fo):
    W, g = normal(2, fi, fo), normal(5, n, fo)
    dX = B.tma_dense_bwd(torch.zeros((n, fi), device="cuda"), None, dev(g), dev(W), B.TMA_ACT_NONE, need_dbias=False)[2]
    assert np.array_equal(dX.cpu().numpy(), product_in_order(g, np.ascontiguousarray(W.T)))


# up to 128 rows are one range of the sum over the rows; longer ones are tested by their error in test_gpu_products.py
@pytest.mark.parametrize("n,fi,fo", [(1, 5, 3), (96, 64, 40), (128, 33, 41), (100, 260, 130), (128, 128, 300)])
def test_weight_gradient_of_few_rows(B, n, fi, fo):
    X, g = normal(1, n, fi), normal(5, n, fo)
    dW = B.tma_dense_bwd(dev(X), None, dev(g), torch.zeros((fi, fo), device="cuda"), B.TMA_ACT_NONE, need_dX=False)[0]
    assert np.array_equal(dW.cpu().numpy(), product_in_order(np.ascontiguousarray(X.T), g))
