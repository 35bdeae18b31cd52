"""The fp32 forward products bit for bit at every tile and at the edges of their slabs of 16 k-values: halves that end
inside a slab, weights whose last row may not be fetched in whole pieces, rows at any pitch and offset, fewer slabs than are
kept in flight.  What lies around the arrays is NaN and must reach nothing.  The order of the sums is the one that
test_gpu_forward_order.py states."""
import numpy as np
import pytest

from test_gpu_forward_order import B, dev, normal, product_in_order  # noqa: F401  (B: the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def inside(a, pitch, before):
    """`a` on the GPU at an offset of `before` elements, rows `pitch` apart, NaN around and between the rows."""
    n, f = a.shape
    t = torch.full((before + n * pitch + 8,), float("nan"), device="cuda")
    view = t[before:before + n * pitch].view(n, pitch)[:, :f]
    view.copy_(dev(a))
    return view


# 64 x 32, 64 x 64, 64 x 128, 128 x 64, 128 x 96, 128 x 128, 128 x 160; k of one slab and less, of two, with every kind of rest
@pytest.mark.parametrize("n,fi,fo", [(70, 1, 20), (65, 16, 32), (129, 17, 33), (200, 31, 64), (24700, 18, 128), (49300, 9, 50), (25700, 15, 90),
                                     (25700, 33, 96), (49153, 20, 128), (25729, 14, 150), (25700, 19, 160), (300, 48, 161), (131, 40, 3), (1, 64, 2), (130, 256, 1), (70, 35, 1),
                                     (70, 34, 2), (70, 33, 2)])
@pytest.mark.parametrize("pitch,before", [(0, 0), (3, 1)])
def test_dense(B, n, fi, fo, pitch, before):
    X, W, b = normal(n, n, fi), normal(2, fi, fo), normal(3, fo)
    Y = B.tma_dense_fwd(inside(X, fi + pitch, before), inside(W, fo, before), dev(b), B.TMA_ACT_RELU).cpu().numpy()
    assert np.array_equal(Y, np.maximum(product_in_order(X, W) + b, 0))


# [H | M] whose halves end at every place of a slab (4 f_out > 2 f_in: the rows are aggregated first), and H [W_self | W_neigh]
@pytest.mark.parametrize("n,fi,fo", [(90, f, 70) for f in (1, 8, 15, 16, 17, 20, 32, 45, 50)] + [(200, 64, f) for f in (4, 15, 17, 31)] + [(25700, 50, 23)])
@pytest.mark.parametrize("before", [0, 2])
def test_halves(B, n, fi, fo, before):
    X, Ws, Wn, b = normal(1, n, fi), normal(2, fi, fo), normal(3, fi, fo), normal(4, fo)
    rowptr = dev(np.arange(n + 1, dtype=np.int32))           # every row has one neighbour: the next
    order = (np.arange(n) + 1) % n
    inv = torch.ones(n, device="cuda")
    out = B.tma_sage_layer_fwd(rowptr, dev(order.astype(np.int32)), inv, inside(X, fi + before, before), inside(Ws, fo, before),
                               inside(Wn, fo, before), dev(b), B.TMA_ACT_NONE)[1].cpu().numpy()[:, :fo]
    if B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_F32):
        want = product_in_order(np.concatenate([X, X[order]], 1), np.concatenate([Ws, Wn], 0)) + b
    else:
        want = product_in_order(X, Wn)[order] + product_in_order(X, Ws) + b
    assert np.array_equal(out, want)
