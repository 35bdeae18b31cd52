"""Backward products of fewer than 65,536 rows, on both sides of each line of the rule that chooses their tile: input gradients by their bits (one order of the
sum for every tile), weight and bias gradients against 64 bits within the bound of test_gpu_products.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_forward_order import B, dev, normal, product_in_order  # noqa: F401
from test_gpu_products import within


# 256 tiles of 64 x 64 and one more, whole and cut; 96 columns and 512 on each side of the wider tile; slabs of 16 with a rest
@pytest.mark.parametrize("n,fi,fo", [(16384, 64, 16), (16385, 64, 17), (16385, 33, 31), (33000, 96, 20), (49153, 96, 33), (49153, 70, 15), (8193, 512, 18), (16384, 512, 21),
                                     (16321, 450, 5), (40004, 150, 16)])
def test_input_gradient(B, n, fi, fo):
    W, g, h = normal(2, fi, fo), normal(5, n, fo), normal(6, n, fo)
    dX = B.tma_dense_bwd(torch.zeros((n, fi), device="cuda"), dev(h), dev(g), dev(W), B.TMA_ACT_RELU)[2]
    assert np.array_equal(dX.cpu().numpy(), product_in_order(np.where(h > 0, g, np.float32(0)), np.ascontiguousarray(W.T)))


@pytest.mark.parametrize("n,fi,fo", [(300, 520, 530), (5000, 200, 150), (5001, 320, 70), (14600, 512, 96), (20001, 257, 65), (40004, 180, 150), (40004, 512, 256), (65535, 64, 96)])
def test_weight_gradient(B, n, fi, fo):
    X, g, h = normal(1, n, fi), normal(5, n, fo), normal(6, n, fo)
    dW, db = B.tma_dense_bwd(dev(X), dev(h), dev(g), torch.zeros((fi, fo), device="cuda"), B.TMA_ACT_RELU, need_dX=False)[:2]
    X, d = X.astype(np.float64), np.where(h > 0, g, 0).astype(np.float64)
    within(dW, X.T, d, "weight gradient")
    within(db.reshape(1, -1), np.ones((1, n)), d, "bias gradient")
