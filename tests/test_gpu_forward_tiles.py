"""Forward products of fp32 storage by their bits, on both sides of the lines between the tiles that they can take: one order of the sum for all of them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_forward_order import B, dev, normal, product_in_order  # noqa: F401


# the last row before a wider tile and the first of it, cut and whole; short k, a k that ends inside a slab, one past 96
@pytest.mark.parametrize("n,fi,fo", [(24576, 17, 96), (24577, 100, 96), (40961, 33, 80), (16385, 98, 150), (21761, 100, 130), (65537, 97, 160), (70977, 20, 150), (12289, 97, 256),
                                     (28673, 97, 200), (57345, 18, 100), (49153, 96, 64), (65537, 33, 64), (16385, 99, 300), (70001, 15, 33), (32769, 31, 32)])
def test_dense_product(B, n, fi, fo):
    X, W, b = normal(1, n, fi), normal(2, fi, fo), normal(3, fo)
    Y = B.tma_dense_fwd(dev(X), dev(W), dev(b), B.TMA_ACT_RELU)
    assert np.array_equal(Y.cpu().numpy(), np.maximum(product_in_order(X, W) + b, np.float32(0)))
