"""bf16 products of dense layers and of layers that transform first, of fewer than 65,536 rows, on both sides of the lines between tiles of 64 x 64 and wider ones.
Operands are -1, 0 and 1, so that the sums are exact (stored in bf16 they stay below 256).  The names of the launches say which tile ran."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_stream_exact import B, equal, masked, product, ring, signs  # noqa: F401


def tiles_are(B, call, narrow):
    """What `call` returns; narrow: product -> whether its launch has tiles of 64 x 64."""
    B.tma_profile_begin(None)
    out = call()
    names = list(B.tma_profile_end())
    for what, so in narrow.items():
        assert ["_64x64" in n for n in names if n.startswith(what)] == [so], (what, names)
    return out


@pytest.mark.parametrize("n,fi,fo,relu,data,weight", [
    (1, 64, 64, False, True, True),
    (8192, 128, 64, False, True, True), (8193, 128, 64, True, False, True),     # against tiles of 128 x 64
    (16385, 128, 64, False, True, False), (16384, 96, 48, True, False, True),
    (28672, 256, 128, True, True, True), (28673, 256, 128, False, False, False),    # 128 x 128
    (49025, 64, 128, False, True, True), (65535, 128, 100, True, False, False),
    (4097, 130, 66, True, True, True), (8193, 130, 66, False, False, True),         # rows that are no groups of four
])
def test_dense(B, n, fi, fo, relu, data, weight):
    pitch = (fo + 3) // 4 * 4
    X, W, g, h = signs(1, n, fi), signs(2, fi, fo), signs(3, n, fo, pitch), signs(4, n, fo, pitch)
    d = masked(g, h) if relu else g
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    dW, db, dX = tiles_are(B, lambda: B.tma_dense_bwd(X, h, g, W.float(), act)[:3], {"gemm_dense_bwd_data": data, "gemm_dense_bwd_weight": weight})
    equal(dX, product(d, W.T), "input gradient")
    equal(dW, product(X.T, d), "weight gradient")
    equal(db, d.double().sum(0), "bias gradient")


@pytest.mark.parametrize("n,fi,fo,forward,weight", [
    (1, 128, 16, True, True), (8192, 256, 47, True, False), (8193, 256, 47, False, True), (12289, 256, 47, False, False), (16385, 256, 47, True, True),
    (4097, 512, 100, False, True), (24449, 200, 47, True, False), (65535, 128, 47, False, False),
])
def test_transform_first(B, n, fi, fo, forward, weight):
    assert not B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16)
    rowptr, nxt, prev, inv = ring(n)
    X, Ws, Wn, g = signs(1, n, fi, (fi + 1) // 2 * 2 + 2), signs(2, fi, fo), signs(3, fi, fo), signs(4, n, fo, (fo + 7) // 8 * 8)
    w = Ws.float(), Wn.float()
    M, out = tiles_are(B, lambda: B.tma_sage_layer_fwd(rowptr, nxt, inv, X, *w, torch.zeros(fo, device="cuda"), B.TMA_ACT_NONE), {"gemm_tf_fwd": forward})
    equal(out, product(X, Ws) + product(X, Wn).roll(-1, 0), "forward")
    dW = tiles_are(B, lambda: B.tma_sage_layer_bwd(rowptr, prev, inv, X, X, None, g, *w, B.TMA_ACT_NONE), {"gemm_tf_bwd_weight": weight, "gemm_tf_bwd_data": False})
    back = torch.cat([g, g.roll(1, 0)], 1)
    equal(torch.cat(dW[:2], 1), product(X.T, back), "weight gradient")
    equal(dW[2], g.double().sum(0), "bias gradient")
    equal(dW[3], product(back, torch.cat([Ws.T, Wn.T])), "input gradient")
