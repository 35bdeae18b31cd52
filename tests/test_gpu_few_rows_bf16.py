"""bf16 products of fewer than 65,536 rows on both sides of the line between tiles of 64 x 64 and wider ones.  Operands are -1, 0 and 1, so that the sums are exact;
results of forward and input gradient are one bf16 number where they stay below 256."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_stream_exact import B, equal, masked, product, ring, signs  # noqa: F401


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("n,fi,fo,relu", [(1, 8, 16, False), (63, 33, 64, True), (65, 64, 66, False), (5000, 100, 130, True), (16385, 40, 128, True), (16385, 64, 250, False),
                                          (27001, 24, 96, True), (40004, 64, 256, True), (65535, 72, 128, False), (65535, 36, 48, True)])
def test_layer(B, n, fi, fo, relu, prepared):
    assert B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16)
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    rowptr, nxt, prev, inv = ring(n)
    X, Ws, Wn = signs(1, n, fi, (fi + 7) // 8 * 8), signs(2, fi, fo), signs(3, fi, fo)
    g, h = signs(4, n, fo, (fo + 7) // 8 * 8), signs(5, n, fo, (fo + 7) // 8 * 8)
    w = Ws.float(), Wn.float()
    more = dict(Wt=B.tma_sage_prepare_weights_bf16(*w)) if prepared and fi % 4 == 0 else {}
    M, out = B.tma_sage_layer_fwd(rowptr, nxt, inv, X, *w, torch.zeros(fo, device="cuda"), act, **more)
    Z, W = torch.cat([X, X.roll(-1, 0)], 1), torch.cat([Ws, Wn])
    want = product(Z, W)
    equal(out[:, :fo], want.clamp(min=0) if relu else want, "forward")
    if relu:
        masked(g, h)
    d = torch.where(h > 0, g, torch.zeros_like(g)) if relu else g
    dWs, dWn, db, dH = B.tma_sage_layer_bwd(rowptr, prev, inv, X, M, h if relu else None, g, *w, act)
    equal(dWs, product(X.T, d), "self weights")
    equal(dWn, product(X.roll(-1, 0).T, d), "neighbour weights")
    equal(db, d.double().sum(0), "bias")
    equal(dH[:, :fi], product(d, Ws.T) + product(d.roll(1, 0), Wn.T), "input gradient")
