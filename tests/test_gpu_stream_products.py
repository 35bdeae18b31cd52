"""The bf16 products over many rows at the edges of their tiles and slabs of 32 k-values (32 nodes in a weight gradient): the last tile of 256 rows whole, cut and
of one row; widths of every tile; halves that end at every kind of place of a slab; padding that holds NaN and must reach nothing.
Bounds as in test_gpu_bf16_products.py."""
import pytest

from test_gpu_bf16_products import B, bf16, within  # noqa: F401  (B: the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def inside(a, pitch, before):
    """`a` on the GPU at an offset of `before` elements, rows `pitch` apart, NaN around and between the rows."""
    n, f = a.shape
    t = torch.full((before + n * pitch + 8,), float("nan"), dtype=a.dtype, device="cuda")
    view = t[before:before + n * pitch].view(n, pitch)[:, :f]
    view.copy_(a)
    return view


def ring(n):
    """Every node's one neighbour is the next: aggregating rolls the rows."""
    nodes = torch.arange(n, dtype=torch.int32)
    return torch.arange(n + 1, dtype=torch.int32).cuda(), ((nodes + 1) % n).cuda(), torch.ones(n, device="cuda")


def even(x):
    return (x + 1) // 2 * 2


# aggregated first: forward [H | M] [W_self ; W_neigh] + b, backward dZ [W_self^T | W_neigh^T] with and without the mask
@pytest.mark.parametrize("n,fi,fo", [(65536, 64, 72), (65537, 32, 96), (65792, 96, 128), (65535 + 256, 128, 256), (65600, 32, 70), (65600, 160, 98),
                                     (65664, 16, 130), (65540, 150, 150), (65540, 66, 300), (65540, 200, 258), (65601, 100, 256)])
@pytest.mark.parametrize("relu", [False, True])
def test_layer(B, n, fi, fo, relu):
    assert B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16)
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    rowptr, col, inv = ring(n)
    X, Ws, Wn, g = bf16(1, n, fi), bf16(2, fi, fo), bf16(3, fi, fo), bf16(4, n, fo)
    pitch = even(fi) + 2
    H = inside(X, pitch, 2)
    M, out = inside(torch.zeros_like(X), pitch, 4), inside(torch.zeros(n, fo).bfloat16(), even(fo) + 4, 2)
    w = Ws.float().cuda(), Wn.float().cuda()
    B.tma_sage_layer_fwd(rowptr, col, inv, H, *w, torch.zeros(fo, device="cuda"), act, M_out=M, Hnext_out=out,
                         Wt=B.tma_sage_prepare_weights_bf16(*w))
    Z = torch.cat([X, X.roll(-1, 0)], 1), torch.cat([Ws, Wn])
    if not relu:
        within(out, *Z, True, "forward")
    h = bf16(5, n, fo)
    h[::7, 1], h[::5, 0] = float("nan"), float("inf")      # not above zero, and above
    h[::3, fo - 1] = 0.0
    d = torch.where(h > 0, g, torch.zeros(()).bfloat16()) if relu else g
    dH = inside(torch.zeros_like(X), pitch, 2)
    back = torch.zeros(n + 1, dtype=torch.int32, device="cuda")          # no entries: dH is dZ W_self^T
    dW = B.tma_sage_layer_bwd(back, col, inv, H, M, inside(h, even(fo) + 4, 2), inside(g, even(fo) + 4, 2), *w, act, dH_out=dH)
    within(dH, d, Ws.T, True, "input gradient")
    within(torch.cat(dW[:2]), Z[0].T, d, False, "weight gradient")
    within(dW[2].reshape(1, -1), torch.ones((1, n)).bfloat16(), d, False, "bias gradient")
    into = (torch.arange(n, dtype=torch.int32) - 1) % n                  # the transposed ring
    B.tma_sage_layer_bwd(rowptr, into.int().cuda(), inv, H, M, inside(h, even(fo) + 4, 2), inside(g, even(fo) + 4, 2), *w, act, dH_out=dH)
    # (two roundings more on the way: of dZ W_neigh^T and of the first part of the sum)
    got, a, b = dH.double().cpu(), torch.cat([d, d.roll(1, 0)], 1).double(), torch.cat([Ws.T, Wn.T]).double()
    bound = 3 * 2.0 ** -8 * ((d.double() @ Ws.T.double()).abs() + (d.roll(1, 0).double() @ Wn.T.double()).abs()) + 2.0 ** -20 * (a.abs() @ b.abs()) + 1e-30
    assert torch.all((got - a @ b).abs() <= bound)


# transformed first: H [W_self | W_neigh], and [dZ | dYn] [W_self | W_neigh]^T, with outputs of odd width too
@pytest.mark.parametrize("n,fi,fo", [(98304, 256, 47), (98305, 128, 41), (98560, 64, 5), (98400, 96, 48), (98432, 96, 33), (98500, 320, 140), (65570, 264, 20),
                                     (98310, 128, 50)])
def test_transform_first(B, n, fi, fo):
    assert not B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16)
    rowptr, col, inv = ring(n)
    X, Ws, Wn, g = bf16(1, n, fi), bf16(2, fi, fo), bf16(3, fi, fo), bf16(4, n, fo)
    w = Ws.float().cuda(), Wn.float().cuda()
    pitch = even(fi) + 2
    H = inside(X, pitch, 2)
    out = B.tma_sage_layer_fwd(rowptr, col, inv, H, *w, torch.zeros(fo, device="cuda"), B.TMA_ACT_NONE)[1]
    x, y = X.double() @ Ws.double(), X.roll(-1, 0).double() @ Wn.double()
    sums = X.abs().double() @ Ws.abs().double() + X.roll(-1, 0).abs().double() @ Wn.abs().double()
    assert torch.all((out.double().cpu() - x - y).abs() <= 2 * 2.0 ** -8 * (x.abs() + y.abs()) + 2.0 ** -20 * sums + 1e-30)
    into = (torch.arange(n, dtype=torch.int32) - 1) % n
    dH = inside(torch.zeros_like(X), pitch, 2)
    room = inside(g, (fo + 7) // 8 * 8, 8)
    dW = B.tma_sage_layer_bwd(rowptr, into.int().cuda(), inv, H, H, None, room, *w, B.TMA_ACT_NONE, dH_out=dH)
    within(torch.cat(dW[:2], 1), X.T, torch.cat([g, g.roll(1, 0)], 1), False, "weight gradient")
    within(dW[2].reshape(1, -1), torch.ones((1, n)).bfloat16(), g, False, "bias gradient")
    within(dH, torch.cat([g, g.roll(1, 0)], 1), torch.cat([Ws.T, Wn.T]), True, "input gradient")


# single-operand backward products, with the row scale that a GCN layer puts into its input gradient left out
@pytest.mark.parametrize("n,fi,fo", [(98304, 256, 64), (98305, 256, 47), (98400, 130, 256), (98320, 264, 130), (98310, 128, 258),
                                     (65600, 264, 66), (65570, 600, 48)])
@pytest.mark.parametrize("relu", [False, True])
def test_dense_backward(B, n, fi, fo, relu):
    X, W, g, h = bf16(1, n, fi), bf16(2, fi, fo), bf16(3, n, fo), bf16(4, n, fo)
    h[::7, 1], h[::3, fo - 1] = float("nan"), 0.0
    pitch = (fo + 3) // 4 * 4
    x, w = X.cuda(), W.float().cuda()
    dW, db, dX = B.tma_dense_bwd(x, inside(h, pitch, 4), inside(g, pitch, 4), w, B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE)[:3]
    d = torch.where(h > 0, g, torch.zeros(()).bfloat16()) if relu else g
    within(dX, d, W.T, True, "input gradient")
    within(dW, X.T, d, False, "weight gradient")
    within(db.reshape(1, -1), torch.ones((1, n)).bfloat16(), d, False, "bias gradient")


# a workspace below what the query asks for: fewer ranges of nodes, the same sums; far below: an error
def test_smaller_workspace(B):
    n, fi, fo = 65600, 128, 256
    X, M, g = bf16(1, n, fi), bf16(2, n, fi), bf16(3, n, fo)
    rowptr, col, inv = ring(n)
    w = torch.zeros(fi, fo, device="cuda"), torch.zeros(fi, fo, device="cuda")
    asked = B.tma_sage_layer_bwd_workspace_bytes(n, fi, fo, B.TMA_BF16, False)
    for share in (1.0, 0.6):
        ws = torch.empty(int(asked * share) // 256 * 256, dtype=torch.uint8, device="cuda")
        dW = B.tma_sage_layer_bwd(rowptr, col, inv, X.cuda(), M.cuda(), None, g.cuda(), *w, B.TMA_ACT_NONE, need_dH=False, ws=ws)
        within(torch.cat(dW[:2]), torch.cat([X, M], 1).T, g, False, "weight gradient")
        within(dW[2].reshape(1, -1), torch.ones((1, n)).bfloat16(), g, False, "bias gradient")
    with pytest.raises(B.TmaError):
        B.tma_sage_layer_bwd(rowptr, col, inv, X.cuda(), M.cuda(), None, g.cuda(), *w, B.TMA_ACT_NONE, need_dH=False, ws=ws[:1 << 20])


# a block's weight gradient, in the workspace that the query asks for, in less, and in less than it needs
def test_block_workspace(B):
    n, fi, fo = 65600, 128, 256
    X, M, g = bf16(1, n, fi), bf16(2, n, fi), bf16(3, n, fo)
    empty = torch.zeros(n + 1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    w = torch.zeros(fi, fo, device="cuda"), torch.zeros(fi, fo, device="cuda")
    dW = torch.empty(fi, fo, device="cuda"), torch.empty(fi, fo, device="cuda"), torch.empty(fo, device="cuda")
    asked = B.tma_sage_block_bwd_workspace_bytes(n, n, 0, fi, fo, B.TMA_BF16, False)

    def call(ws):
        B.tma_sage_block_bwd(n, n, 0, *empty, torch.ones(n, device="cuda"), X.cuda(), M.cuda(), None, g.cuda(), *w, B.TMA_ACT_NONE, *dW, ws=ws)

    for share in (1.0, 0.6):
        ws = torch.empty(int(asked * share) // 256 * 256, dtype=torch.uint8, device="cuda")
        call(ws)
        within(torch.cat(dW[:2]), torch.cat([X, M], 1).T, g, False, "weight gradient")
        within(dW[2].reshape(1, -1), torch.ones((1, n)).bfloat16(), g, False, "bias gradient")
    with pytest.raises(B.TmaError):
        call(ws[:1 << 20])
