"""Where the streamed bf16 products put their columns: a lane holds an even one and its odd neighbour, which lie in two fragments, and the last 32 columns of
a tile of 96 the other way.  Operands are -1, 0 and 1 and biases whole numbers, so that every result is one bf16 number; every column has a bias of its own."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_stream_exact import MANY, equal, product, ring, signs, streamed


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09887_amd import binding
    binding.lib()
    return binding


# one tile of 96 cut inside its pairs of 64, inside its last 32, not at all; tiles of 128 and 256 cut at an odd and an even column
@pytest.mark.parametrize("fo", [66, 80, 95, 96, 97, 126, 128, 130, 191, 254, 256, 300])
def test_forward(B, fo):
    n, fi = MANY + 5, 64
    rowptr, nxt, _, inv = ring(n)
    X, Ws, Wn = signs(1, n, fi), signs(2, fi, fo), signs(3, fi, fo)
    bias = (torch.arange(fo, device="cuda") % 67 - 33).float()
    w = Ws.float(), Wn.float()
    _, out = streamed(B, lambda: B.tma_sage_layer_fwd(rowptr, nxt, inv, X, *w, bias, B.TMA_ACT_NONE, Wt=B.tma_sage_prepare_weights_bf16(*w)), ["gemm_fwd"])
    equal(out[:, :fo], product(torch.cat([X, X.roll(-1, 0)], 1), torch.cat([Ws, Wn])) + bias.double(), "forward")


# [dH | dM] in one row of tiles: halves that end at an odd column, inside a pair of fragments, with one
@pytest.mark.parametrize("fi,relu", [(128, False), (129, False), (130, False), (130, True), (160, True), (175, True), (192, False)])
def test_input_gradient(B, fi, relu):
    n, fo = MANY + 5, 128
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    rowptr, nxt, prev, inv = ring(n)
    X, Ws, Wn, g, h = signs(1, n, fi, fi + fi % 2), signs(2, fi, fo), signs(3, fi, fo), signs(4, n, fo), signs(5, n, fo)
    dH = streamed(B, lambda: B.tma_sage_layer_bwd(rowptr, prev, inv, X, X.roll(-1, 0), h, g, Ws.float(), Wn.float(), act), ["gemm_bwd_data"])[3]
    d = torch.where(h > 0, g, torch.zeros_like(g)) if relu else g
    equal(dH[:, :fi], product(d, Ws.T) + product(d.roll(1, 0), Wn.T), "input gradient")
