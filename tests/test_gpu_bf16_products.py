"""The bf16 products at the edges of their main loops: every number of whole slabs from none to six, with and without a rest,
for operands fetched in groups of four and element by element, against 64 bits.

Operands are bf16 numbers (the weights too, which the kernel rounds), so a product of two is exact in fp32 and the sum is within
K 2^-24 of the sum of |a b|; a result that is stored in bf16 is rounded once more, by 2^-8 of it at most.
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


def bf16(seed, *shape):
    return torch.randn(shape, generator=torch.Generator().manual_seed(seed)).bfloat16()


def within(got, a, b, stored, what):
    got = got.double().cpu().numpy()
    a, b = a.double().numpy(), b.double().numpy()
    want = a @ b
    bound = a.shape[1] * 2.0 ** -24 * (np.abs(a) @ np.abs(b)) + (2.0 ** -8 * np.abs(want) if stored else 0.0) + 1e-30
    off = np.abs(got - want) / bound
    assert np.all(off <= 1.0), f"{what}: {off.max():.2f} of the bound"


K = [32 * s + rest for s in range(7) for rest in (0, 4, 13, 20) if 32 * s + rest > 0]


# k is F_in forward, F_out for the input gradient and n for the weight gradient; 100 columns take 128 wide tiles at 50,000 rows
@pytest.mark.parametrize("k", K)
@pytest.mark.parametrize("n,f", [(130, 60), (130, 37), (50000, 100), (50000, 101)])
def test_dense(B, n, f, k):
    X, W, g = bf16(1, n, k), bf16(2, k, f), bf16(3, n, f)
    x, w = X.cuda(), W.float().cuda()
    within(B.tma_dense_fwd(x, w, None, B.TMA_ACT_NONE), X, W, True, "forward")
    # the roles turned for the input gradient: [n, k] gradients, f inputs
    dX = B.tma_dense_bwd(g.cuda(), None, x, W.T.contiguous().float().cuda(), B.TMA_ACT_NONE, need_dbias=False)[2]
    within(dX, X, W, True, "input gradient")
    if n == 130:      # k rows
        A, G = bf16(4, k, 64 + f % 2), bf16(5, k, f)
        dW, db, _ = B.tma_dense_bwd(A.cuda(), None, G.cuda(), torch.zeros((A.shape[1], f), device="cuda"), B.TMA_ACT_NONE, need_dX=False)
        within(dW, A.T, G, False, "weight gradient")
        within(db.reshape(1, -1), torch.ones((1, k)), G, False, "bias gradient")


@pytest.mark.parametrize("k,fo", [(k, fo) for k in K[::3] for fo in (48, 128, 200) if 2 * ((fo + 7) // 8 * 8) > k])
def test_two_weight_matrices(B, k, fo):
    """The aggregate-first layer, [H | M] against both weights; every node has one neighbour, so M is a copy of a row."""
    n = 50000 if fo == 128 else 300
    assert B.tma_sage_layer_aggregates_first(k, fo, B.TMA_BF16)
    X, Ws, Wn = bf16(1, n, k), bf16(2, k, fo), bf16(3, k, fo)
    ring = torch.arange(n, dtype=torch.int32)
    rowptr, inv = torch.arange(n + 1, dtype=torch.int32), torch.ones(n)
    M, out = B.tma_sage_layer_fwd(rowptr.cuda(), ((ring + 1) % n).cuda(), inv.cuda(), X.cuda(), Ws.float().cuda(), Wn.float().cuda(),
                                  torch.zeros(fo, device="cuda"), B.TMA_ACT_NONE)
    assert torch.equal(M.cpu(), X.roll(-1, 0))
    within(out, torch.cat([X, X.roll(-1, 0)], 1), torch.cat([Ws, Wn]), True, "forward")
