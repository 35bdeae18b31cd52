"""Gathers of rows whose 16-byte pieces do not fill their lane group, a multiple of four lanes: every remainder, with rows of no entry at the ends and between,
graphs without entries, matrices past 4 GB and sums on top of what is there.  Values are small whole numbers and a row's weight a power of two, so that results
are exact in both types."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_stream_exact import equal, product, ring, signs


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09887_amd import binding
    binding.lib()
    return binding


def graph(deg, rows, seed):
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.random.default_rng(seed).integers(0, rows, rowptr[-1]).astype(np.int32)
    return rowptr, col


def mean_is(B, rowptr, col, H, F):
    n = len(rowptr) - 1
    inv = torch.full((n,), 0.5, device="cuda")
    out = B.tma_mean_aggregate(torch.as_tensor(rowptr).cuda(), torch.as_tensor(col).cuda(), inv, H, out=torch.empty((n, F), dtype=H.dtype, device="cuda"))
    want = torch.zeros((n, F), dtype=torch.float64, device="cuda")
    want.index_add_(0, torch.as_tensor(np.repeat(np.arange(n), np.diff(rowptr))).cuda(), H[torch.as_tensor(col).cuda().long()].double())
    equal(out, want * 0.5, "mean")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("pieces", [1, 2, 3, 4, 5, 6, 7, 9, 13, 17, 21, 33, 63, 64])
def test_pieces(B, dtype, pieces):
    F, n = pieces * (4 if dtype == torch.float32 else 8), 517
    deg = np.array([0, 0, 1, 4, 0, 5, 3, 0, 8, 2, 130, 0, 7])[np.arange(n) % 13]
    deg[-3:] = 0
    H = torch.randint(-1, 2, (n, F), device="cuda").to(dtype)
    mean_is(B, *graph(deg, n, pieces), H, F)
    mean_is(B, np.zeros(n + 1, np.int32), np.zeros(0, np.int32), H, F)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_past_four_gigabytes(B, dtype):
    n, F, pitch = 9001, 40, 1 << (17 if dtype == torch.float32 else 18)   # rows half a megabyte apart
    H = torch.empty((n, pitch), dtype=dtype, device="cuda")[:, :F]
    H.copy_(torch.randint(-1, 2, (n, F), device="cuda"))
    mean_is(B, *graph(np.arange(n) % 11, n, 7), H, F)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fi", [8, 24, 40, 56, 72, 104])
def test_on_top(B, dtype, fi):
    n, fo = 300, 64
    rowptr, nxt, prev, inv = ring(n)
    X, Ws, Wn, g, h = (signs(s, *d).to(dtype) for s, d in enumerate([(n, fi), (fi, fo), (fi, fo), (n, fo), (n, fo)], 1))
    dH = B.tma_sage_layer_bwd(rowptr, prev, inv, X, X.roll(-1, 0).contiguous(), h, g, Ws.float(), Wn.float(), B.TMA_ACT_RELU)[3]
    d = torch.where(h > 0, g, torch.zeros_like(g))
    equal(dH[:, :fi], product(d, Ws.T) + product(d.roll(1, 0), Wn.T), "input gradient")
