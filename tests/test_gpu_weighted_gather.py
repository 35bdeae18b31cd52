"""The gathers of the transform-first backward pass without an activation, dYn = Abar^T dZ with the rows of dZ weighted as they
come in or copied and scaled first (the device takes one by the graph's entries), and the gather of rows that are no multiples
of 16 bytes, with rows long enough to be cut into shares.  Row padding holds NaN throughout."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
sparse = pytest.importorskip("scipy.sparse")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09887_amd import binding
    binding.lib()
    return binding


def symmetric(n, degree, hubs, seed):
    """A symmetric graph of about n * degree entries, the first `hubs` nodes joined to every seventh node besides."""
    r = np.random.default_rng(seed)
    m = int(n * degree / 2)
    u, v = r.integers(0, n, m), r.integers(0, n, m)
    for h in range(hubs):
        u, v = np.concatenate([u, np.full(len(range(h, n, 7)), h)]), np.concatenate([v, np.arange(h, n, 7)])
    keep = u != v
    u, v = u[keep], v[keep]
    A = sparse.coo_matrix((np.ones(2 * len(u)), (np.concatenate([u, v]), np.concatenate([v, u]))), (n, n)).tocsr()
    A.data[:] = 1.0
    A.sort_indices()
    deg = np.diff(A.indptr)
    inv = np.where(deg > 0, 1.0 / np.maximum(deg, 1), 0.0).astype(np.float32)
    return A, inv, [torch.as_tensor(t).cuda() for t in (A.indptr.astype(np.int32), A.indices.astype(np.int32), inv)]


def nan_padded(B, t, dtype):
    p = B._padded(*t.shape, dtype, "cuda")
    p._base.fill_(float("nan"))
    return p.copy_(torch.as_tensor(t))


# fp32: weights from 2^16 to 2^18 rows of 32 elements and more; above, and in bf16 above 2^20, by entries up to n Fp / 8 or not
@pytest.mark.parametrize("n,degree,hubs,fi,fo,dtype", [
    (66000, 3, 2, 96, 47, "f32"), (66000, 0.5, 0, 64, 30, "f32"), (65536, 4, 1, 88, 41, "f32"), (66000, 3, 1, 48, 20, "f32"), (1500, 4, 3, 96, 47, "f32"), (1500, 4, 3, 88, 41, "f32"), (900, 0.5, 0, 64, 30, "f32"), (33000, 3, 1, 16, 7, "f32"), (70, 2, 1, 600, 300, "f32"),
    (265000, 2, 1, 72, 33, "f32"), (265000, 6, 1, 72, 33, "f32"),
    (1500, 4, 3, 96, 47, "bf16"), (1050000, 1.5, 1, 96, 41, "bf16"), (1050000, 8, 0, 96, 41, "bf16")])
def test_backward_without_activation(B, n, degree, hubs, fi, fo, dtype):
    T = torch.float32 if dtype == "f32" else torch.bfloat16
    A, inv, graph = symmetric(n, degree, hubs, n)
    r = np.random.default_rng(7)
    normal = lambda *s: torch.as_tensor(r.standard_normal(s, dtype=np.float32)).to(T).float().numpy()
    X, g, Ws, Wn = normal(n, fi), normal(n, fo), normal(fi, fo) * np.float32(0.125), normal(fi, fo) * np.float32(0.125)
    assert not B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_F32 if dtype == "f32" else B.TMA_BF16)
    x, dZ = nan_padded(B, X, T), nan_padded(B, g, T)
    w = [torch.as_tensor(t).cuda() for t in (Ws, Wn)]
    dWs, dWn, db, dH = B.tma_sage_layer_bwd(*graph, x, x, None, dZ, *w, B.TMA_ACT_NONE)
    dYn = A @ (inv[:, None].astype(np.float64) * g)
    # fp32: a few roundings per term, 2^-24 each.  bf16: dYn is stored with one rounding of 2^-9 per element, dH with another
    tol = 2e-6 if dtype == "f32" else 8e-3

    def close(got, want, what):
        got = got.double().cpu().numpy()
        err = np.linalg.norm(got - want) / np.linalg.norm(want)
        assert err <= tol, f"{what}: {err:.2e}"

    close(dWn, X.T.astype(np.float64) @ dYn, "neighbour weights")
    close(dWs, X.T.astype(np.float64) @ g, "self weights")
    close(db, g.sum(0, dtype=np.float64), "bias")
    rows = np.arange(n) if n < 2000 else np.unique(np.concatenate([np.arange(5), r.integers(0, n, 2000), [n - 1]]))
    close(dH[torch.as_tensor(rows).cuda()], g[rows].astype(np.float64) @ Ws.T + dYn[rows] @ Wn.T, "input gradient")


@pytest.mark.parametrize("f,dtype", [(47, "f32"), (90, "f32"), (255, "f32"), (90, "bf16"), (46, "bf16"), (254, "bf16")])
@pytest.mark.parametrize("n,degree", [(4000, 3), (300, 60)])
def test_mean_of_unaligned_rows_with_hubs(B, f, dtype, n, degree):
    """Rows side by side (no padding); the hubs' rows have 570 entries at 4,000 nodes."""
    T = torch.float32 if dtype == "f32" else torch.bfloat16
    A, inv, graph = symmetric(n, degree, 5, f)
    x = torch.randn((n, f), generator=torch.Generator().manual_seed(f)).to(T)
    M = B.tma_mean_aggregate(*graph, x.cuda(), out=torch.empty((n, f), dtype=T, device="cuda")).double().cpu().numpy()
    X, deg = x.double().numpy(), np.diff(A.indptr)[:, None]
    want, size = inv[:, None] * (A @ X), inv[:, None] * (A @ np.abs(X))
    bound = (deg + 2) * 2.0 ** -24 * size + (2.0 ** -8 * np.abs(want) if dtype == "bf16" else 0.0)
    assert np.all(np.abs(M - want) <= bound)
