"""The streamed bf16 products from the number of rows on from which each is taken, to the last bit: operands are -1, 0 and 1, so every partial sum is a whole number
that fp32 holds (below 2^24) and the results are right in whatever order they are added; those that are stored in bf16 are below 256 in size.  (At these numbers
of nodes a bound on rounding errors would let a lost slab of nodes pass.)  The names of the launches say which kernel ran."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MANY, TRANSFORM, STREAM = 65536, 98304, 1 << 20


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09887_amd import binding
    binding.lib()
    return binding


def signs(seed, n, f, pitch=None):
    """[n, f] in rows `pitch` apart, NaN between them."""
    g = torch.Generator("cuda").manual_seed(seed)
    t = torch.full((n, pitch or f), float("nan"), dtype=torch.bfloat16, device="cuda")[:, :f]
    t.copy_(torch.randint(-1, 2, (n, f), generator=g, device="cuda"))
    return t


def masked(g, h):
    """(-1, 0, 1, infinity and NaN in h) what a ReLU lets through of g."""
    h[::7, 1], h[::5, 0] = float("nan"), float("inf")
    return torch.where(h > 0, g, torch.zeros_like(g))


def product(a, b):
    return a.double() @ b.double()


def equal(got, want, what):
    if got.dtype == torch.bfloat16:
        assert want.abs().max() < 256
    assert torch.equal(got.double(), want), f"{what}: {int((got.double() != want).sum())} of {want.numel()}, the first at {(got.double() != want).nonzero()[0].tolist()}"


def streamed(B, call, what, also=()):
    """What `call` returns; its launches of these products are tiles of 256 rows."""
    B.tma_profile_begin(None)
    out = call()
    names = list(B.tma_profile_end())
    for w in what:
        assert [n for n in names if w in n and "_256x" in n], (w, names)
    for w in also:
        assert [n for n in names if w in n and "_256x" not in n], (w, names)
    return out


def ring(n):
    """Every node's one neighbour is the next, and the transpose."""
    nodes = torch.arange(n, dtype=torch.int32, device="cuda")
    return torch.arange(n + 1, dtype=torch.int32, device="cuda"), (nodes + 1) % n, (nodes - 1) % n, torch.ones(n, device="cuda")


# layers that aggregate first: what of forward, input and weight gradient is streamed
@pytest.mark.parametrize("n,fi,fo,relu,what", [
    (STREAM, 64, 128, False, ("fwd", "bwd_data", "bwd_weight")),            # 128 columns of input gradients
    (STREAM + 1, 48, 96, False, ("fwd", "bwd_data", "bwd_weight")),         # 96
    (STREAM + 1, 100, 120, True, ("fwd", "bwd_data", "bwd_weight")),        # the masked tile not filled; halves that end inside a slab
    (STREAM, 100, 120, False, ("fwd", "bwd_data", "bwd_weight")),
    (STREAM + 33, 72, 130, True, ("fwd", "bwd_data", "bwd_weight")),
    (STREAM, 64, 136, True, ("fwd", "bwd_weight")),
    (2 * MANY, 100, 300, False, ("fwd", "bwd_weight")),
    (2 * MANY + 1, 128, 100, False, ("bwd_data", "bwd_weight")),
    (4 * MANY + 255, 128, 100, True, ("bwd_data", "bwd_weight")),
    (MANY, 150, 128, True, ("bwd_data", "bwd_weight")),                     # a cut tile of 256
    (MANY + 1, 192, 384, False, ("fwd", "bwd_data", "bwd_weight")),         # odd numbers of 128 columns
])
def test_layer(B, n, fi, fo, relu, what):
    assert B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16)
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    rowptr, nxt, prev, inv = ring(n)
    X, Ws, Wn = signs(1, n, fi, (fi + 1) // 2 * 2 + 2), signs(2, fi, fo), signs(3, fi, fo)
    w, pitch = (Ws.float(), Wn.float()), (fo + 3) // 4 * 4 + 4
    g, h = signs(4, n, fo, pitch), signs(5, n, fo, pitch)
    M, out = streamed(B, lambda: B.tma_sage_layer_fwd(rowptr, nxt, inv, X, *w, torch.zeros(fo, device="cuda"), act,
                                                      Wt=B.tma_sage_prepare_weights_bf16(*w)), ["gemm_fwd"] if "fwd" in what else [])
    Z, W = torch.cat([X, X.roll(-1, 0)], 1), torch.cat([Ws, Wn])
    equal(out, product(Z, W).clamp(min=0) if relu else product(Z, W), "forward")
    d = masked(g, h) if relu else g
    dW = streamed(B, lambda: B.tma_sage_layer_bwd(rowptr, prev, inv, X, M, h, g, *w, act), ["gemm_" + p for p in what if p != "fwd"])
    equal(torch.cat(dW[:2]), product(Z.T, d), "weight gradient")
    equal(dW[2], d.double().sum(0), "bias gradient")
    equal(dW[3], product(d, Ws.T) + product(d, Wn.T).roll(1, 0), "input gradient")


# layers that transform first
@pytest.mark.parametrize("n,fi,fo,what", [
    (STREAM + 1, 100, 41, ("fwd", "bwd_data", "bwd_weight")),
    (STREAM, 128, 20, ("fwd", "bwd_data")),
    (2 * STREAM + 1, 64, 20, ("fwd", "bwd_data", "bwd_weight")),
    (2 * STREAM, 40, 5, ("fwd", "bwd_data")),
    (STREAM + 31, 256, 5, ("fwd", "bwd_data")),
    (STREAM, 128, 40, ("fwd", "bwd_data", "bwd_weight")),
    (STREAM // 2 + 1, 128, 32, ("fwd", "bwd_data")),
    (4 * MANY, 128, 47, ("fwd", "bwd_data")),
    (4 * MANY + 1, 256, 40, ("fwd", "bwd_data", "bwd_weight")),
    (2 * MANY + 1, 256, 47, ("fwd", "bwd_data", "bwd_weight")),
    (2 * MANY, 384, 140, ("fwd", "bwd_data", "bwd_weight")),
    (TRANSFORM + 1, 256, 47, ("fwd", "bwd_weight")),
])
def test_transform_first(B, n, fi, fo, what):
    assert not B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16)
    rowptr, nxt, prev, inv = ring(n)
    X, Ws, Wn, g = signs(1, n, fi, (fi + 1) // 2 * 2 + 2), signs(2, fi, fo), signs(3, fi, fo), signs(4, n, fo, (fo + 7) // 8 * 8)
    w = Ws.float(), Wn.float()
    M, out = streamed(B, lambda: B.tma_sage_layer_fwd(rowptr, nxt, inv, X, *w, torch.zeros(fo, device="cuda"), B.TMA_ACT_NONE),
                      ["gemm_tf_fwd"] if "fwd" in what else [])
    equal(out, product(X, Ws) + product(X, Wn).roll(-1, 0), "forward")
    dW = streamed(B, lambda: B.tma_sage_layer_bwd(rowptr, prev, inv, X, X, None, g, *w, B.TMA_ACT_NONE), ["gemm_tf_" + p for p in what if p != "fwd"])
    back = torch.cat([g, g.roll(1, 0)], 1)
    equal(torch.cat(dW[:2], 1), product(X.T, back), "weight gradient")
    equal(dW[2], g.double().sum(0), "bias gradient")
    equal(dW[3], product(back, torch.cat([Ws.T, Wn.T])), "input gradient")


# half of the input's width for the outputs, padded: no room for narrowed weights beside them
def test_transform_first_without_room(B):
    n, fi, fo = 2 * MANY, 128, 64
    assert not B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16)
    rowptr, nxt, _, inv = ring(n)
    X, Ws, Wn = signs(1, n, fi), signs(2, fi, fo), signs(3, fi, fo)
    out = streamed(B, lambda: B.tma_sage_layer_fwd(rowptr, nxt, inv, X, Ws.float(), Wn.float(), torch.zeros(fo, device="cuda"), B.TMA_ACT_NONE),
                   [], ["gemm_tf_fwd"])[1]
    equal(out, product(X, Ws) + product(X, Wn).roll(-1, 0), "forward")


@pytest.mark.parametrize("n,fi,fo,relu,what", [
    (STREAM, 150, 150, False, ("bwd_data", "bwd_weight")),
    (STREAM + 1, 150, 150, True, ("bwd_data", "bwd_weight")),
    (STREAM, 128, 97, True, ("bwd_weight",)),
    (STREAM // 2 + 1, 384, 66, True, ("bwd_data", "bwd_weight")),
    (2 * MANY, 256, 100, True, ("bwd_data", "bwd_weight")),
    (2 * MANY + 1, 300, 100, False, ("bwd_data", "bwd_weight")),
    (TRANSFORM, 256, 64, False, ("bwd_data", "bwd_weight")),
    (TRANSFORM + 1, 384, 256, True, ("bwd_data", "bwd_weight")),
    (MANY + 1, 600, 48, False, ("bwd_weight",)),
])
def test_dense(B, n, fi, fo, relu, what):
    pitch = (fo + 3) // 4 * 4
    X, W, g, h = signs(1, n, fi), signs(2, fi, fo), signs(3, n, fo, pitch), signs(4, n, fo, pitch)
    d = masked(g, h) if relu else g
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    dW, db, dX = streamed(B, lambda: B.tma_dense_bwd(X, h, g, W.float(), act)[:3], ["gemm_dense_" + p for p in what])
    equal(dX, product(d, W.T), "input gradient")
    equal(dW, product(X.T, d), "weight gradient")
    equal(db, d.double().sum(0), "bias gradient")


# a GCN layer that aggregates first scales the rows of its input gradient: by a half or one, on both sides of the sum over itself and its neighbour
@pytest.mark.parametrize("n,fi,fo,relu", [(TRANSFORM, 256, 256, False), (TRANSFORM + 1, 256, 256, True), (2 * MANY + 1, 264, 300, False)])
def test_gcn(B, n, fi, fo, relu):
    rowptr, _, prev, _ = ring(n)
    s = torch.where(torch.arange(n, device="cuda") % 3 == 1, 0.5, 1.0)
    pitch = (fo + 3) // 4 * 4
    X, M, W, g, h = signs(1, n, fi), signs(2, n, fi), signs(3, fi, fo), signs(4, n, fo, pitch), signs(5, n, fo, pitch)
    d = masked(g, h) if relu else g
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    dW, db, dH = streamed(B, lambda: B.tma_gcn_layer_bwd(rowptr, prev, s, X, M, h, g, W.float(), act), ["gemm_dense_bwd_data", "gemm_dense_bwd_weight"])[:3]
    P = product(d, W.T) * s[:, None]
    want = (P + P.roll(1, 0)) * s[:, None]
    assert P.abs().max() < 128      # (halves: 8 bits hold them)
    equal(dH, want.bfloat16().double(), "input gradient")
    equal(dW, product(M.T, d), "weight gradient")
    equal(db, d.double().sum(0), "bias gradient")


# a prepared copy of the weights takes the product to the streamed kernel; without one it is the other: of any values the same bits
@pytest.mark.parametrize("n,fi,fo", [(MANY, 128, 256), (MANY + 1, 150, 150), (2 * MANY, 100, 300), (STREAM + 7, 100, 120)])
def test_prepared_weights_change_no_bit(B, n, fi, fo):
    g = torch.Generator("cuda").manual_seed(1)
    X = torch.randn((n, fi), generator=g, device="cuda").bfloat16()
    w = [torch.randn(s, generator=g, device="cuda") for s in ((fi, fo), (fi, fo), (fo,))]
    rowptr, nxt, _, inv = ring(n)
    for act in (B.TMA_ACT_NONE, B.TMA_ACT_RELU):
        plain = streamed(B, lambda: B.tma_sage_layer_fwd(rowptr, nxt, inv, X, *w, act), [], ["gemm_fwd"])[1]
        ready = streamed(B, lambda: B.tma_sage_layer_fwd(rowptr, nxt, inv, X, *w, act, Wt=B.tma_sage_prepare_weights_bf16(*w[:2])), ["gemm_fwd"])[1]
        assert torch.equal(plain, ready)
