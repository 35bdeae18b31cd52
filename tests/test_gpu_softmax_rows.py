"""Softmax loss and its gradient for every number of columns a lane can hold and more, rows around what a block walks over, and rows of infinities and NaN.
A probability is an exponential (two roundings and two of its difference, which is at most 100 here, so 100 2^-24 of it) over a sum of C, each rounded once
per step of its sum: within (C / 16 + 112) 2^-24 of itself.  The difference to the label, 1 / n and their product are three more roundings, of p + 1 at the
label at most; a bf16 result is rounded once more.  The loss is a mean of at most 2^-24 (C / 16 + 112) off a row's and of its own sum."""
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


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("C", [1, 2, 15, 16, 17, 31, 32, 33, 41, 47, 48, 49, 64, 65, 130])
@pytest.mark.parametrize("n", [1, 15, 17, 1000, 32768 + 31])
def test_rows(B, dtype, C, n):
    g = torch.Generator().manual_seed(C + n)
    Z = torch.full((n, C + C % 2), float("nan"), dtype=dtype, device="cuda")[:, :C]
    Z.copy_(torch.randn((n, C), generator=g) * 5)
    y = torch.randint(0, C, (n,), generator=g, dtype=torch.int32).cuda()
    loss, dZ = B.tma_softmax_ce(Z, y)
    z = Z.double()
    p = torch.softmax(z, 1)
    hot = torch.nn.functional.one_hot(y.long(), C).double()
    want = (p - hot) / n
    bound = ((C / 16 + 112) * 2.0 ** -24 * p + 3 * 2.0 ** -24 * (p + hot)) / n + (2.0 ** -8 * want.abs() if dtype == torch.bfloat16 else 0.0) + 1e-38
    assert bool(((dZ[:, :C].double() - want).abs() <= bound).all())
    terms = torch.logsumexp(z, 1) - z.gather(1, y.long()[:, None])[:, 0]
    size = (terms.abs() + z.abs().amax(1) + 1).mean()
    assert abs(float(loss) - float(terms.mean())) <= (C / 16 + 112 + n ** 0.5) * 2.0 ** -24 * float(size) + 1e-38


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("C", [5, 16, 33, 47, 64, 70])
def test_infinities(B, dtype, C):
    Z = torch.zeros((6, C), dtype=dtype, device="cuda")
    Z[0, 0], Z[1, C - 1], Z[2], Z[3, :2], Z[4, C // 2] = -float("inf"), float("inf"), -float("inf"), -float("inf"), float("nan")
    y = torch.full((6,), C - 1, dtype=torch.int32, device="cuda")
    dZ = B.tma_softmax_ce(Z, y)[1][:, :C].double()
    want = (torch.softmax(Z.double(), 1) - torch.nn.functional.one_hot(y.long(), C)) / 6
    assert torch.equal(dZ.isnan(), want.isnan())
    assert torch.allclose(dZ[~want.isnan()], want[~want.isnan()], rtol=2.0 ** -7 if dtype == torch.bfloat16 else 1e-5, atol=0)
