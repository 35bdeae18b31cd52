"""Mean aggregation over rows of every length around the steps of four neighbours, alone and mixed in a wavefront, for pieces of a
row that fill a wavefront, share it by two, four and more, and rows at any pitch.  A sum of d fp32 values is within d roundings of the
sum of their sizes, its scale one more; a bf16 result is rounded once more, by 2^-8 of it at most."""
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


@pytest.mark.parametrize("dtype,F,pitch", [(torch.bfloat16, 512, 0), (torch.bfloat16, 256, 8), (torch.bfloat16, 128, 0), (torch.bfloat16, 48, 0),
                                           (torch.float32, 256, 0), (torch.float32, 128, 4), (torch.float32, 48, 0), (torch.float32, 8, 0)])
@pytest.mark.parametrize("lengths", ["4", "8", "mixed", "long"])
def test_mean(B, dtype, F, pitch, lengths):
    n, r = 1003, np.random.default_rng(F)
    deg = {"4": np.full(n, 4), "8": np.full(n, 8), "mixed": np.arange(n) % 14, "long": np.where(np.arange(n) % 97 == 5, 333, 12)}[lengths]
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = r.integers(0, n, rowptr[-1]).astype(np.int32)
    X = torch.as_tensor(r.standard_normal((n, F)).astype(np.float32)).to(dtype)
    H = torch.full((n, F + pitch), float("nan"), dtype=dtype, device="cuda")[:, :F]
    H.copy_(X)
    inv = np.where(deg > 0, 1.0 / np.maximum(deg, 1), 0.0).astype(np.float32)
    out = B.tma_mean_aggregate(torch.as_tensor(rowptr).cuda(), torch.as_tensor(col).cuda(), torch.as_tensor(inv).cuda(), H).double().cpu().numpy()
    rows, x = np.repeat(np.arange(n), deg), X.double().numpy()
    want, size = np.zeros((n, F)), np.zeros((n, F))
    np.add.at(want, rows, x[col])
    np.add.at(size, rows, np.abs(x[col]))
    want, size = want * inv[:, None], size * inv[:, None]
    bound = (deg[:, None] + 2) * 2.0 ** -24 * size + (2.0 ** -8 * np.abs(want) if dtype == torch.bfloat16 else 0.0) + 1e-30
    assert np.all(np.abs(out - want) <= bound)
