"""The gradient rows that the transform-first backward scales and masks before it gathers them: widths of every remainder of a 16-byte piece, rows at odd pitches, NaN
between them, few and more than one round of blocks.  Whole numbers and a scale of a half: exact in both types."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_stream_exact import B, equal, masked, product, ring, signs  # noqa: F401


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("n,fo,pad", [(7, 1, 0), (300, 3, 1), (300, 7, 0), (300, 8, 1), (301, 9, 1), (300, 15, 2), (301, 16, 0), (300, 23, 1), (40000, 41, 0), (40001, 47, 3), (65000, 48, 0)])
def test_input_gradient(B, dtype, relu, n, fo, pad):
    fi = 128
    assert not B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16 if dtype == torch.bfloat16 else B.TMA_F32)
    rowptr, _, prev, inv = ring(n)

    def rows(seed, m, f, pitch):
        t = torch.full((m, pitch), float("nan"), dtype=dtype, device="cuda")[:, :f]
        t.copy_(signs(seed, m, f))
        return t

    X, Ws, Wn = rows(1, n, fi, fi), signs(2, fi, fo), signs(3, fi, fo)
    g, h = rows(4, n, fo, fo + pad), rows(5, n, fo, fo + pad)
    if relu and fo > 1:
        masked(g, h)
    d = torch.where(h > 0, g, torch.zeros_like(g)) if relu else g
    dH = B.tma_sage_layer_bwd(rowptr, prev, inv * 0.5, X, X, h if relu else None, g, Ws.float(), Wn.float(), B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE)[3]
    equal(dH[:, :fi], product(d, Ws.T) + 0.5 * product(d.roll(1, 0), Wn.T), "input gradient")
