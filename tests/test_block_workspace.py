"""A block's backward asks for as much room for partial sums as the layer's of as many rows: the weight gradient is the same product."""
import pytest

from paper_2305_09887_amd import binding as B


@pytest.mark.parametrize("n,fi,fo", [(65535, 128, 256), (65536, 128, 256), (400000, 256, 256), (100000, 100, 128), (1 << 20, 64, 96), (70000, 41, 300)])
@pytest.mark.parametrize("dtype", [B.TMA_F32, B.TMA_BF16])
def test_query(n, fi, fo, dtype):
    assert B.tma_sage_layer_aggregates_first(fi, fo, dtype)
    assert B.tma_sage_block_bwd_workspace_bytes(n, n + 5, 7, fi, fo, dtype, False) == B.tma_sage_layer_bwd_workspace_bytes(n, fi, fo, dtype, False)
