"""A block's backward asks for as much room for partial sums as the layer's of as many rows: the weight gradient is the same product."""
import pytest

from paper_2305_09887_amd import binding as B


@pytest.mark.parametrize("n,fi,fo", [(65535, 128, 256), (65536, 128, 256), (400000, 256, 256), (100000, 100, 128), (1 << 20, 64, 96), (70000, 41, 300)])
@pytest.mark.parametrize("dtype", [B.TMA_F32, B.TMA_BF16])
def test_query(n, fi, fo, dtype):
    assert B.tma_sage_layer_aggregates_first(fi, fo, dtype)
    assert B.tma_sage_block_bwd_workspace_bytes(n, n + 5, 7, fi, fo, dtype, False) == B.tma_sage_layer_bwd_workspace_bytes(n, fi, fo, dtype, False)


@pytest.mark.parametrize("fi,fo", [(128, 256), (256, 256), (64, 64), (90, 41), (16, 300)])
@pytest.mark.parametrize("dtype", [B.TMA_F32, B.TMA_BF16])
@pytest.mark.parametrize("query", [B.tma_sage_block_bwd_workspace_bytes, B.tma_gcn_block_bwd_workspace_bytes])
def test_more_rows_need_no_less(query, fi, fo, dtype):
    """A trainer reserves once, for a block's most rows; every batch has fewer.  (From 65,536 rows on a bf16 query adds what the streamed product would make
    use of and can do without.)"""
    least = 0
    for n in list(range(1, 4200, 7)) + list(range(4200, 65536, 811)):
        room = query(n, n, n, fi, fo, dtype, True)
        assert room >= least, n
        least = room
