"""Long rows among those of a sampled block that are sources only: whether one is shared out depends on these rows' own mean, not on the entries of the rows
before them.  One entry of 2^24 in front of ones shows it: added one after the other in fp32 every one is lost, in shares only those of the first."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_stream_exact import B  # noqa: F401


@pytest.mark.parametrize("gcn", [False, True])
def test_long_row_of_a_tail(B, gcn):
    n_dst, n_tail, F, taken = 512, 16, 16, 40
    n_src, hub = n_dst + n_tail, n_dst + 5
    near = (np.arange(n_dst)[:, None] + np.arange(1, taken + 1)) % n_dst        # 20,480 entries of the first rows' transpose, 512 of the tail's
    cols = np.concatenate([near, np.full((n_dst, 1), hub)], 1).astype(np.int32)
    rowptr = torch.arange(n_dst + 1, dtype=torch.int32).cuda() * (taken + 1)
    rows = torch.arange(n_dst, dtype=torch.int32).repeat_interleave(taken + 1).cuda()
    cols, items, one = torch.as_tensor(cols.ravel()).cuda(), n_dst * (taken + 1), torch.ones(n_dst, device="cuda")
    g = torch.ones((n_dst, F), device="cuda")
    g[0] = 2.0 ** 24
    H, M, dH, W, zero = (torch.zeros((r, F), device="cuda") for r in (n_src, n_dst, n_src, F, F))
    W.fill_diagonal_(1)
    db = torch.empty(F, device="cuda")
    if gcn:
        B.tma_gcn_block_bwd(n_dst, n_src, items, rowptr, cols, rows, one, M, None, g, W, B.TMA_ACT_NONE, torch.empty_like(W), db, dH_out=dH)
    else:
        B.tma_sage_block_bwd(n_dst, n_src, items, rowptr, cols, rows, one, H, M, None, g, zero, W, B.TMA_ACT_NONE, torch.empty_like(W), torch.empty_like(W), db, dH_out=dH)
    assert torch.equal(dH[n_dst:hub], torch.zeros_like(dH[n_dst:hub])) and torch.equal(dH[hub + 1:], torch.zeros_like(dH[hub + 1:]))
    # 64 shares of eight entries: the seven ones of the first are lost
    assert torch.equal(dH[hub], torch.full((F,), 2.0 ** 24 + n_dst - 8, device="cuda"))
