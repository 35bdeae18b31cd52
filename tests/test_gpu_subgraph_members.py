"""The extraction's list of a tile's members (2,048 nodes): none, one, all, runs that end at a tile's edges, four and more to a thread; room for exactly them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle
from paper_2305_09887_amd import synth


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09887_amd import binding
    binding.lib()
    return binding


MEMBERS = {"all": lambda i, n: i >= 0, "first": lambda i, n: i == 0, "last": lambda i, n: i == n - 1, "third": lambda i, n: i % 3 == 1, "one tile": lambda i, n: i // 2048 == 1,
           "to the edge": lambda i, n: (i >= 2040) & (i < 2048), "thinned": lambda i, n: (i // 700) % 2 == 0}


@pytest.mark.parametrize("n", [33, 2047, 2048, 2049, 4096, 6150])
@pytest.mark.parametrize("members", list(MEMBERS))
@pytest.mark.parametrize("spare", [0, 9])
def test_members(B, n, members, spare):
    rowptr, colidx = synth.uniform_graph(n, 4 * n, seed=n)
    part = np.where(MEMBERS[members](np.arange(n), n), 2, 1).astype(np.int32)
    want = oracle.induced_subgraph(rowptr, colidx, part, 2)
    n_loc, nnz = len(want["l2g"]), len(want["colidx"])
    d = lambda a: torch.as_tensor(a).cuda()
    out = B.tma_induced_subgraph_async(d(rowptr), d(colidx), d(part), 2, max(n_loc + spare, 1), max(nnz + spare, 1))
    assert out["sizes"].cpu().tolist() == [n_loc, nnz]
    assert np.array_equal(out["g2l"][:n].cpu().numpy(), want["g2l"])
    assert np.array_equal(out["l2g"][:n_loc].cpu().numpy(), want["l2g"])
    assert np.array_equal(out["rowptr"][:n_loc + 1].cpu().numpy(), want["rowptr"])
    assert np.array_equal(out["colidx"][:nnz].cpu().numpy(), want["colidx"])
